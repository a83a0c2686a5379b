// rowsort.hip -- lexicographic row order of tables (Sec. 4.3: results merged
// to distinct values; the canonical order of every result) by merge sort of
// packed keys, for one table or for the tables of a whole batch round.
//
// A row's columns, at their known bit widths, are concatenated into W 64-bit
// words (W <= 4); rows that compare equal are the same row, so the sort needs
// neither stability nor a permutation, and the sorted rows are unpacked from
// the keys: no gather.
//   tile sort  a workgroup packs its tile of rows, each thread sorts kVT keys
//              in registers (odd-even transposition, Habermann), then runs are merged pairwise in LDS, every
//              thread finding the kVT keys it produces by a binary search
//              along its diagonal (the merge path of Green, McColl and Bader,
//              "GPU merge path").  A table of one tile is written out here;
//   rank merge tables of up to 114,688 rows: a launch puts eight runs together
//              (row_rank_merge);
//   radix      one-word keys, many rows for their bits: the radix passes of
//              sort.hip on the packed keys, then unpacked (radix_better); such
//              tables of a batch round all together (radix_bits_of_round);
//   merge      other larger ones: one launch per doubling of the run length: a workgroup
//              produces kMergeTile rows, finds its two diagonals with a
//              64-way search by a wave each, and merges out of LDS.  The last
//              level writes the table's columns.
//
// Bound: a level reads and writes 8 W bytes a row from cache or HBM; below
// about a million rows it is bound by the latency of the diagonal searches
// and of the launch.  kVT is odd, so that the blocked accesses of a wave's
// lanes fall on different LDS banks.  Why merge sort and not an LSD radix
// sort of row numbers (three launches per 8 key bits, and the rows gathered at
// the end): see the sizes measured at rows_mergeable() below.
#include "batch.hpp"
#include "compact.hpp"

#include <algorithm>

namespace tid {

void exclusive_scan_async(tid_ctx *ctx, const uint32_t *in, uint64_t n, uint64_t *out);
bool sort_words(tid_ctx *ctx, uint64_t *k0, uint64_t *k1, uint64_t n, int bits);

namespace {

constexpr int kVT = 7;                       // keys per thread
constexpr int kMergeBlock = 256;
constexpr uint32_t kMergeTile = kMergeBlock * kVT;
constexpr int kMaxWords = 4;

// threads of a tile sort: the tile's keys, 8 W bytes each, stay in LDS
constexpr int tile_block(int words) { return words <= 2 ? 1024 : 512; }
constexpr uint32_t tile_rows(int words) { return (uint32_t)tile_block(words) * kVT; }

constexpr int kRankBlock = 256;
constexpr uint32_t kWays = 8;                // runs that row_rank_merge puts together
constexpr uint32_t kRankPart = 2560;         // rows of other runs in LDS (about 7 * kRankBlock)
constexpr int kSmallTile = 256;              // threads of a tile sort before it
static_assert(kSmallTile * kVT % kRankBlock == 0 && kRankBlock == 2 * kWays * 16, "");

struct RowJob {
    const uint32_t *in[TID_MAX_COLS];
    uint32_t *out[TID_MAX_COLS];
    uint64_t *key[2];              // W planes of n words each, double buffered
    uint64_t *count;               // DISTINCT: the row count (else null)
    uint32_t *kept;                // DISTINCT, last merge level: a tile's first-of-equals
    uint32_t n;
    uint32_t tile0, mtile0;        // the job's first tile in the two kinds of launch
    int32_t levels;                // merge launches the job takes part in
    uint64_t tag;                  // radix sort of several tables: their order, above the key
    int16_t ncols;
    int16_t distinct;              // one tile: keep the first of equal rows; several: the
                                   // last row_merge keeps them, tile by tile; the last
                                   // row_rank_merge leaves the sorted keys
    uint8_t word[TID_MAX_COLS];    // bit position of a column from the key's end:
    uint8_t shift[TID_MAX_COLS];   // word (0 = least significant) and bit in it
    uint8_t width[TID_MAX_COLS];   // bits (0: a column of zeros)
};

__device__ __forceinline__ uint32_t gload(const uint32_t *p) {
    return *(const __attribute__((address_space(1))) uint32_t *)p;
}
__device__ __forceinline__ uint64_t gload(const uint64_t *p) {
    return *(const __attribute__((address_space(1))) uint64_t *)p;
}
template <class T>
__device__ __forceinline__ void gstore(T *p, T v) {
    *(__attribute__((address_space(1))) T *)p = v;
}

template <int W>
struct Key {
    uint64_t w[W];  // most significant first
};

template <int W>
__device__ __forceinline__ bool key_less(const Key<W> &a, const Key<W> &b) {
#pragma unroll
    for (int x = 0; x < W - 1; ++x)
        if (a.w[x] != b.w[x]) return a.w[x] < b.w[x];
    return a.w[W - 1] < b.w[W - 1];
}

template <int W>
__device__ __forceinline__ Key<W> lds_key(const uint64_t *s, uint32_t stride, uint32_t i) {
    Key<W> k;
#pragma unroll
    for (int x = 0; x < W; ++x) k.w[x] = s[x * stride + i];
    return k;
}

template <int W>
__device__ __forceinline__ void lds_put(uint64_t *s, uint32_t stride, uint32_t i,
                                        const Key<W> &k) {
#pragma unroll
    for (int x = 0; x < W; ++x) s[x * stride + i] = k.w[x];
}

// kVT rows of a tile.  Which rows a thread starts with does not matter: in a
// whole tile they are BLOCK apart, so that a column's loads are coalesced; in
// the last one they are consecutive, so that the rows fill the first threads.
// A column's loads are in flight together (a row after the other they were most
// of a small tile's time: 15.8 us for small tiles of two columns, now 14.3).
// Past the end the largest key (a row holding that key is the same key, so
// either may be written).
template <int W, int BLOCK>
__device__ __forceinline__ void pack_rows(const RowJob &p, uint32_t t0, uint32_t cnt,
                                          Key<W> (&k)[kVT]) {
    const bool whole = cnt == (uint32_t)BLOCK * kVT;
    const uint32_t i0 = whole ? threadIdx.x : threadIdx.x * kVT, step = whole ? BLOCK : 1;
#pragma unroll
    for (int v = 0; v < kVT; ++v)
#pragma unroll
        for (int x = 0; x < W; ++x) k[v].w[x] = i0 + v * step < cnt ? 0ull : ~0ull;
    for (int c = 0; c < p.ncols; ++c) {
        if (p.width[c] == 0) continue;
        const uint32_t *col = p.in[c] + t0;
        const int lw = p.word[c], sh = p.shift[c];
        const bool over = sh + p.width[c] > 64;
        uint32_t val[kVT];
#pragma unroll
        for (int v = 0; v < kVT; ++v) val[v] = gload(col + min(i0 + v * step, cnt - 1));
#pragma unroll
        for (int v = 0; v < kVT; ++v)
#pragma unroll
            for (int x = 0; x < W; ++x) {  // static indices: the keys stay in registers
                if (W - 1 - x == lw) k[v].w[x] |= (uint64_t)val[v] << sh;
                if (W - 1 - x == lw + 1 && over) k[v].w[x] |= (uint64_t)val[v] >> (64 - sh);
            }
    }
}

// column c of the key whose word x (most significant first) is word(x)
template <int W, class Word>
__device__ __forceinline__ uint32_t column_of(const RowJob &p, int c, const Word &word) {
    const int b = p.width[c];
    if (b == 0) return 0;
    const int lw = p.word[c], sh = p.shift[c];
    uint64_t v = word(W - 1 - lw) >> sh;
    if (sh + b > 64) v |= word(W - 2 - lw) << (64 - sh);
    return (uint32_t)(v & ((1ull << b) - 1));
}

// how many of the first d merged keys come from A (ties from A first): A is
// the na keys at a, B the nb keys at b of LDS plane s
template <int W>
__device__ __forceinline__ uint32_t lds_diagonal(const uint64_t *s, uint32_t stride, uint32_t a,
                                                 uint32_t na, uint32_t b, uint32_t nb,
                                                 uint32_t d) {
    uint32_t lo = d > nb ? d - nb : 0, hi = min(d, na);
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (!key_less(lds_key<W>(s, stride, b + d - 1 - mid), lds_key<W>(s, stride, a + mid)))
            lo = mid + 1;
        else
            hi = mid;
    }
    return lo;
}

// the next kVT keys of the merge of s[a, a1) and s[b, b1)
template <int W>
__device__ __forceinline__ void serial_merge(const uint64_t *s, uint32_t stride, uint32_t a,
                                             uint32_t a1, uint32_t b, uint32_t b1,
                                             Key<W> (&out)[kVT]) {
    Key<W> ka{}, kb{};
    if (a < a1) ka = lds_key<W>(s, stride, a);
    if (b < b1) kb = lds_key<W>(s, stride, b);
#pragma unroll
    for (int v = 0; v < kVT; ++v) {
        const bool from_a = b >= b1 || (a < a1 && !key_less(kb, ka));
        a += from_a ? 1u : 0u;
        b += from_a ? 0u : 1u;
        const uint32_t at = from_a ? a : b;
        const bool more = at < (from_a ? a1 : b1);
#pragma unroll
        for (int x = 0; x < W; ++x) {  // word by word: the keys stay in registers
            out[v].w[x] = from_a ? ka.w[x] : kb.w[x];
            const uint64_t w = more ? s[x * stride + at] : 0ull;
            ka.w[x] = from_a ? w : ka.w[x];
            kb.w[x] = from_a ? kb.w[x] : w;
        }
    }
}

// rows [0, cnt) of LDS plane s to the job's columns, from row `at` on
template <int W, int BLOCK>
__device__ __forceinline__ void write_columns(const RowJob &p, const uint64_t *s, uint32_t stride,
                                              uint32_t cnt, uint32_t at) {
    for (int c = 0; c < p.ncols; ++c) {
        uint32_t *out = p.out[c] + at;
        for (uint32_t i = threadIdx.x; i < cnt; i += BLOCK)
            gstore(out + i, column_of<W>(p, c, [&](int x) { return s[x * stride + i]; }));
    }
}

template <int W, int BLOCK>
__device__ __forceinline__ void write_keys(const RowJob &p, uint64_t *dst, const uint64_t *s,
                                           uint32_t stride, uint32_t cnt, uint32_t at) {
#pragma unroll
    for (int x = 0; x < W; ++x)
        for (uint32_t i = threadIdx.x; i < cnt; i += BLOCK)
            gstore(dst + (uint64_t)x * p.n + at + i, s[x * stride + i]);
}

// the job of a tile: the last one whose first tile is <= tile
template <bool MERGE>
__device__ __forceinline__ int row_job_of(const RowJob *jobs, int J, uint32_t tile) {
    int lo = 0, hi = J - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if ((MERGE ? jobs[mid].mtile0 : jobs[mid].tile0) <= tile) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

template <int W, int BLOCK>
__device__ __forceinline__ void tile_sort_body(const RowJob &p, uint32_t tile) {
    constexpr uint32_t TILE = (uint32_t)BLOCK * kVT;
    constexpr int NW = BLOCK / dev::kWave;
    extern __shared__ __attribute__((aligned(16))) uint64_t s_tile[];
    __shared__ uint32_t s_w[NW];
    const uint32_t tid = threadIdx.x;
    const uint32_t t0 = tile * TILE;
    const uint32_t cnt = min(TILE, p.n - t0);
    Key<W> k[kVT];
    pack_rows<W, BLOCK>(p, t0, cnt, k);
#pragma unroll
    for (int r = 0; r < kVT; ++r)  // odd-even transposition
#pragma unroll
        for (int v = r & 1; v + 1 < kVT; v += 2) {
            const bool swap = key_less(k[v + 1], k[v]);
#pragma unroll
            for (int x = 0; x < W; ++x) {
                const uint64_t lo = swap ? k[v + 1].w[x] : k[v].w[x];
                k[v + 1].w[x] = swap ? k[v].w[x] : k[v + 1].w[x];
                k[v].w[x] = lo;
            }
        }
    // runs of `run` threads merge pairwise while one run is shorter than the tile
    for (uint32_t run = 1; run * kVT < cnt; run *= 2) {
#pragma unroll
        for (int v = 0; v < kVT; ++v) lds_put(s_tile, TILE, tid * kVT + v, k[v]);
        __syncthreads();
        const uint32_t first = tid & ~(2 * run - 1);
        const uint32_t a = first * kVT, len = run * kVT, b = a + len;
        const uint32_t d = (tid - first) * kVT;
        const uint32_t da = lds_diagonal<W>(s_tile, TILE, a, len, b, len, d);
        serial_merge<W>(s_tile, TILE, a + da, a + len, b + d - da, b + len, k);
        __syncthreads();
    }
#pragma unroll
    for (int v = 0; v < kVT; ++v) lds_put(s_tile, TILE, tid * kVT + v, k[v]);
    __syncthreads();
    if (p.levels > 0) {
        write_keys<W, BLOCK>(p, p.key[0], s_tile, TILE, cnt, t0);
        return;
    }
    if (!p.distinct) {
        write_columns<W, BLOCK>(p, s_tile, TILE, cnt, 0);
        return;
    }
    // one tile, DISTINCT: the first of each run of equal rows
    bool keep[kVT];
    uint32_t mine = 0;
#pragma unroll
    for (int v = 0; v < kVT; ++v) {
        const uint32_t i = tid * kVT + v;
        keep[v] = i < cnt;
        if (i < cnt && i > 0) {
            const Key<W> before = lds_key<W>(s_tile, TILE, i - 1);
            bool same = true;
#pragma unroll
            for (int x = 0; x < W; ++x) same &= before.w[x] == k[v].w[x];
            keep[v] = !same;
        }
        mine += keep[v];
    }
    const uint32_t incl = dev::wave_inclusive_sum(mine);
    const int lane = tid % dev::kWave, wave = tid / dev::kWave;
    if (lane == dev::kWave - 1) s_w[wave] = incl;
    __syncthreads();
    uint32_t at = incl - mine, all = 0;
#pragma unroll
    for (int x = 0; x < NW; ++x) {
        if (x < wave) at += s_w[x];
        all += s_w[x];
    }
#pragma unroll
    for (int v = 0; v < kVT; ++v)
        if (keep[v]) lds_put(s_tile, TILE, at++, k[v]);  // every key is in registers
    __syncthreads();
    write_columns<W, BLOCK>(p, s_tile, TILE, all, 0);
    if (tid == 0) *p.count = all;
}

template <int W, int BLOCK>
__global__ __launch_bounds__(BLOCK) void row_tile_sort(RowJob p) {
    tile_sort_body<W, BLOCK>(p, blockIdx.x);
}

template <int W>
__global__ __launch_bounds__(tile_block(W)) void row_tile_sort_many(const RowJob *jobs,
                                                                    int J) {
    const uint32_t tile = blockIdx.x;
    const RowJob &p = jobs[row_job_of<false>(jobs, J, tile)];
    tile_sort_body<W, tile_block(W)>(p, tile - p.tile0);
}

// One launch for three merge levels, for tables that leave the chip idle: a
// workgroup finds the places of kRankBlock consecutive rows of one run among
// the kWays runs that are put together (rows that compare equal in the order
// of their runs).  In each of the other runs the rows' places lie between
// those of the workgroup's first and last row, which 16 lanes each find with a
// 16-way search; that part of the run is then searched in LDS (in memory, if
// the parts together do not fit).  Reads src's keys; the last launch writes
// the table's columns.
template <int W>
__global__ __launch_bounds__(kRankBlock) void row_rank_merge(RowJob p, uint32_t run, int src,
                                                             int last) {
    extern __shared__ __attribute__((aligned(16))) uint64_t s_part[];  // W planes of kRankPart
    __shared__ uint32_t s_cut[2][kWays];
    const uint32_t tid = threadIdx.x, lane = tid % dev::kWave;
    const uint32_t e0 = blockIdx.x * kRankBlock, e1 = min(p.n, e0 + kRankBlock);
    const uint64_t *key = p.key[src];
    auto load = [&](uint32_t i) {
        Key<W> k;
#pragma unroll
        for (int x = 0; x < W; ++x) k.w[x] = gload(key + (uint64_t)x * p.n + i);
        return k;
    };
    // a run is a multiple of kRankBlock rows: the workgroup's rows are of one run
    const uint32_t group = e0 / (kWays * run) * (kWays * run), own = (e0 - group) / run;
    auto rows_of = [&](uint32_t j) {
        const uint64_t first = (uint64_t)group + j * run;
        return j == own || first >= p.n ? 0u : (uint32_t)min((uint64_t)run, p.n - first);
    };
    auto precedes = [&](uint32_t j, const Key<W> &q, const Key<W> &k) {  // q of run j, k of own
        return j < own ? !key_less(k, q) : key_less(q, k);
    };
    const uint32_t i = min(e0 + tid, e1 - 1);
    const Key<W> k = load(i);
    {
        const uint32_t q = tid / 16, j = q / 2, l16 = tid % 16;
        const Key<W> edge = load(q % 2 ? e1 - 1 : e0);
        const uint32_t first = group + j * run;
        uint32_t lo = 0, hi = rows_of(j);
        while (dev::ballot(lo < hi)) {
            const uint32_t step = (hi - lo + 15) / 16, m = lo + l16 * step;
            const bool before = m < hi && precedes(j, load(first + m), edge);
            const uint32_t t = __popc((uint32_t)(dev::ballot(before) >> (lane & 48)) & 0xffffu);
            const uint32_t next = t == 0 ? lo : lo + (t - 1) * step + 1;
            hi = min(hi, lo + t * step);
            lo = next;
        }
        if (l16 == 0) s_cut[q % 2][j] = lo;
    }
    __syncthreads();
    uint32_t before[kWays], len[kWays], off[kWays], all = 0, most = 0;
#pragma unroll
    for (uint32_t j = 0; j < kWays; ++j) {
        before[j] = s_cut[0][j];
        len[j] = s_cut[1][j] - before[j];
        off[j] = all;
        all += len[j];
        most = max(most, len[j]);
    }
    uint32_t at = i - own * run;  // rows of the same run
#pragma unroll
    for (uint32_t j = 0; j < kWays; ++j) at += before[j];
    const bool fits = all <= kRankPart;
    if (fits) {
        Key<W> v[kWays];
#pragma unroll
        for (uint32_t j = 0; j < kWays; ++j) {
            v[j] = k;
            if (tid < len[j]) v[j] = load(group + j * run + before[j] + tid);
        }
#pragma unroll
        for (uint32_t j = 0; j < kWays; ++j) {
            if (tid < len[j]) lds_put(s_part, kRankPart, off[j] + tid, v[j]);
            for (uint32_t y = tid + kRankBlock; y < len[j]; y += kRankBlock)
                lds_put(s_part, kRankPart, off[j] + y, load(group + j * run + before[j] + y));
        }
        __syncthreads();
    }
    uint32_t c[kWays] = {};
    for (uint32_t step = most ? 1u << (31 - __builtin_clz(most)) : 0u; step; step >>= 1) {
#pragma unroll
        for (uint32_t j = 0; j < kWays; ++j) {
            const uint32_t to = c[j] + step;
            if (to > len[j]) continue;
            const Key<W> q = fits ? lds_key<W>(s_part, kRankPart, off[j] + to - 1)
                                  : load(group + j * run + before[j] + to - 1);
            c[j] = precedes(j, q, k) ? to : c[j];
        }
    }
#pragma unroll
    for (uint32_t j = 0; j < kWays; ++j) at += c[j];
    if (e0 + tid >= e1) return;
    if (last && !p.distinct) {
        for (int col = 0; col < p.ncols; ++col)
            gstore(p.out[col] + at, column_of<W>(p, col, [&](int x) {
                       uint64_t w = 0;
#pragma unroll
                       for (int y = 0; y < W; ++y) w = x == y ? k.w[y] : w;
                       return w;
                   }));
        return;
    }
    uint64_t *to = p.key[src ^ 1];
#pragma unroll
    for (int x = 0; x < W; ++x) gstore(to + (uint64_t)x * p.n + at, k.w[x]);
}

// The same cut as lds_diagonal, for keys in global memory (planes of `stride`
// words): the 64 lanes probe evenly spaced places of the interval and a
// ballot keeps the part that holds the cut, so about log64(n) dependent reads.
template <int W>
__device__ __forceinline__ uint32_t wave_diagonal(const uint64_t *key, uint64_t stride,
                                                  uint32_t a, uint32_t na, uint32_t b,
                                                  uint32_t nb, uint32_t d) {
    const uint32_t lane = (uint32_t)dev::lane_id();
    uint32_t lo = d > nb ? d - nb : 0, hi = min(d, na);
    while (lo < hi) {  // the same for every lane
        const uint32_t step = (hi - lo + dev::kWave - 1) / dev::kWave;
        const uint32_t m = lo + lane * step;
        bool before = false;  // the cut is past A's key m
        if (m < hi) {
            Key<W> ka, kb;
#pragma unroll
            for (int x = 0; x < W; ++x) {
                ka.w[x] = gload(key + (uint64_t)x * stride + a + m);
                kb.w[x] = gload(key + (uint64_t)x * stride + b + d - 1 - m);
            }
            before = !key_less(kb, ka);
        }
        const uint32_t t = (uint32_t)__popcll(dev::ballot(before));  // a prefix of the lanes
        const uint32_t next = t == 0 ? lo : lo + (t - 1) * step + 1;
        hi = min(hi, lo + t * step);
        lo = next;
    }
    return lo;
}

// The first of each run of equal keys in a sorted tile (in s_key, a thread's
// kVT keys also in k; before: the key before the tile, if `leads`) to the front
// of s_key; their number.
template <int W>
__device__ __forceinline__ uint32_t keep_firsts(uint64_t *s_key, const Key<W> (&k)[kVT],
                                                Key<W> before, bool leads, uint32_t cnt) {
    __shared__ uint32_t s_w[kMergeBlock / dev::kWave];
    const uint32_t tid = threadIdx.x, wave = tid / dev::kWave;
    bool keep[kVT];
    uint32_t mine = 0;
    if (tid > 0) before = lds_key<W>(s_key, kMergeTile, tid * kVT - 1);
#pragma unroll
    for (int v = 0; v < kVT; ++v) {
        bool same = v > 0 || tid > 0 || leads;
#pragma unroll
        for (int x = 0; x < W; ++x) same &= k[v].w[x] == (v ? k[v - 1].w[x] : before.w[x]);
        keep[v] = !same && tid * kVT + v < cnt;
        mine += keep[v];
    }
    const uint32_t incl = dev::wave_inclusive_sum(mine);
    if (tid % dev::kWave == dev::kWave - 1) s_w[wave] = incl;
    __syncthreads();  // also: every thread has read its keys
    uint32_t at = incl - mine, all = 0;
#pragma unroll
    for (uint32_t x = 0; x < kMergeBlock / dev::kWave; ++x) {
        at += x < wave ? s_w[x] : 0u;
        all += s_w[x];
    }
#pragma unroll
    for (int v = 0; v < kVT; ++v)
        if (keep[v]) lds_put(s_key, kMergeTile, at++, k[v]);
    __syncthreads();
    return all;
}

// Output rows [tile * kMergeTile, ...) of one merge level: runs of `run` rows
// (a multiple of kMergeTile) pairwise into runs of 2 * run.
template <int W>
__device__ __forceinline__ void merge_body(const RowJob &p, uint32_t tile, int level) {
    __shared__ uint64_t s_key[W * kMergeTile];
    __shared__ uint32_t s_cut[2];
    const uint32_t tid = threadIdx.x, wave = tid / dev::kWave;
    const uint64_t run = (uint64_t)tile_rows(W) << level;
    const uint64_t o0 = (uint64_t)tile * kMergeTile;
    const uint32_t cnt = (uint32_t)min((uint64_t)kMergeTile, p.n - o0);
    const uint64_t base = o0 / (2 * run) * (2 * run);
    const uint32_t a = (uint32_t)base, na = (uint32_t)min(run, p.n - base);
    const uint32_t b = a + na;
    const uint32_t nb = (uint32_t)min(run, p.n - base - na);
    const uint64_t *src = p.key[level & 1];
    const uint32_t d0 = (uint32_t)(o0 - base), d1 = d0 + cnt;
    if (wave < 2) {
        const uint32_t cut = wave_diagonal<W>(src, p.n, a, na, b, nb, wave == 0 ? d0 : d1);
        if (tid % dev::kWave == 0) s_cut[wave] = cut;
    }
    __syncthreads();
    const uint32_t a0 = s_cut[0], a1 = s_cut[1];
    const uint32_t b0 = d0 - a0, b1 = d1 - a1;
    const uint32_t ca = a1 - a0, cb = b1 - b0;  // ca + cb = cnt
#pragma unroll
    for (int x = 0; x < W; ++x) {
        const uint64_t *plane = src + (uint64_t)x * p.n;
        uint64_t v[kVT];
#pragma unroll
        for (int u = 0; u < kVT; ++u) {
            const uint32_t i = u * kMergeBlock + tid;
            v[u] = 0;
            if (i < cnt) v[u] = gload(plane + (i < ca ? a + a0 + i : b + b0 + (i - ca)));
        }
#pragma unroll
        for (int u = 0; u < kVT; ++u) s_key[x * kMergeTile + u * kMergeBlock + tid] = v[u];
    }
    __syncthreads();
    Key<W> k[kVT];
    const uint32_t d = min(tid * kVT, cnt);
    const uint32_t da = lds_diagonal<W>(s_key, kMergeTile, 0, ca, ca, cb, d);
    serial_merge<W>(s_key, kMergeTile, da, ca, ca + d - da, cnt, k);
    __syncthreads();
#pragma unroll
    for (int v = 0; v < kVT; ++v) lds_put(s_key, kMergeTile, tid * kVT + v, k[v]);
    __syncthreads();
    uint64_t *const dst = p.key[(level & 1) ^ 1];
    if (level + 1 < p.levels || !p.distinct) {
        if (level + 1 == p.levels)
            write_columns<W, kMergeBlock>(p, s_key, kMergeTile, cnt, (uint32_t)o0);
        else
            write_keys<W, kMergeBlock>(p, dst, s_key, kMergeTile, cnt, (uint32_t)o0);
        return;
    }
    // DISTINCT, last level: the first of each run of equal keys; the key before
    // the tile is the larger of the last ones cut off from the two runs
    Key<W> before{};
    const bool leads = tid == 0 && o0 > 0;
    if (leads) {
#pragma unroll
        for (int x = 0; x < W; ++x) {
            const uint64_t *plane = src + (uint64_t)x * p.n;
            before.w[x] = gload(plane + (a0 > 0 ? a + a0 - 1 : b + b0 - 1));
        }
        if (a0 > 0 && b0 > 0) {
            Key<W> q;
#pragma unroll
            for (int x = 0; x < W; ++x) q.w[x] = gload(src + (uint64_t)x * p.n + b + b0 - 1);
            const bool less = key_less(before, q);
#pragma unroll
            for (int x = 0; x < W; ++x) before.w[x] = less ? q.w[x] : before.w[x];
        }
    }
    const uint32_t all = keep_firsts<W>(s_key, k, before, leads, cnt);
    write_keys<W, kMergeBlock>(p, dst, s_key, kMergeTile, all, (uint32_t)o0);
    if (tid == 0) p.kept[tile] = all;
}

// The same for sorted keys in memory (key[from]).  p.kept null, for a few
// tiles: straight to the columns, every workgroup counting the first-of-equals
// before its tile itself; else into the other buffer.
template <int W>
__global__ __launch_bounds__(kMergeBlock) void row_keep_firsts(RowJob p, int from) {
    __shared__ uint64_t s_key[W * kMergeTile];
    __shared__ uint32_t s_sum[kMergeBlock / dev::kWave];
    const uint32_t tid = threadIdx.x, tile = blockIdx.x;
    const uint32_t o0 = tile * kMergeTile, cnt = min(kMergeTile, p.n - o0);
    const uint64_t *src = p.key[from];
#pragma unroll
    for (int x = 0; x < W; ++x)
        for (uint32_t i = tid; i < cnt; i += kMergeBlock)
            s_key[x * kMergeTile + i] = gload(src + (uint64_t)x * p.n + o0 + i);
    Key<W> before{};
    const bool leads = tid == 0 && o0 > 0;
    if (leads) {
#pragma unroll
        for (int x = 0; x < W; ++x) before.w[x] = gload(src + (uint64_t)x * p.n + o0 - 1);
    }
    uint32_t earlier = 0;
    if (!p.kept) {
#pragma unroll 4
        for (uint32_t i = tid; i < o0; i += kMergeBlock) {
            bool same = i > 0;
#pragma unroll
            for (int x = 0; x < W; ++x) {
                const uint64_t *w = src + (uint64_t)x * p.n + i;
                same &= i > 0 && gload(w) == gload(w - 1);
            }
            earlier += !same;
        }
        earlier = dev::wave_sum(earlier);
        if (tid % dev::kWave == 0) s_sum[tid / dev::kWave] = earlier;
    }
    __syncthreads();
    Key<W> k[kVT];
#pragma unroll
    for (int v = 0; v < kVT; ++v) k[v] = lds_key<W>(s_key, kMergeTile, tid * kVT + v);
    const uint32_t all = keep_firsts<W>(s_key, k, before, leads, cnt);
    if (p.kept) {
        write_keys<W, kMergeBlock>(p, p.key[from ^ 1], s_key, kMergeTile, all, o0);
        if (tid == 0) p.kept[tile] = all;
        return;
    }
    earlier = 0;
#pragma unroll
    for (int x = 0; x < kMergeBlock / dev::kWave; ++x) earlier += s_sum[x];
    write_columns<W, kMergeBlock>(p, s_key, kMergeTile, all, earlier);
    if (tile + 1 == gridDim.x && tid == 0) *p.count = earlier + all;
}

// The kept keys of every tile (first: exclusive sums of their numbers) to the
// table's columns.
template <int W>
__global__ __launch_bounds__(kMergeBlock) void kept_to_columns(RowJob p, int from,
                                                              const uint64_t *first) {
    const uint32_t tile = blockIdx.x;
    const uint64_t *key = p.key[from] + (uint64_t)tile * kMergeTile;
    const uint64_t at = first[tile];
    const uint32_t cnt = (uint32_t)(first[tile + 1] - at);
    for (uint32_t i = threadIdx.x; i < cnt; i += kMergeBlock) {
        Key<W> k;
#pragma unroll
        for (int x = 0; x < W; ++x) k.w[x] = gload(key + (uint64_t)x * p.n + i);
        for (int c = 0; c < p.ncols; ++c)
            gstore(p.out[c] + at + i, column_of<W>(p, c, [&](int x) {
                       uint64_t w = 0;
#pragma unroll
                       for (int y = 0; y < W; ++y) w = x == y ? k.w[y] : w;
                       return w;
                   }));
    }
    if (tile + 1 == gridDim.x && threadIdx.x == 0) *p.count = at + cnt;
}

template <int W>
__global__ __launch_bounds__(kMergeBlock) void row_merge(RowJob p, int level) {
    merge_body<W>(p, blockIdx.x, level);
}

template <int W>
__global__ __launch_bounds__(kMergeBlock) void row_merge_many(const RowJob *jobs, int J,
                                                              int level) {
    const uint32_t tile = blockIdx.x;
    const RowJob &p = jobs[row_job_of<true>(jobs, J, tile)];
    merge_body<W>(p, tile - p.mtile0, level);
}

// rows of one-word keys to keys, and sorted keys to columns (radix sort)
__device__ __forceinline__ void words_body(const RowJob &p, uint32_t tile) {
    const uint32_t t0 = tile * kMergeTile, cnt = min(kMergeTile, p.n - t0);
    Key<1> k[kVT];
    pack_rows<1, kMergeBlock>(p, t0, cnt, k);
    const bool whole = cnt == kMergeTile;
#pragma unroll
    for (int v = 0; v < kVT; ++v) {
        const uint32_t i = whole ? v * kMergeBlock + threadIdx.x : threadIdx.x * kVT + v;
        if (i < cnt) gstore(p.key[0] + t0 + i, k[v].w[0] | p.tag);
    }
}

__device__ __forceinline__ void columns_body(const RowJob &p, uint32_t tile, int from) {
    const uint32_t t0 = tile * kMergeTile, cnt = min(kMergeTile, p.n - t0);
    const uint64_t *key = p.key[from] + t0;
    uint64_t k[kVT];
#pragma unroll
    for (int v = 0; v < kVT; ++v) k[v] = gload(key + min(v * kMergeBlock + threadIdx.x, cnt - 1));
    for (int c = 0; c < p.ncols; ++c)
#pragma unroll
        for (int v = 0; v < kVT; ++v) {
            const uint32_t i = v * kMergeBlock + threadIdx.x;
            if (i < cnt) gstore(p.out[c] + t0 + i, column_of<1>(p, c, [&](int) { return k[v]; }));
        }
}

__global__ __launch_bounds__(kMergeBlock) void rows_to_words(RowJob p) {
    words_body(p, blockIdx.x);
}

__global__ __launch_bounds__(kMergeBlock) void words_to_columns(RowJob p, int from) {
    columns_body(p, blockIdx.x, from);
}

__global__ __launch_bounds__(kMergeBlock) void rows_to_words_many(const RowJob *jobs, int J) {
    const RowJob &p = jobs[row_job_of<true>(jobs, J, blockIdx.x)];
    words_body(p, blockIdx.x - p.mtile0);
}

__global__ __launch_bounds__(kMergeBlock) void words_to_columns_many(const RowJob *jobs, int J,
                                                                     int from) {
    const RowJob &p = jobs[row_job_of<true>(jobs, J, blockIdx.x)];
    columns_body(p, blockIdx.x - p.mtile0, from);
}

int bits_of(uint32_t v) { return v ? 32 - __builtin_clz(v) : 0; }

// words of a row's packed key, by the columns' bounds
int key_words(const tid_table *t) {
    int bits = 0;
    for (int c = 0; c < t->ncols; ++c) bits += bits_of(t->maxv[c]);
    return std::max(1, (bits + 63) / 64);
}

RowJob row_job(const tid_table *in, const tid_table *out, uint64_t n, int words, int distinct) {
    RowJob p{};
    p.ncols = (int16_t)in->ncols;
    p.n = (uint32_t)n;
    p.distinct = (int16_t)distinct;
    int at = 0;  // bits below the column
    for (int c = in->ncols - 1; c >= 0; --c) {
        p.in[c] = in->col[c];
        p.out[c] = out->col[c];
        p.width[c] = (uint8_t)bits_of(in->maxv[c]);
        p.word[c] = (uint8_t)(at / 64);
        p.shift[c] = (uint8_t)(at % 64);
        at += p.width[c];
    }
    for (uint64_t run = tile_rows(words); run < n; run *= 2) ++p.levels;
    return p;
}

template <int W>
void allow_lds() {
    // above 64 KB a kernel must be allowed its dynamic LDS first
    constexpr size_t lds = (size_t)tile_rows(W) * 8 * W;
    (void)resident_blocks((const void *)row_rank_merge<W>, kRankBlock, (size_t)kRankPart * 8 * W);
    (void)resident_blocks((const void *)row_tile_sort<W, tile_block(W)>, tile_block(W), lds);
    (void)resident_blocks((const void *)row_tile_sort_many<W>, tile_block(W), lds);
}

// Up to two levels of row_rank_merge: beyond, its reads (eight of every row, a
// level) cost more than the launches it spares.  A sort of one table, small
// tiles with row_rank_merge against large tiles with row_merge, one key word /
// two, with the call's own 40 us:
//    14,000 rows   55 /  70 us against  63 /  97 us
//   100,000 rows   77 / 104 us against 101 / 151 us
//   250,000 rows  114 / 175 us against 120 / 183 us
//   500,000 rows  157 / 246 us against 143 / 216 us
// (the last two with a third level; where between them the two are equal was not
// measured, so the line stands where two levels end).
// DISTINCT after it in one launch (row_keep_firsts) for so many merge tiles,
// else in three: 14,000 rows of one word 69 us against 83, 28,000 rows 102 against 95.
constexpr uint32_t kFewTiles = 8;
constexpr uint32_t kRankRows = kSmallTile * kVT * kWays * kWays;  // 114,688

int key_bits(const RowJob &p) {
    int bits = 0;
    for (int c = 0; c < p.ncols; ++c) bits += p.width[c];
    return std::max(1, bits);
}

// Passes of sort_words over keys of so many bits.
int radix_passes(int bits) { return std::max(1, std::min((bits + 8) / 9, (bits + 9) / 10)); }

// Whether a table of one-word keys is sorted by the radix passes of sort.hip on
// the packed keys instead of merge levels.  For large tables a pass costs about as
// much as 1.75 levels, for small ones two and a half.  A sort of two columns (one
// for 2 and 10 bits), merge (up to 114,688 rows: rank merge) / radix, in us:
//     bits (passes)   4,000 rows  16,000     100,000    200,000    400,000
//      2 (1)          60 / 55    77 / 58    93 / 61    99 / 64   113 / 65
//      8 (1)          60 / 58
//     10 (1)                     74 / 63    81 / 67   102 / 69   116 / 72
//     16 (2)                                86 / 90   109 / 94   126 / 97
//     20 (2)                                86 / 98   109 / 106  126 / 111
//     26 (3)                                          110 / 121  126 / 121
//     bits (passes)   500,000 rows    1M          2M          4M          16M
//     30 (3)          143 / 126   172 / 142   229 / 180   364 / 229  1360 /  693
//     36 (4)          139 / 132   171 / 149   227 / 181   368 / 242  1363 /  697
//     46 (5)          138 / 160   171 / 183   226 / 237   366 / 309  1359 /  943
//     54 (6)          139 / 167   171 / 191   226 / 236   366 / 316  1365 /  943
//     64 (7)          138 / 202   171 / 231   227 / 306   364 / 400  1364 / 1253
// Rows of one small tile (1,792) take one launch, which is as good (54 / 55).
bool radix_better(uint64_t n, int bits) {
    const int passes = radix_passes(bits);
    return n > (passes == 1   ? kSmallTile * kVT
                : passes == 2 ? kRankRows
                : passes <= 4 ? (1u << 19) - 1
                : passes <= 6 ? (3u << 20) - 1
                              : (3u << 22) - 1);
}

// One table; false, and nothing done, if there is no memory for two or more
// words a row: the radix sort of row numbers takes 24 B a row for any width.
template <int W>
bool sort_one(tid_ctx *ctx, RowJob &p) {
    allow_lds<W>();
    constexpr size_t lds = (size_t)tile_rows(W) * 8 * W;
    const int bits = key_bits(p);
    // DISTINCT of rows that fit one large tile is done there
    const bool one_tile = p.distinct && p.n <= tile_rows(W);
    const bool radix = W == 1 && !one_tile && radix_better(p.n, bits);
    const bool ranked = !radix && !one_tile && p.n <= kRankRows;
    if (radix) p.levels = std::max(p.levels, 1);  // it takes the key buffers
    if (ranked) {
        p.levels = 0;
        for (uint64_t run = (uint64_t)kSmallTile * kVT; run < p.n; run *= kWays) ++p.levels;
    }
    const uint32_t mtiles = (p.n + kMergeTile - 1) / kMergeTile;
    DevBuf keys, kept, first;
    try {
        if (p.levels) keys = DevBuf(ctx, 2 * (size_t)p.n * 8 * W);
        if (p.distinct && p.levels && !(ranked && mtiles <= kFewTiles)) {
            kept = DevBuf(ctx, (size_t)mtiles * 4);
            first = DevBuf(ctx, ((size_t)mtiles + 1) * 8);
        }
    } catch (const Error &) {
        if (W == 1) throw;
        return false;
    }
    if (p.levels) {
        p.key[0] = keys.get<uint64_t>();
        p.key[1] = p.key[0] + (size_t)p.n * W;
    }
    p.kept = kept.get<uint32_t>();
    int from = p.levels & 1;  // the buffer of the sorted keys
    if (radix) {
        hipLaunchKernelGGL(rows_to_words, dim3(mtiles), dim3(kMergeBlock), 0, ctx->stream, p);
        TID_HIP(hipGetLastError());
        from = sort_words(ctx, p.key[0], p.key[1], p.n, bits);
        if (p.distinct) {
            hipLaunchKernelGGL(row_keep_firsts<W>, dim3(mtiles), dim3(kMergeBlock), 0,
                               ctx->stream, p, from);
            from ^= 1;
        } else {
            hipLaunchKernelGGL(words_to_columns, dim3(mtiles), dim3(kMergeBlock), 0, ctx->stream,
                               p, from);
        }
        TID_HIP(hipGetLastError());
    } else if (ranked) {
        constexpr uint32_t rows = (uint32_t)kSmallTile * kVT;
        hipLaunchKernelGGL((row_tile_sort<W, kSmallTile>), dim3((p.n + rows - 1) / rows),
                           dim3(kSmallTile), (size_t)rows * 8 * W, ctx->stream, p);
        TID_HIP(hipGetLastError());
        constexpr size_t part = (size_t)kRankPart * 8 * W;
        uint32_t run = rows;
        for (int l = 0; l < p.levels; ++l, run *= kWays) {
            hipLaunchKernelGGL(row_rank_merge<W>, dim3((p.n + kRankBlock - 1) / kRankBlock),
                               dim3(kRankBlock), part, ctx->stream, p, run, l & 1,
                               (int)(l + 1 == p.levels));
            TID_HIP(hipGetLastError());
        }
        if (p.distinct) {
            hipLaunchKernelGGL(row_keep_firsts<W>, dim3(mtiles), dim3(kMergeBlock), 0,
                               ctx->stream, p, from);
            TID_HIP(hipGetLastError());
            from ^= 1;
        }
    } else {
        const uint32_t tiles = (p.n + tile_rows(W) - 1) / tile_rows(W);
        hipLaunchKernelGGL((row_tile_sort<W, tile_block(W)>), dim3(tiles), dim3(tile_block(W)),
                           lds, ctx->stream, p);
        TID_HIP(hipGetLastError());
        for (int l = 0; l < p.levels; ++l) {
            hipLaunchKernelGGL(row_merge<W>, dim3(mtiles), dim3(kMergeBlock), 0, ctx->stream, p,
                               l);
            TID_HIP(hipGetLastError());
        }
    }
    if (!p.kept) return true;
    exclusive_scan_async(ctx, p.kept, mtiles, first.get<uint64_t>());
    hipLaunchKernelGGL(kept_to_columns<W>, dim3(mtiles), dim3(kMergeBlock), 0, ctx->stream, p,
                       from, first.get<const uint64_t>());
    TID_HIP(hipGetLastError());
    return true;
}

template <int W>
void sort_many(tid_ctx *ctx, std::vector<RowJob *> jobs, const RowJob *dev) {
    allow_lds<W>();
    constexpr size_t lds = (size_t)tile_rows(W) * 8 * W;
    const int J = (int)jobs.size();
    const RowJob &last = *jobs.back();
    const uint32_t tiles = last.tile0 + (last.n + tile_rows(W) - 1) / tile_rows(W);
    hipLaunchKernelGGL(row_tile_sort_many<W>, dim3(tiles), dim3(tile_block(W)), lds, ctx->stream,
                       dev, J);
    TID_HIP(hipGetLastError());
    // jobs stand in order of falling size: a level's jobs are the first ones
    int active = J;
    for (int l = 0;; ++l) {
        while (active && jobs[active - 1]->levels <= l) --active;
        if (!active) break;
        const RowJob &p = *jobs[active - 1];
        const uint32_t mt = p.mtile0 + (p.n + kMergeTile - 1) / kMergeTile;
        hipLaunchKernelGGL(row_merge_many<W>, dim3(mt), dim3(kMergeBlock), 0, ctx->stream, dev,
                           active, l);
        TID_HIP(hipGetLastError());
    }
}

// Which of a round's one-word tables are sorted together by radix passes, their
// order above the keys: those of at most the bits that this returns, besides the
// order's (0: none).  A pass over R rows takes about 24 us + 13.6 ps a row, a merge
// level 9.5 us + 7.6 ps for every row of its tables, whose levels grow with the
// rows; so tables of few bits and many rows take the passes.  More than three
// passes are left to the levels.  A batch of whole-predicate plans, levels /
// passes, in us:
//     8 tables of 100,000 rows, 5 bits     114 /  72
//     8 of 1M, 5 bits                      491 / 146
//     8 of 1M, 10 bits                     500 / 202
//     64 of 400,000, 10 bits              1236 / 708
//     4 of 5M, 5 bits                     1262 / 250
int radix_bits_of_round(const std::vector<RowJob> &jobs, int order_bits) {
    double best = 0;
    int bits = 0;
    for (int passes = 0; passes <= 3; ++passes) {
        const int most = passes ? 10 * passes - order_bits : 0;
        double rows = 0, us = 0;
        std::vector<double> merged;  // rows of every level
        for (const RowJob &p : jobs) {
            if (p.levels && key_bits(p) <= most) {
                rows += p.n;
                continue;
            }
            merged.resize(std::max(merged.size(), (size_t)p.levels));
            for (int l = 0; l < p.levels; ++l) merged[l] += p.n;
        }
        if (passes && rows == 0) continue;
        us += passes * (24 + 13.6e-6 * rows);
        for (const double m : merged) us += 9.5 + 7.6e-6 * m;
        if (passes == 0 || us < best) {
            best = us;
            bits = most;
        }
    }
    return bits;
}

// bits that hold 0 .. n - 1
int index_bits(size_t n) {
    int bits = 0;
    while (n > 1 && (n - 1) >> bits) ++bits;
    return bits;
}

// Several tables of one-word keys by radix passes of all their rows at once: a
// row's key has the number of its table above it, so that every table's rows
// end at its own place.  The jobs' key buffers are parts of two arrays, in order.
void sort_round(tid_ctx *ctx, const std::vector<RowJob *> &jobs, const RowJob *dev, int bits) {
    const int J = (int)jobs.size();
    const RowJob &last = *jobs.back();
    const uint32_t tiles = last.mtile0 + (last.n + kMergeTile - 1) / kMergeTile;
    const uint64_t rows = (uint64_t)(last.key[0] - jobs[0]->key[0]) + last.n;
    hipLaunchKernelGGL(rows_to_words_many, dim3(tiles), dim3(kMergeBlock), 0, ctx->stream, dev, J);
    TID_HIP(hipGetLastError());
    const int from = sort_words(ctx, jobs[0]->key[0], jobs[0]->key[1], rows, bits);
    hipLaunchKernelGGL(words_to_columns_many, dim3(tiles), dim3(kMergeBlock), 0, ctx->stream, dev,
                       J, from);
    TID_HIP(hipGetLastError());
}

}  // namespace

// Whether the merge sort takes a table's rows: column bounds on the host, at
// most kMaxWords key words, and key buffers (16 B a row and word) no larger
// than the radix sort's arrays (24 B a row) once a table is large.  Measured
// on one MI355X, one table, merge sort against the LSD radix sort with its
// gather (2 columns of 23 bits, one word / 7 columns of 25 bits, three words):
//      7,168 rows    57 /  103 us against   110 /   309 us
//     50,000 rows    99 /  164 us against   197 /   660 us
//  1,000,000 rows   197 /  377 us against   281 /  1034 us
//  4,000,000 rows   413 / 1099 us against   755 /  3038 us
// 16,000,000 rows  1424 / 4653 us against  2586 / 11557 us
// so it is the faster one wherever it is allowed.
constexpr uint64_t kMergeRows1 = 1ull << 31;  // one key word
constexpr uint64_t kMergeRows = 1ull << 26;   // more

bool rows_mergeable(const tid_table *t, uint64_t n) {
    if (!t->maxv_known || t->ncols <= 0) return false;
    const int w = key_words(t);
    return w == 1 ? n <= kMergeRows1 : w <= kMaxWords && n <= kMergeRows;
}

// The n >= 1 rows of `in` in lexicographic order into `out` (n rows
// allocated); distinct = 1: without repeats, the count left to the kernels.
// False, and nothing done, if there is no memory for the keys.
bool merge_sort_rows(tid_ctx *ctx, const tid_table *in, uint64_t n, tid_table *out,
                     int distinct) {
    const int w = key_words(in);
    RowJob p = row_job(in, out, n, w, distinct);
    if (distinct) p.count = out->d_count;
    return w == 1 ? sort_one<1>(ctx, p) : w == 2 ? sort_one<2>(ctx, p)
         : w == 3 ? sort_one<3>(ctx, p) : sort_one<4>(ctx, p);
}

// The same for many tables in shared launches (no DISTINCT, counts set by the
// caller); every table must be rows_mergeable.  Returns the jobs that there was
// no memory for, with nothing done for them.
std::vector<RowSortJob> merge_sort_rows_batched(tid_ctx *ctx, const std::vector<RowSortJob> &all,
                                                std::vector<DevBuf> &keep,
                                                std::vector<std::vector<char>> &host_keep) {
    std::vector<RowSortJob> left;
    // chunks of jobs in order, each with at most kChunkBytes of keys (a larger job
    // alone); a chunk's key buffers go back, in stream order, before the next
    // chunk's are taken
    constexpr uint64_t kChunkBytes = 4ull << 30;
    for (size_t j0 = 0; j0 < all.size();) {
        std::vector<RowJob> by_words[kMaxWords + 1];
        uint64_t bytes = 0;
        size_t j1 = j0;
        for (; j1 < all.size(); ++j1) {
            const RowSortJob &r = all[j1];
            const int w = key_words(r.in);
            RowJob p = row_job(r.in, r.out, r.n, w, 0);
            const uint64_t need = p.levels ? 2 * r.n * 8 * (uint64_t)w : 0;
            if (j1 > j0 && bytes + need > kChunkBytes) break;
            bytes += need;
            by_words[w].push_back(p);
        }
        // by_words[0]: the one-word tables that are sorted together by radix passes
        const int few = radix_bits_of_round(by_words[1], index_bits(by_words[1].size()));
        int bits = 0;
        if (few) {
            std::vector<RowJob> rest;
            for (const RowJob &p : by_words[1])
                (p.levels && key_bits(p) <= few ? by_words[0] : rest).push_back(p);
            by_words[1].swap(rest);
            for (const RowJob &p : by_words[0]) bits = std::max(bits, key_bits(p));
            for (size_t x = 0; x < by_words[0].size(); ++x)
                by_words[0][x].tag = (uint64_t)x << bits;
            bits += index_bits(by_words[0].size());
        }
        DevBuf arena;
        try {
            arena = DevBuf(ctx, std::max<uint64_t>(bytes, 8));
        } catch (const Error &) {
            left.insert(left.end(), all.begin() + j0, all.begin() + j1);
            j0 = j1;
            continue;
        }
        uint64_t *at = arena.get<uint64_t>();
        std::vector<RowJob> table;
        size_t first[kMaxWords + 2] = {};
        for (int w = 0; w <= kMaxWords; ++w) {
            std::vector<RowJob> &v = by_words[w];
            const uint64_t words = std::max(w, 1);
            uint64_t together = 0;  // rows sorted together: all of one buffer, then the other
            if (w == 0)
                for (const RowJob &p : v) together += p.n;
            else
                std::stable_sort(v.begin(), v.end(),
                                 [](const RowJob &x, const RowJob &y) { return x.n > y.n; });
            uint32_t tiles = 0, mtiles = 0;
            for (RowJob &p : v) {
                if (p.levels) {
                    p.key[0] = at;
                    p.key[1] = at + (together ? together : p.n * words);
                    at += (together ? 1 : 2) * p.n * words;
                }
                p.tile0 = tiles;
                p.mtile0 = mtiles;
                tiles += (p.n + tile_rows(words) - 1) / tile_rows(words);
                mtiles += (p.n + kMergeTile - 1) / kMergeTile;
            }
            at += together;
            first[w] = table.size();
            table.insert(table.end(), v.begin(), v.end());
        }
        first[kMaxWords + 1] = table.size();
        const size_t tb = table.size() * sizeof(RowJob);
        host_keep.emplace_back(reinterpret_cast<const char *>(table.data()),
                               reinterpret_cast<const char *>(table.data()) + tb);
        keep.emplace_back(ctx, tb);
        const RowJob *dev = keep.back().get<const RowJob>();
        TID_HIP(hipMemcpyAsync(keep.back().get(), host_keep.back().data(), tb,
                               hipMemcpyHostToDevice, ctx->stream));
        for (int w = 0; w <= kMaxWords; ++w) {
            std::vector<RowJob *> v;
            for (size_t x = first[w]; x < first[w + 1]; ++x) v.push_back(&table[x]);
            if (v.empty()) continue;
            if (w == 0) sort_round(ctx, v, dev, bits);
            else if (w == 1) sort_many<1>(ctx, v, dev + first[w]);
            else if (w == 2) sort_many<2>(ctx, v, dev + first[w]);
            else if (w == 3) sort_many<3>(ctx, v, dev + first[w]);
            else sort_many<4>(ctx, v, dev + first[w]);
        }
        j0 = j1;
    }
    return left;
}

}  // namespace tid
