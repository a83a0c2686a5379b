// scan_pages.hip -- the multi-pattern pass of Sec. 4.1 (keysArray /
// positionArray[i].query) for up to 16 patterns and outputs of any density,
// in one read of the graph.
//
// A workgroup walks one contiguous range of the graph, tile by tile, and
// appends each pattern's matches, in triple order, to pages of kPageRows rows;
// which page holds which rows of which (range, pattern) is in the page's
// header.  Pages are taken from one counter, kPoolPages at a time, and nothing
// else is shared between workgroups while they run.  A second launch adds up
// the ranges' counts and copies every page to its place in the pattern's
// table.
//
// Bound: the graph's 12 bytes a triple once, the vector instructions of the
// tests, and 12 bytes a column of a matching row: written to its page, read
// from it, written to the table.  So:
//  - a pattern with a constant predicate costs one compare a triple to count
//    and one to place; its other tests run only in waves that hold the
//    predicate;
//  - where no triple can match two patterns (DISJOINT), a lane first finds the
//    place of its triple under any of the patterns and stores once;
//  - rows are stored by position (subject, predicate, object planes), not by
//    output column, so storing does not depend on the pattern.
// The block-ranged kernel (passes of at most four patterns) stages rows in LDS
// and reads the graph a second time where they do not fit; it stays for up to
// four patterns whose rows do fit, unless they are a predicate each
// (scan_pages_better).  Measured on one
// MI355X: 12 patterns with 3.6M rows in all on 30M triples 884 us in three
// block-ranged passes, 145 us here; 3 patterns with 45M rows on 200M triples
// 3353 us, 803 us here (2.4 GB read: 348 us at the plain read rate).
#include "scan_common.hpp"

#include <algorithm>

namespace tid {

namespace {

constexpr int kPgBlock = 512;
constexpr int kPgIPT = 8;
constexpr int kPgNW = kPgBlock / dev::kWave;
constexpr uint32_t kPgWaveRows = dev::kWave * kPgIPT;  // consecutive triples of a wave's tile part
constexpr uint64_t kPgTile = (uint64_t)kPgBlock * kPgIPT;
constexpr uint32_t kPageShift = 10;
constexpr uint32_t kPageRows = 1u << kPageShift;
constexpr int kRing = 8;  // a tile touches at most 4096 / kPageRows + 2 pages of a pattern
constexpr uint32_t kPoolPages = 16;
constexpr uint32_t kPgMaxRanges = 2048;
constexpr uint32_t kNoRow = 0xFFFFFFFFu;
constexpr uint64_t kUnused = ~0ull;  // header of a page that holds no rows

// how a pattern is tested: every position at once, or its predicate first
constexpr int kGeneral = 0, kPredicateFirst = 1;

struct PageArgs {
    DevPattern pat[TID_MAX_MULTI];
    int32_t kind[TID_MAX_MULTI];
    int32_t k;
    uint32_t P;           // ranges (= workgroups)
    const uint32_t *g;
    uint64_t n, range;    // triples; triples per range, a multiple of the tile
    uint32_t *cnt;        // k x P matches per pattern and range
    uint32_t *plane[3];   // page rows' subjects, predicates, objects (null: no pattern
                          // puts the position out)
    uint64_t *hdr;        // per page: range << 40 | pattern << 32 | its number in the list
    uint32_t *npages;
    uint32_t max_pages;
    uint32_t *flags;
};

struct GatherOut {
    uint32_t *col[3];
    const uint32_t *plane[3];
    uint64_t cap;
    uint64_t *count;
    int32_t ncols;
};

struct PageGather {
    GatherOut out[TID_MAX_MULTI];
    int32_t k;
    uint32_t P;
    const uint32_t *cnt, *npages;
    const uint64_t *hdr;
    uint32_t max_pages;
};

// What every wave of a workgroup keeps of the patterns' row lists, lane j for
// pattern j: the rows so far and, for the tile at hand, where the wave's own
// rows go.
struct PageLists {
    uint32_t run = 0;                 // rows of the range so far
    uint32_t base = 0;                // the wave's first row of the tile
    uint32_t off0 = 0, off1 = 0;      // row r is page row r + off0 before `edge`, r + off1
    uint32_t edge = 0;                // from it on (a wave's rows, at most 512 a tile, lie
    bool two = false;                 // in one page, or in two)
    uint32_t pool = 0, pool_end = 0;  // wave 0: pages taken and not yet used
};

// After every wave has put its matches c of a tile (lane j: pattern j): the
// wave's place in every list, and pages for the rows the tile adds.  Pages
// beyond max_pages (there are none: the host sized them) report an error and
// their rows go to page 0.
__device__ __forceinline__ void place_tile(const PageArgs &a, PageLists &l, uint32_t c, int wave,
                                           int lane, bool stores,
                                           const uint32_t (*s_c)[TID_MAX_MULTI],
                                           uint32_t (*s_page)[kRing]) {
    const int lj = min(lane, a.k - 1);
    uint32_t before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < kPgNW; ++w) {
        const uint32_t x = s_c[w][lj];
        before += w < wave ? x : 0u;
        tot += x;
    }
    l.base = l.run + before;
    const uint32_t have = (l.run + kPageRows - 1) >> kPageShift;
    l.run += tot;
    const uint32_t want = (l.run + kPageRows - 1) >> kPageShift;
    const bool grow = lane < a.k && stores && want > have;
    if (dev::ballot(grow)) {  // the same in every wave
        if (wave == 0) {
            const uint32_t add = grow ? want - have : 0u;
            const uint32_t incl = dev::wave_inclusive_sum(add);
            const uint32_t all = __builtin_amdgcn_readlane(incl, dev::kWave - 1);
            const uint32_t left = l.pool_end - l.pool;
            const uint32_t take = all > left ? max(all - left, kPoolPages) : 0u;
            uint32_t fresh = 0;
            if (take) {
                if (lane == 0) fresh = atomicAdd(a.npages, take);
                fresh = __builtin_amdgcn_readfirstlane(fresh);
            }
            for (uint32_t x = 0; x < add; ++x) {  // leftover pages first
                const uint32_t at = incl - add + x;
                uint32_t page = at < left ? l.pool + at : fresh + (at - left);
                if (page < a.max_pages) {
                    a.hdr[page] = (uint64_t)blockIdx.x << 40 | (uint64_t)lane << 32 | (have + x);
                } else {
                    dev::raise(&a.flags[0]);
                    page = 0;
                }
                s_page[lane][(have + x) & (kRing - 1)] = page;
            }
            if (take) {
                l.pool = fresh + (all - left);
                l.pool_end = fresh + take;
            } else {
                l.pool += all;
            }
        }
        __syncthreads();
    }
    const uint32_t seq = l.base >> kPageShift;
    l.edge = (seq + 1) << kPageShift;
    l.two = l.base + c > l.edge;
    const uint32_t p0 = c ? s_page[lj][seq & (kRing - 1)] : 0u;
    const uint32_t p1 = l.two ? s_page[lj][(seq + 1) & (kRing - 1)] : 0u;
    l.off0 = (p0 - seq) << kPageShift;
    l.off1 = (p1 - (seq + 1)) << kPageShift;
}

// the tile at t0 of a wave, item by item 64 consecutive triples; a triple past
// the range is all zeros, which no constant matches
__device__ __forceinline__ void load_tile(const PageArgs &a, uint64_t t0, uint64_t r1, int wave,
                                          int lane, Tri (&t)[kPgIPT]) {
    const uint64_t w0 = t0 + (uint64_t)wave * kPgWaveRows + lane;
    if (t0 + kPgTile <= r1) {
#pragma unroll
        for (int it = 0; it < kPgIPT; ++it)
#pragma unroll
            for (int x = 0; x < 3; ++x)
                t[it].v[x] = __builtin_nontemporal_load(a.g + 3 * (w0 + it * dev::kWave) + x);
        return;
    }
#pragma unroll
    for (int it = 0; it < kPgIPT; ++it) {
        const uint64_t i = w0 + it * dev::kWave;
#pragma unroll
        for (int x = 0; x < 3; ++x)
            t[it].v[x] = i < r1 ? __builtin_nontemporal_load(a.g + 3 * i + x) : 0u;
    }
}

__device__ __forceinline__ void put_row(uint32_t *plane, uint32_t row, uint32_t v) {
    // the planes are smaller than 4 GiB: a 32-bit byte offset
    *reinterpret_cast<uint32_t *>(reinterpret_cast<char *>(plane) + (row << 2)) = v;
}

// Patterns that are a constant predicate each, all different, and nothing
// else: the rows of several predicates.
__global__ __launch_bounds__(kPgBlock) void predicates_to_pages(PageArgs a) {
    __shared__ uint32_t s_c[2][kPgNW][TID_MAX_MULTI];  // matches per wave of a tile
    __shared__ uint32_t s_page[TID_MAX_MULTI][kRing];  // a pattern's latest pages
    __shared__ uint32_t s_key[TID_MAX_MULTI];
    __shared__ int32_t s_cols[TID_MAX_MULTI];
    const int tid = threadIdx.x, lane = tid % dev::kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / dev::kWave);
    const int k = a.k;
#pragma unroll
    for (int j = 0; j < TID_MAX_MULTI; ++j)  // static indices into the kernel arguments
        if (tid == j && j < k) {
            s_key[j] = a.pat[j].key[1];
            s_cols[j] = a.pat[j].ncols;
        }
    __syncthreads();
    const int lj = min(lane, k - 1);
    const uint32_t v_key = s_key[lj];
    const bool stores = s_cols[lj] > 0;
    PageLists l;
    const uint64_t r0 = (uint64_t)blockIdx.x * a.range, r1 = min(a.n, r0 + a.range);
    uint32_t *const ps = a.plane[0], *const po = a.plane[2];
    Tri next[kPgIPT], t[kPgIPT];
    if (r0 < r1) load_tile(a, r0, r1, wave, lane, next);
    int par = 0;
    for (uint64_t t0 = r0; t0 < r1; t0 += kPgTile, par ^= 1) {
#pragma unroll
        for (int it = 0; it < kPgIPT; ++it) t[it] = next[it];
        if (t0 + kPgTile < r1) load_tile(a, t0 + kPgTile, r1, wave, lane, next);
        uint32_t v_c = 0;
        for (int j = 0; j < k; ++j) {
            const uint32_t key = __builtin_amdgcn_readlane(v_key, j);
            uint32_t c = 0;
#pragma unroll
            for (int it = 0; it < kPgIPT; ++it)
                c += (uint32_t)__popcll(dev::ballot(t[it].v[1] == key));
            v_c = lane == j ? c : v_c;
        }
        if (lane < k) s_c[par][wave][lane] = v_c;
        __syncthreads();
        place_tile(a, l, v_c, wave, lane, stores, s_c[par], s_page);
        uint32_t at[kPgIPT];
#pragma unroll
        for (int it = 0; it < kPgIPT; ++it) at[it] = kNoRow;
        uint64_t todo = dev::ballot(lane < k && stores && v_c > 0);
        while (todo) {
            const int j = __builtin_ctzll(todo);
            todo &= todo - 1;
            const uint32_t key = __builtin_amdgcn_readlane(v_key, j);
            const uint32_t base = __builtin_amdgcn_readlane(l.base, j);
            const uint32_t off0 = __builtin_amdgcn_readlane(l.off0, j);
            if (!__builtin_amdgcn_readlane((int)l.two, j)) {
                uint32_t r = base + off0;
#pragma unroll
                for (int it = 0; it < kPgIPT; ++it) {
                    const bool m = t[it].v[1] == key;
                    const uint64_t b = dev::ballot(m);
                    at[it] = m ? dev::rank_in_mask(b) + r : at[it];
                    r += (uint32_t)__popcll(b);
                }
            } else {
                const uint32_t edge = __builtin_amdgcn_readlane(l.edge, j);
                const uint32_t off1 = __builtin_amdgcn_readlane(l.off1, j);
                uint32_t r = base;
#pragma unroll
                for (int it = 0; it < kPgIPT; ++it) {
                    const bool m = t[it].v[1] == key;
                    const uint64_t b = dev::ballot(m);
                    const uint32_t x = dev::rank_in_mask(b) + r;
                    at[it] = m ? x + (x < edge ? off0 : off1) : at[it];
                    r += (uint32_t)__popcll(b);
                }
            }
        }
#pragma unroll
        for (int it = 0; it < kPgIPT; ++it)
            if (at[it] != kNoRow) {
                put_row(ps, at[it], t[it].v[0]);
                put_row(po, at[it], t[it].v[2]);
            }
    }
    if (wave == 0 && lane < k) a.cnt[(size_t)lane * a.P + blockIdx.x] = l.run;
}

// The same by a table of the patterns' predicates in LDS: the work of a triple
// does not grow with the patterns, and places are found in the same walk that
// counts.  For more than kFewKeys patterns with predicates below kTableIds: on 30M
// triples 131 us with compares and 142 with the table for 5 patterns, 166 and
// 159 for 8, 272 and 212 for 16.
constexpr int kFewKeys = 6;
constexpr uint32_t kTableIds = 8192;
__global__ __launch_bounds__(kPgBlock) void table_to_pages(PageArgs a) {
    constexpr uint32_t kNone = 0xFFu;
    __shared__ uint32_t s_c[2][kPgNW][TID_MAX_MULTI];  // matches per wave of a tile
    __shared__ uint32_t s_page[TID_MAX_MULTI][kRing];  // a pattern's latest pages
    __shared__ int32_t s_cols[TID_MAX_MULTI];
    __shared__ uint32_t s_table[kTableIds / 4];        // a byte an ID: its pattern
    __shared__ uint32_t s_run[kPgNW][TID_MAX_MULTI];   // a wave's matches so far in the tile
    __shared__ uint4 s_list[kPgNW][TID_MAX_MULTI];     // its PageLists, by pattern
    uint8_t *s_id = reinterpret_cast<uint8_t *>(s_table);
    const int tid = threadIdx.x, lane = tid % dev::kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / dev::kWave);
    const int k = a.k;
    for (uint32_t i = tid; i < kTableIds / 4; i += kPgBlock) s_table[i] = 0xFFFFFFFFu;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < TID_MAX_MULTI; ++j)  // static indices into the kernel arguments
        if (tid == j && j < k) {
            s_id[a.pat[j].key[1]] = (uint8_t)j;  // all different
            s_cols[j] = a.pat[j].ncols;
        }
    __syncthreads();
    const bool stores = s_cols[min(lane, k - 1)] > 0;
    const uint32_t storing = (uint32_t)dev::ballot(lane < k && stores);
    PageLists l;
    const uint64_t r0 = (uint64_t)blockIdx.x * a.range, r1 = min(a.n, r0 + a.range);
    const uint64_t lt = (1ull << lane) - 1ull;
    uint32_t *const ps = a.plane[0], *const po = a.plane[2];
    Tri next[kPgIPT], t[kPgIPT];
    if (r0 < r1) load_tile(a, r0, r1, wave, lane, next);
    int par = 0;
    for (uint64_t t0 = r0; t0 < r1; t0 += kPgTile, par ^= 1) {
#pragma unroll
        for (int it = 0; it < kPgIPT; ++it) t[it] = next[it];
        if (t0 + kPgTile < r1) load_tile(a, t0 + kPgTile, r1, wave, lane, next);
        if (lane < k) s_run[wave][lane] = 0;
        uint32_t id[kPgIPT], rank[kPgIPT];
#pragma unroll
        for (int it = 0; it < kPgIPT; ++it)
            id[it] = t[it].v[1] < kTableIds ? s_id[t[it].v[1]] : kNone;
#pragma unroll
        for (int it = 0; it < kPgIPT; ++it) {
            const bool m = id[it] != kNone;
            rank[it] = 0;
            if (dev::ballot(m) == 0) continue;
            const uint64_t peers = dev::match_digit<4>(id[it], m);
            const uint32_t before = m ? s_run[wave][id[it]] : 0u;
            rank[it] = before + (uint32_t)__popcll(peers & lt);
            if (m && lane == __builtin_ctzll(peers))
                s_run[wave][id[it]] = before + (uint32_t)__popcll(peers);
        }
        const uint32_t v_c = lane < k ? s_run[wave][lane] : 0u;
        if (lane < k) s_c[par][wave][lane] = v_c;
        __syncthreads();
        place_tile(a, l, v_c, wave, lane, stores, s_c[par], s_page);
        if (lane < k) s_list[wave][lane] = make_uint4(l.base, l.edge, l.off0, l.off1);
#pragma unroll
        for (int it = 0; it < kPgIPT; ++it) {
            if (id[it] == kNone || !(storing >> id[it] & 1u)) continue;
            const uint4 list = s_list[wave][id[it]];
            const uint32_t x = list.x + rank[it], at = x + (x < list.y ? list.z : list.w);
            put_row(ps, at, t[it].v[0]);
            put_row(po, at, t[it].v[2]);
        }
    }
    if (wave == 0 && lane < k) a.cnt[(size_t)lane * a.P + blockIdx.x] = l.run;
}

// Any patterns.  EXT: some pattern's test reads memory (a value set, a
// filter), so the match masks of a tile are kept; DISJOINT: no triple matches
// two of the patterns.
template <bool EXT, bool DISJOINT>
__global__ __launch_bounds__(kPgBlock) void scan_to_pages(PageArgs a) {
    __shared__ DevPattern s_pat[TID_MAX_MULTI];
    __shared__ int32_t s_kind[TID_MAX_MULTI];
    __shared__ uint32_t s_c[2][kPgNW][TID_MAX_MULTI];
    __shared__ uint32_t s_page[TID_MAX_MULTI][kRing];
    __shared__ uint64_t s_mask[EXT ? kPgNW : 1][EXT ? TID_MAX_MULTI : 1][kPgIPT];
    const int tid = threadIdx.x, lane = tid % dev::kWave;
    const int wave = __builtin_amdgcn_readfirstlane(tid / dev::kWave);
    const int k = a.k;
    // thread j copies pattern j (static indices into the kernel arguments)
#pragma unroll
    for (int j = 0; j < TID_MAX_MULTI; ++j)
        if (tid == j && j < k) {
            s_pat[j] = a.pat[j];
            s_kind[j] = a.kind[j];
        }
    __syncthreads();
    const int lj = min(lane, k - 1);
    const uint32_t v_key = s_pat[lj].key[1];
    const int v_kind = s_kind[lj];
    const bool stores = s_pat[lj].ncols > 0;
    PageLists l;
    const uint64_t r0 = (uint64_t)blockIdx.x * a.range, r1 = min(a.n, r0 + a.range);
    Tri next[kPgIPT], t[kPgIPT];
    auto test = [&](int j, const Tri &x) {
        return EXT ? match_pattern(s_pat[j], x) : match_plain(s_pat[j], x);
    };
    // the lanes whose item `it` of the tile at t0 matches pattern j
    auto matches = [&](int j, int kind, uint32_t key, int it, uint64_t t0) -> uint64_t {
        if (kind == kGeneral)
            return dev::ballot(t0 + (uint64_t)wave * kPgWaveRows + it * dev::kWave + lane < r1 &&
                               test(j, t[it]));
        const uint64_t b = dev::ballot(t[it].v[1] == key);
        if (b == 0) return b;
        return dev::ballot(t[it].v[1] == key && test(j, t[it]));
    };
    auto store = [&](uint32_t row, const Tri &x) {
#pragma unroll
        for (int p = 0; p < 3; ++p)
            if (a.plane[p]) put_row(a.plane[p], row, x.v[p]);
    };
    if (r0 < r1) load_tile(a, r0, r1, wave, lane, next);
    int par = 0;
    for (uint64_t t0 = r0; t0 < r1; t0 += kPgTile, par ^= 1) {
#pragma unroll
        for (int it = 0; it < kPgIPT; ++it) t[it] = next[it];
        if (t0 + kPgTile < r1) load_tile(a, t0 + kPgTile, r1, wave, lane, next);
        uint32_t v_c = 0;
        for (int j = 0; j < k; ++j) {
            const int kind = __builtin_amdgcn_readlane(v_kind, j);
            const uint32_t key = __builtin_amdgcn_readlane(v_key, j);
            uint32_t c = 0;
            uint64_t mine = 0;
#pragma unroll
            for (int it = 0; it < kPgIPT; ++it) {
                const uint64_t b = matches(j, kind, key, it, t0);
                c += (uint32_t)__popcll(b);
                if (EXT && lane == it) mine = b;
            }
            if (EXT && lane < kPgIPT) s_mask[EXT ? wave : 0][EXT ? j : 0][lane] = mine;
            v_c = lane == j ? c : v_c;
        }
        if (lane < k) s_c[par][wave][lane] = v_c;
        __syncthreads();
        place_tile(a, l, v_c, wave, lane, stores, s_c[par], s_page);
        uint32_t at[kPgIPT];
#pragma unroll
        for (int it = 0; it < kPgIPT; ++it) at[it] = kNoRow;
        uint64_t todo = dev::ballot(lane < k && stores && v_c > 0);
        while (todo) {
            const int j = __builtin_ctzll(todo);
            todo &= todo - 1;
            const int kind = __builtin_amdgcn_readlane(v_kind, j);
            const uint32_t key = __builtin_amdgcn_readlane(v_key, j);
            const uint32_t off0 = __builtin_amdgcn_readlane(l.off0, j);
            const uint32_t off1 = __builtin_amdgcn_readlane(l.off1, j);
            const uint32_t edge = __builtin_amdgcn_readlane(l.edge, j);
            uint32_t r = __builtin_amdgcn_readlane(l.base, j);
#pragma unroll
            for (int it = 0; it < kPgIPT; ++it) {
                const uint64_t b = EXT ? s_mask[EXT ? wave : 0][EXT ? j : 0][it]
                                       : matches(j, kind, key, it, t0);
                const bool m = (b >> lane) & 1u;
                uint32_t x = dev::rank_in_mask(b) + r;
                x += x < edge ? off0 : off1;
                if (DISJOINT)
                    at[it] = m ? x : at[it];
                else if (m)
                    store(x, t[it]);
                r += (uint32_t)__popcll(b);
            }
        }
        if (DISJOINT) {
#pragma unroll
            for (int it = 0; it < kPgIPT; ++it)
                if (at[it] != kNoRow) store(at[it], t[it]);
        }
    }
    if (wave == 0 && lane < k) a.cnt[(size_t)lane * a.P + blockIdx.x] = l.run;
}

// The sum of c[0, m), the same in every thread of the workgroup.
constexpr int kGatherBlock = 256;
__device__ __forceinline__ uint64_t block_sum(const uint32_t *c, uint32_t m, uint64_t *s_w) {
    uint64_t sum = 0;
    for (uint32_t i = threadIdx.x; i < m; i += kGatherBlock) sum += c[i];
    sum = dev::wave_sum(sum);
    __syncthreads();  // s_w is free again
    if (threadIdx.x % dev::kWave == 0) s_w[threadIdx.x / dev::kWave] = sum;
    __syncthreads();
    uint64_t all = 0;
    for (int w = 0; w < kGatherBlock / dev::kWave; ++w) all += s_w[w];
    return all;
}

// Pages to their places: a page's rows start after the pattern's rows in
// earlier ranges and in the range's earlier pages.  Workgroup j < k also
// writes pattern j's row count.
__global__ __launch_bounds__(kGatherBlock) void pages_to_tables(PageGather a) {
    __shared__ uint64_t s_w[kGatherBlock / dev::kWave];
    __shared__ GatherOut s_out[TID_MAX_MULTI];
    const int tid = threadIdx.x;
#pragma unroll
    for (int j = 0; j < TID_MAX_MULTI; ++j)
        if (tid == j && j < a.k) s_out[j] = a.out[j];
    __syncthreads();
    if ((int)blockIdx.x < a.k) {
        const uint64_t all = block_sum(a.cnt + (size_t)blockIdx.x * a.P, a.P, s_w);
        if (tid == 0) *s_out[blockIdx.x].count = all;
    }
    const uint32_t np = min(*a.npages, a.max_pages);
    for (uint32_t q = blockIdx.x; q < np; q += gridDim.x) {
        const uint64_t h = a.hdr[q];
        if (h == kUnused) continue;  // taken and not needed
        const uint32_t wg = (uint32_t)(h >> 40), j = (uint32_t)(h >> 32) & 0xFFu, seq = (uint32_t)h;
        const uint32_t *c = a.cnt + (size_t)j * a.P;
        const uint32_t rows = min(kPageRows, c[wg] - (seq << kPageShift));
        const uint64_t at = block_sum(c, wg, s_w) + ((uint64_t)seq << kPageShift);
        const GatherOut &o = s_out[j];
        for (int x = 0; x < o.ncols; ++x) {
            const uint32_t *src = o.plane[x] + ((uint64_t)q << kPageShift);
            for (uint32_t i = tid; i < rows; i += kGatherBlock)
                if (at + i < o.cap) dev::put(&o.col[x][at + i], src[i]);
        }
    }
}

__global__ void clear_pages(uint32_t *npages, uint64_t *hdr, uint32_t pages) {
    if (blockIdx.x == 0 && threadIdx.x == 0) *npages = 0;
    for (uint32_t q = blockIdx.x * blockDim.x + threadIdx.x; q < pages; q += gridDim.x * blockDim.x)
        hdr[q] = kUnused;
}

// ranges of a pass, and the pages its outputs can need
uint64_t ranges_of(tid_ctx *ctx, uint64_t n, uint64_t *range) {
    const uint64_t tiles = (n + kPgTile - 1) / kPgTile;
    const uint64_t resident = 2ull * (uint64_t)device_cus(ctx);  // 512 threads, two to a CU
    uint64_t P = std::max<uint64_t>(1, std::min<uint64_t>({tiles, resident, kPgMaxRanges}));
    *range = (tiles + P - 1) / P * kPgTile;
    return (n + *range - 1) / *range;
}

uint64_t pages_bound(uint64_t P, tid_table *const *outs, int k) {
    uint64_t pages = P * kPoolPages;  // taken and not needed
    for (int j = 0; j < k; ++j)       // every range can leave one page part filled
        if (outs[j]->ncols) pages += outs[j]->cap / kPageRows + P;
    return pages;
}

// pages of a pass are taken from the pool while it runs: larger passes (and
// graphs of 2^32 triples or more) stay with the kernels that write in place
constexpr uint64_t kMaxPageBytes = 4ull << 30;

}  // namespace

// Whether one paged pass can answer the patterns: the tables must hold every
// row the histograms allow, since pages are sized by the tables.
bool scan_pages_ok(tid_ctx *ctx, const tid_graph *g, int k, tid_table *const *outs) {
    if (k < 2 || k > TID_MAX_MULTI || g->n == 0 || g->n >= (1ull << 32)) return false;
    uint64_t range;
    const uint64_t P = ranges_of(ctx, g->n, &range);
    return pages_bound(P, outs, k) * 12 * kPageRows <= kMaxPageBytes;
}

// two patterns that hold different constants at one position match no triple both
static bool apart(const tid_pattern &p, const tid_pattern &q) {
    return (p.s && q.s && p.s != q.s) || (p.p && q.p && p.p != q.p) || (p.o && q.o && p.o != q.o);
}

// a constant predicate, and nothing else to test
static bool predicate_alone(const DevPattern &d) {
    bool only = d.msk[1] != 0 && d.key[1] != 0 && d.msk[0] == 0 && d.msk[2] == 0 && d.eq == 0 &&
                d.set_pos < 0 && d.fpos < 0;
    for (int x = 0; x < 3; ++x) only &= d.rlo[x] == 0 && d.rmax[x] == 0xFFFFFFFFu;
    return only;
}

// Whether the paged pass is the better one also where the staged one holds every
// row: for the rows of several predicates, whose tests it does with one compare
// or table read a triple.  Staged / paged, 0.1% of the triples or less out
// (1%), in us:
//                 2 patterns      3               4
//   1M triples     31 /  34       38 /  38        43 /  42
//   4M             45 /  45       56 /  48        64 /  52
//   30M           114 /  91      166 /  94       204 /  99   (276 / 123)
//   100M          285 / 218      445 / 221       563 / 226
// Patterns with other tests as well are the staged pass's (two ranges of one
// predicate on 30M triples: 132 / 171).
bool scan_pages_better(const tid_graph *g, const tid_pattern *pats, int k, const PatternSet *sets,
                       const ScanFilter *filters) {
    for (int j = 0; j < k; ++j) {
        if (!predicate_alone(compile_pattern(pats[j], sets ? &sets[j] : nullptr,
                                             filters ? &filters[j] : nullptr)))
            return false;
        for (int i = 0; i < j; ++i)
            if (!apart(pats[i], pats[j])) return false;
    }
    return k > 2 || g->n >= (1ull << 22);
}

// The pass; false, and nothing done, if there is no memory for the pages.
bool run_scan_pages(tid_ctx *ctx, const tid_graph *g, const tid_pattern *pats, int k,
                    tid_table *const *outs, const PatternSet *sets, const ScanFilter *filters) {
    PageArgs a{};
    PageGather b{};
    const uint64_t P = ranges_of(ctx, g->n, &a.range);
    const uint64_t pages = pages_bound(P, outs, k);
    bool disjoint = true, preds = true, used[3] = {false, false, false};
    for (int j = 0; j < k; ++j) {
        DevPattern &d = a.pat[j];
        d = compile_pattern(pats[j], sets ? &sets[j] : nullptr, filters ? &filters[j] : nullptr);
        a.kind[j] = d.msk[1] != 0 && d.key[1] != 0 ? kPredicateFirst : kGeneral;
        preds &= predicate_alone(d);
        for (int i = 0; i < j; ++i) disjoint &= apart(pats[i], pats[j]);
        // a value set stands where the pattern holds one of its constants
        disjoint &= d.set_pos < 0;
        for (int c = 0; c < d.ncols; ++c) used[d.src[c]] = true;
        b.out[j].cap = outs[j]->cap;
        b.out[j].count = outs[j]->d_count;
        b.out[j].ncols = outs[j]->ncols;
    }
    preds &= disjoint;
    if (preds) used[0] = used[2] = true;  // both planes are written
    const size_t o_cnt = 256, o_hdr = align_up(o_cnt + (size_t)k * P * 4);
    const size_t o_data = align_up(o_hdr + pages * 8);
    const size_t plane = (size_t)pages * kPageRows * 4;
    DevBuf buf;
    try {
        buf = DevBuf(ctx, o_data + plane * (size_t)(used[0] + used[1] + used[2]) + 4);
    } catch (const Error &) {
        return false;
    }
    char *base = buf.get<char>(), *at = base + o_data;
    for (int x = 0; x < 3; ++x)
        if (used[x]) {
            a.plane[x] = reinterpret_cast<uint32_t *>(at);
            at += plane;
        }
    for (int j = 0; j < k; ++j)
        for (int c = 0; c < outs[j]->ncols; ++c) {
            b.out[j].col[c] = outs[j]->col[c];
            b.out[j].plane[c] = a.plane[a.pat[j].src[c]];
        }
    a.k = b.k = k;
    a.P = b.P = (uint32_t)P;
    a.g = g->triples();
    a.n = g->n;
    a.flags = ctx->d_flags;
    a.max_pages = b.max_pages = (uint32_t)pages;
    b.npages = a.npages = reinterpret_cast<uint32_t *>(base);
    b.cnt = a.cnt = reinterpret_cast<uint32_t *>(base + o_cnt);
    b.hdr = a.hdr = reinterpret_cast<uint64_t *>(base + o_hdr);
    hipLaunchKernelGGL(clear_pages, dim3((unsigned)std::min<uint64_t>((pages + 255) / 256, 1024)),
                       dim3(256), 0, ctx->stream, a.npages, a.hdr, (uint32_t)pages);
    TID_HIP(hipGetLastError());
    const bool ext = any_ext(k, sets, filters);
    bool table = preds && k > kFewKeys;
    for (int j = 0; j < k; ++j) table &= a.pat[j].key[1] < kTableIds;
    auto kern = table   ? table_to_pages
                : preds ? predicates_to_pages
                : ext ? (disjoint ? scan_to_pages<true, true> : scan_to_pages<true, false>)
                      : (disjoint ? scan_to_pages<false, true> : scan_to_pages<false, false>);
    hipLaunchKernelGGL(kern, dim3((uint32_t)P), dim3(kPgBlock), 0, ctx->stream, a);
    TID_HIP(hipGetLastError());
    const unsigned grid =
        (unsigned)std::max<uint64_t>(k, std::min<uint64_t>(pages, 8ull * device_cus(ctx)));
    hipLaunchKernelGGL(pages_to_tables, dim3(grid), dim3(kGatherBlock), 0, ctx->stream, b);
    TID_HIP(hipGetLastError());
    return true;
}

}  // namespace tid
