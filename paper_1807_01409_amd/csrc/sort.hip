// sort.hip -- stable LSD radix sort of 64-bit keys, alone or with 32-bit
// values, the row sorts built on it and on the merge sort of rowsort.hip (the canonical
// lexicographic order, DISTINCT), and union.
//
// The paper sorts subquery results before joining them and merges final
// results to distinct values (Sec. 4.2 step 3 with Mgpu's mergesort, Sec. 4.3
// DISTINCT).  The radix sort, written for wave64, orders the triples of the
// partitioned layout, the build sides of large joins, sort-merge joins and rows
// too wide for packed keys.  A pass over a digit of at most 9 bits (10 where
// that spares a pass):
//   hist     each workgroup owns one contiguous range of the input and counts
//            the digits of its range in LDS;
//   offsets  one workgroup per digit scans that digit's counts over the
//            ranges; the scatter kernel adds the bases of the smaller digits
//            to find, for every (range, digit), the place where its first
//            element goes;
//   scatter  each workgroup walks its range tile by tile, finds every
//            element's stable rank with ballots that group the lanes holding
//            equal digits, puts the tile in digit order in LDS and writes each
//            digit's run to its place.
// Up to 8192 pairs are sorted by one workgroup instead, every pass in LDS,
// in one launch (small sorts are otherwise bound by launches, three a pass).
// A row of k columns is sorted as one or more packed 64-bit keys (as many
// leading columns as fit their bit widths), least significant group first,
// carrying the row permutation as the value.
#include "batch.hpp"
#include "compact.hpp"

#include <algorithm>
#include <mutex>
#include <numeric>

namespace tid {

bool rows_mergeable(const tid_table *t, uint64_t n);
bool merge_sort_rows(tid_ctx *ctx, const tid_table *in, uint64_t n, tid_table *out, int distinct);
std::vector<RowSortJob> merge_sort_rows_batched(tid_ctx *ctx, const std::vector<RowSortJob> &all,
                                                std::vector<DevBuf> &keep,
                                                std::vector<std::vector<char>> &host_keep);

constexpr int kRadixBits = 8;                 // digit of the small sort
constexpr uint32_t kRadix = 1u << kRadixBits;
constexpr int kDigitBits = 9;                 // widest digit of a pass over memory,
constexpr int kWideBits = 10;                 // and where that spares a pass
constexpr int kSortBlock = 512;
constexpr int kSortIPT = 8;
constexpr int kSortNW = kSortBlock / dev::kWave;
constexpr uint32_t kSortTile = (uint32_t)kSortBlock * kSortIPT;

// item `it` of lane `lane` in wave `wave` of a tile: each wave owns 64*IPT
// consecutive items, so every load instruction reads 64 consecutive items
__device__ __forceinline__ uint32_t sort_item(int wave, int it, int lane) {
    return (uint32_t)(wave * (dev::kWave * kSortIPT) + it * dev::kWave + lane);
}

// Digit counts of every range.  A digit has kCopies counters side by side and a
// lane adds to the one of its number: lanes with different digits in one bank
// are then few.  50M keys took 293 us with the ballots of the scatter in place
// of LDS atomics, 114 us with a set of counters a wave, now 93.
template <class In, int BITS>
__global__ __launch_bounds__(kSortBlock) void radix_hist(In in, uint64_t n, uint64_t range,
                                                          int shift, int nbits,
                                                          uint32_t *counts) {
    constexpr uint32_t kCopies = 8192u >> BITS;  // 32 KB of counters
    __shared__ uint32_t s_h[kCopies << BITS];
    const int tid = threadIdx.x, wave = tid / dev::kWave, lane = tid % dev::kWave;
    const uint32_t R = 1u << nbits, copy = lane % kCopies;
    for (uint32_t d = tid; d < R * kCopies; d += kSortBlock) s_h[d] = 0;
    __syncthreads();
    const uint32_t w = blockIdx.x;
    const uint64_t r0 = (uint64_t)w * range, r1 = min(n, r0 + range);
    for (uint64_t t0 = r0; t0 < r1; t0 += kSortTile) {
        const In at = in.from(t0);
        const uint32_t cnt = (uint32_t)min((uint64_t)kSortTile, r1 - t0);
        if (cnt == kSortTile) {
            uint32_t d[kSortIPT];
#pragma unroll
            for (int it = 0; it < kSortIPT; ++it)
                d[it] = (uint32_t)(at.key(sort_item(wave, it, lane)) >> shift) & (R - 1);
#pragma unroll
            for (int it = 0; it < kSortIPT; ++it) atomicAdd(&s_h[d[it] * kCopies + copy], 1u);
        } else {
            for (int it = 0; it < kSortIPT; ++it) {
                const uint32_t i = sort_item(wave, it, lane);
                if (i < cnt)
                    atomicAdd(&s_h[((uint32_t)(at.key(i) >> shift) & (R - 1)) * kCopies + copy],
                              1u);
            }
        }
    }
    __syncthreads();
    for (uint32_t dd = tid; dd < R; dd += kSortBlock) {
        uint32_t s = 0;
        for (uint32_t c = 0; c < kCopies; ++c) s += s_h[dd * kCopies + (c + dd) % kCopies];
        counts[(size_t)w * R + dd] = s;
    }
}

// Where each (range, digit) goes is base[d] + scan[w][d]: base[d] counts every
// element of a smaller digit, scan[w][d] the elements of digit d in ranges
// before w.  One workgroup per digit scans its column of the range-major count
// matrix and writes the digit's total; the scatter kernel turns the totals into
// bases itself.
constexpr int kColThreads = 256;
__global__ __launch_bounds__(kColThreads) void digit_scan(const uint32_t *__restrict__ counts,
                                                           uint32_t *__restrict__ scan,
                                                           uint32_t *__restrict__ totals,
                                                           uint32_t P) {
    __shared__ uint32_t s_w[kColThreads / dev::kWave];
    const uint32_t d = blockIdx.x, R = gridDim.x;
    const int tid = threadIdx.x, wave = tid / dev::kWave, lane = tid % dev::kWave;
    const uint32_t per = (P + kColThreads - 1) / kColThreads;
    const uint32_t w0 = min(P, (uint32_t)tid * per), w1 = min(P, w0 + per);
    uint32_t sum = 0;
    for (uint32_t w = w0; w < w1; ++w) sum += counts[(size_t)w * R + d];
    const uint32_t incl = dev::wave_inclusive_sum(sum);
    if (lane == dev::kWave - 1) s_w[wave] = incl;
    __syncthreads();
    uint32_t run = incl - sum;
    for (int x = 0; x < wave; ++x) run += s_w[x];
    for (uint32_t w = w0; w < w1; ++w) {
        const uint32_t c = counts[(size_t)w * R + d];
        scan[(size_t)w * R + d] = run;
        run += c;
    }
    if (tid == kColThreads - 1) totals[d] = run;
}

// The stable scatter.  A tile is put in digit order in LDS first, so that the
// lanes of a wave write runs of consecutive places (on average tile / digits
// items, 64-200 B of keys): the same pass with every lane writing its own item
// to its place took 407 us for 50M pairs of 8-bit digits, now 392 us for 9-bit
// ones, and keys alone 287 us.  Keys and values go through the same LDS one
// after the other, which leaves three workgroups to a CU; what hides the
// latencies is those workgroups: tiles twice as large (347 us for keys alone),
// six waves to a SIMD and, with pairs, requesting the next tile early were
// slower.
template <class In, class Out, int BITS>
__global__ __launch_bounds__(kSortBlock) void radix_scatter(In in, Out out, uint64_t n,
                                                             uint64_t range, int shift, int nbits,
                                                             const uint32_t *scan,
                                                             const uint32_t *totals) {
    constexpr uint32_t kMaxDigits = 1u << BITS;
    constexpr int kPer = kMaxDigits > kSortBlock ? kMaxDigits / kSortBlock : 1;
    __shared__ uint64_t s_item[kSortTile];
    __shared__ uint16_t s_wh[kSortNW][kMaxDigits];  // a wave's items per digit, then those before
    __shared__ uint32_t s_run[kMaxDigits];          // where the range's next item of a digit goes
    __shared__ uint32_t s_loc[kMaxDigits];          // first item of a digit in the sorted tile
    __shared__ uint32_t s_off[kMaxDigits];          // place of sorted item i: s_off[digit] + i
    __shared__ uint32_t s_w[kSortNW];
    const uint32_t tid = threadIdx.x;
    const int wave = tid / dev::kWave, lane = tid % dev::kWave;
    const uint32_t R = 1u << nbits, w = blockIdx.x;
    // exclusive sums over the digits (a thread's kPer digits at x), in place
    auto digit_prefix = [&](uint32_t (&x)[kPer]) {
        uint32_t sum = 0;
#pragma unroll
        for (int q = 0; q < kPer; ++q) sum += x[q];
        const uint32_t incl = dev::wave_inclusive_sum(sum);
        if (lane == dev::kWave - 1) s_w[wave] = incl;
        __syncthreads();
        uint32_t run = incl - sum;
#pragma unroll
        for (int y = 0; y < kSortNW; ++y) run += y < wave ? s_w[y] : 0u;
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const uint32_t c = x[q];
            x[q] = run;
            run += c;
        }
    };
    {
        uint32_t base[kPer];
#pragma unroll
        for (int q = 0; q < kPer; ++q) base[q] = tid * kPer + q < R ? totals[tid * kPer + q] : 0u;
        digit_prefix(base);
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const uint32_t d = tid * kPer + q;
            if (d < R) s_run[d] = base[q] + scan[(size_t)w * R + d];
        }
    }
    const uint64_t r0 = (uint64_t)w * range, r1 = min(n, r0 + range);
    const uint64_t lt = (1ull << lane) - 1ull;
    for (uint64_t t0 = r0; t0 < r1; t0 += kSortTile) {
        uint64_t key[kSortIPT];
        uint32_t val[kSortIPT], rank[kSortIPT];
        const In tile = in.from(t0);
        const uint32_t cnt = (uint32_t)min((uint64_t)kSortTile, r1 - t0);
        if (cnt == kSortTile) {
#pragma unroll
            for (int it = 0; it < kSortIPT; ++it)
                tile.load(sort_item(wave, it, lane), key[it], val[it]);
        } else {
#pragma unroll
            for (int it = 0; it < kSortIPT; ++it) {
                const uint32_t i = sort_item(wave, it, lane);
                key[it] = 0;
                val[it] = 0;
                if (i < cnt) tile.load(i, key[it], val[it]);
            }
        }
        for (uint32_t d = lane; d < R; d += dev::kWave) s_wh[wave][d] = 0;
#pragma unroll
        for (int it = 0; it < kSortIPT; ++it) {
            const bool valid = sort_item(wave, it, lane) < cnt;
            const uint32_t d = (uint32_t)(key[it] >> shift) & (R - 1);
            const uint64_t peers = dev::match_digit<BITS>(d, valid, nbits);
            const uint32_t before = valid ? s_wh[wave][d] : 0u;
            rank[it] = before + (uint32_t)__popcll(peers & lt);
            if (valid && lane == __builtin_ctzll(peers))
                s_wh[wave][d] = (uint16_t)(before + (uint32_t)__popcll(peers));
        }
        __syncthreads();
        uint32_t tot[kPer], loc[kPer];
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const uint32_t d = tid * kPer + q;
            tot[q] = 0;
            if (d < R)
                for (int ww = 0; ww < kSortNW; ++ww) {  // waves in item order
                    const uint32_t c = s_wh[ww][d];
                    s_wh[ww][d] = (uint16_t)tot[q];
                    tot[q] += c;
                }
            loc[q] = tot[q];
        }
        digit_prefix(loc);
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const uint32_t d = tid * kPer + q;
            if (d < R) {
                const uint32_t run = s_run[d];
                s_loc[d] = loc[q];
                s_off[d] = run - loc[q];
                s_run[d] = run + tot[q];
            }
        }
        __syncthreads();
        uint32_t at[kSortIPT];
#pragma unroll
        for (int it = 0; it < kSortIPT; ++it) {
            const uint32_t d = (uint32_t)(key[it] >> shift) & (R - 1);
            at[it] = s_loc[d] + s_wh[wave][d] + rank[it];
            if (sort_item(wave, it, lane) < cnt) s_item[at[it]] = key[it];
        }
        __syncthreads();
        if constexpr (!In::kPairs) {
#pragma unroll
            for (int u = 0; u < kSortIPT; ++u) {
                const uint32_t i = u * kSortBlock + tid;
                if (i < cnt) {
                    const uint64_t k = s_item[i];
                    out.put(s_off[(uint32_t)(k >> shift) & (R - 1)] + i, k, 0);
                }
            }
            __syncthreads();
            continue;
        }
        uint64_t skey[kSortIPT];
#pragma unroll
        for (int u = 0; u < kSortIPT; ++u) skey[u] = s_item[u * kSortBlock + tid];
        __syncthreads();
        uint32_t *s_val = reinterpret_cast<uint32_t *>(s_item);
#pragma unroll
        for (int it = 0; it < kSortIPT; ++it)
            if (sort_item(wave, it, lane) < cnt) s_val[at[it]] = val[it];
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kSortIPT; ++u) {
            const uint32_t i = u * kSortBlock + tid;
            if (i < cnt) {
                const uint32_t d = (uint32_t)(skey[u] >> shift) & (R - 1);
                out.put(s_off[d] + i, skey[u], s_val[i]);
            }
        }
        __syncthreads();
    }
}

// where a pass takes its pairs (or its keys alone) from, and where it puts them
struct PairIn {
    static constexpr bool kPairs = true;
    const uint64_t *k;
    const uint32_t *v;
    __device__ __forceinline__ PairIn from(uint64_t t0) const { return PairIn{k + t0, v + t0}; }
    __device__ __forceinline__ uint64_t key(uint32_t i) const { return k[i]; }
    __device__ __forceinline__ void load(uint32_t i, uint64_t &key, uint32_t &val) const {
        key = k[i];
        val = v[i];
    }
};

struct PairOut {
    uint64_t *k;
    uint32_t *v;
    __device__ __forceinline__ void put(uint32_t at, uint64_t key, uint32_t val) const {
        k[at] = key;
        v[at] = val;
    }
};

// 32-bit keys (v null: the item's number)
struct KeyIn {
    static constexpr bool kPairs = true;
    const uint32_t *k, *v;
    uint32_t first;
    __device__ __forceinline__ KeyIn from(uint64_t t0) const {
        return KeyIn{k + t0, v ? v + t0 : nullptr, first + (uint32_t)t0};
    }
    __device__ __forceinline__ uint64_t key(uint32_t i) const { return k[i]; }
    __device__ __forceinline__ void load(uint32_t i, uint64_t &key, uint32_t &val) const {
        key = k[i];
        val = v ? v[i] : first + i;
    }
};

struct KeyOut {
    uint32_t *k, *v;
    __device__ __forceinline__ void put(uint32_t at, uint64_t key, uint32_t val) const {
        k[at] = (uint32_t)key;
        v[at] = val;
    }
};

// a triple as (its predicate and, below it in `bits` bits, the value at position
// lo, 0 or 2; the value at the other one)
struct TripleIn {
    static constexpr bool kPairs = true;
    const uint32_t *g;
    int32_t lo, bits;
    __device__ __forceinline__ TripleIn from(uint64_t t0) const {
        return TripleIn{g + 3 * t0, lo, bits};
    }
    __device__ __forceinline__ uint64_t key(uint32_t i) const {
        const uint32_t *t = g + 3 * i;
        return (uint64_t)t[1] << bits | (lo == 0 ? t[0] : t[2]);
    }
    __device__ __forceinline__ void load(uint32_t i, uint64_t &key, uint32_t &val) const {
        const uint32_t *t = g + 3 * i;
        const uint32_t s = t[0], p = t[1], o = t[2];  // one 12-byte load
        key = (uint64_t)p << bits | (lo == 0 ? s : o);
        val = lo == 0 ? o : s;
    }
};

// a whole triple in a key: the predicate, below it the value at position lo (0
// or 2), below that, in `bits` bits, the other one
struct PackIn {
    static constexpr bool kPairs = false;
    const uint32_t *g;
    int32_t lo, lo_bits, bits;
    __device__ __forceinline__ PackIn from(uint64_t t0) const {
        return PackIn{g + 3 * t0, lo, lo_bits, bits};
    }
    __device__ __forceinline__ uint64_t key(uint32_t i) const {
        const uint32_t *t = g + 3 * i;
        const uint32_t s = t[0], p = t[1], o = t[2];  // one 12-byte load
        const uint64_t a = lo == 0 ? s : o, b = lo == 0 ? o : s;
        return ((uint64_t)p << lo_bits | a) << bits | b;
    }
    __device__ __forceinline__ void load(uint32_t i, uint64_t &k, uint32_t &) const { k = key(i); }
};

struct WordIn {
    static constexpr bool kPairs = false;
    const uint64_t *k;
    __device__ __forceinline__ WordIn from(uint64_t t0) const { return WordIn{k + t0}; }
    __device__ __forceinline__ uint64_t key(uint32_t i) const { return k[i]; }
    __device__ __forceinline__ void load(uint32_t i, uint64_t &key, uint32_t &) const { key = k[i]; }
};

struct WordOut {
    uint64_t *k;
    __device__ __forceinline__ void put(uint32_t at, uint64_t key, uint32_t) const { k[at] = key; }
};

// PackIn's keys back to two columns
struct UnpackOut {
    uint32_t *lo, *hi;
    int32_t bits;
    uint32_t lo_mask, mask;
    __device__ __forceinline__ void put(uint32_t at, uint64_t key, uint32_t) const {
        lo[at] = (uint32_t)(key >> bits) & lo_mask;
        hi[at] = (uint32_t)key & mask;
    }
};

struct ColumnsOut {
    uint32_t *lo, *hi;
    uint64_t mask;
    __device__ __forceinline__ void put(uint32_t at, uint64_t key, uint32_t val) const {
        lo[at] = (uint32_t)(key & mask);
        hi[at] = val;
    }
};

// One workgroup sorts n <= kSmallBlock * kSmallIPT pairs on key bits
// [0, bits), in place: the pairs stay in LDS between passes, and each pass
// ranks items like the scatter kernel (waves in item order, ballots within a
// wave) and writes them back to LDS at their new places.
constexpr int kSmallBlock = 1024;
constexpr int kSmallIPT = 8;
constexpr int kSmallNW = kSmallBlock / dev::kWave;
constexpr uint64_t kSmallMax = (uint64_t)kSmallBlock * kSmallIPT;
constexpr size_t kSmallLds = kSmallMax * 12 + (size_t)kSmallNW * kRadix * 4 + kRadix * 4;

// item `it` of lane `lane` in wave `wave`: each wave owns 64 * kSmallIPT
// consecutive items
__device__ __forceinline__ uint32_t small_item(int wave, int it, int lane) {
    return (uint32_t)(wave * (dev::kWave * kSmallIPT) + it * dev::kWave + lane);
}

__global__ __launch_bounds__(kSmallBlock) void small_sort(uint64_t *keys, uint32_t *vals,
                                                          uint32_t n, int bits) {
    extern __shared__ __attribute__((aligned(16))) uint32_t lds[];
    uint64_t *s_key = reinterpret_cast<uint64_t *>(lds);
    uint32_t *s_val = lds + 2 * kSmallMax;
    uint32_t(*s_wh)[kRadix] = reinterpret_cast<uint32_t(*)[kRadix]>(s_val + kSmallMax);
    uint32_t *s_run = s_val + kSmallMax + kSmallNW * kRadix;
    const int tid = threadIdx.x, wave = tid / dev::kWave, lane = tid % dev::kWave;
    const uint64_t lt = (1ull << lane) - 1ull;
    constexpr int kPer = kRadix / dev::kWave;
    for (int shift = 0; shift < bits; shift += kRadixBits) {
        uint64_t key[kSmallIPT];
        uint32_t val[kSmallIPT], rank[kSmallIPT];
#pragma unroll
        for (int it = 0; it < kSmallIPT; ++it) {
            const uint32_t i = small_item(wave, it, lane);
            key[it] = 0;
            val[it] = 0;
            if (i < n) {
                key[it] = shift == 0 ? keys[i] : s_key[i];
                val[it] = shift == 0 ? vals[i] : s_val[i];
            }
        }
        for (uint32_t d = lane; d < kRadix; d += dev::kWave) s_wh[wave][d] = 0;
#pragma unroll
        for (int it = 0; it < kSmallIPT; ++it) {
            const bool valid = small_item(wave, it, lane) < n;
            const uint32_t d = (uint32_t)(key[it] >> shift) & (kRadix - 1);
            const uint64_t peers = dev::match_digit<kRadixBits>(d, valid);
            const uint32_t before = valid ? s_wh[wave][d] : 0u;
            rank[it] = before + (uint32_t)__popcll(peers & lt);
            if (valid && lane == __builtin_ctzll(peers)) s_wh[wave][d] = before + (uint32_t)__popcll(peers);
        }
        __syncthreads();  // every item is in registers and every wave has counted
        if (tid < (int)kRadix) {
            uint32_t t = 0;
            for (int w = 0; w < kSmallNW; ++w) t += s_wh[w][tid];
            s_run[tid] = t;
        }
        __syncthreads();
        if (wave == 0) {  // digit totals -> digit bases
            uint32_t v[kPer], loc = 0;
#pragma unroll
            for (int x = 0; x < kPer; ++x) {
                v[x] = s_run[lane * kPer + x];
                loc += v[x];
            }
            uint32_t run = dev::wave_inclusive_sum(loc) - loc;
#pragma unroll
            for (int x = 0; x < kPer; ++x) {
                s_run[lane * kPer + x] = run;
                run += v[x];
            }
        }
        __syncthreads();
        if (tid < (int)kRadix) {  // per-wave bases of each digit, waves in item order
            uint32_t run = s_run[tid];
            for (int w = 0; w < kSmallNW; ++w) {
                const uint32_t c = s_wh[w][tid];
                s_wh[w][tid] = run;
                run += c;
            }
        }
        __syncthreads();
#pragma unroll
        for (int it = 0; it < kSmallIPT; ++it) {
            if (small_item(wave, it, lane) < n) {
                const uint32_t d = (uint32_t)(key[it] >> shift) & (kRadix - 1);
                const uint32_t pos = s_wh[wave][d] + rank[it];
                s_key[pos] = key[it];
                s_val[pos] = val[it];
            }
        }
        __syncthreads();  // the next pass reads the new order
    }
    for (uint32_t i = tid; i < n; i += kSmallBlock) {
        keys[i] = s_key[i];
        vals[i] = s_val[i];
    }
}

__global__ void iota_u32(uint32_t *v, uint64_t n) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        v[i] = (uint32_t)i;
}

struct PackArgs {
    const uint32_t *col[TID_MAX_COLS];
    int shift[TID_MAX_COLS];
    int ncols;
};

// key[i] = concatenation of the group's columns of row perm[i] (or row i)
__global__ void pack_keys(PackArgs a, const uint32_t *perm, uint64_t n, uint64_t *key) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint64_t r = perm ? perm[i] : i;
        uint64_t k = 0;
        for (int c = 0; c < a.ncols; ++c) k |= (uint64_t)a.col[c][r] << a.shift[c];
        key[i] = k;
    }
}

struct GatherArgs {
    const uint32_t *in[TID_MAX_COLS];
    uint32_t *out[TID_MAX_COLS];
    int ncols;
};

__global__ void gather_rows(GatherArgs a, const uint32_t *perm, uint64_t n) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint32_t r = perm[i];
        for (int c = 0; c < a.ncols; ++c) a.out[c][i] = a.in[c][r];
    }
}

// per-column maximum: one atomic per workgroup after an LDS reduction
__global__ __launch_bounds__(256) void column_max(const uint32_t *const *cols, uint64_t n,
                                                   uint32_t *mx) {
    __shared__ uint32_t s_m[4];
    const uint32_t *col = cols[blockIdx.y];
    uint32_t m = 0;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        m = max(m, col[i]);
    for (int d = 32; d >= 1; d >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, d, 64));
    if (dev::lane_id() == 0) s_m[threadIdx.x / 64] = m;
    __syncthreads();
    if (threadIdx.x == 0) atomicMax(&mx[blockIdx.y], max(max(s_m[0], s_m[1]), max(s_m[2], s_m[3])));
}

__global__ void fill_u32(uint32_t *p, uint64_t n, uint32_t v) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}

// rows of a sorted table that differ from the row before them
struct UniqueSrc {
    const uint32_t *col[TID_MAX_COLS];
    int ncols;
    uint64_t n;
    using Item = uint64_t;
    __device__ __forceinline__ Item load(uint64_t i) const { return i; }
    __device__ __forceinline__ bool match(int, Item i) const {
        if (i == 0) return true;
        for (int c = 0; c < ncols; ++c)
            if (col[c][i] != col[c][i - 1]) return true;
        return false;
    }
    __device__ __forceinline__ uint32_t value(int, int c, Item i, uint64_t) const {
        return col[c][i];
    }
};

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

static unsigned grid_for(uint64_t n, unsigned block = 256, unsigned cap = 8192) {
    return (unsigned)std::max<uint64_t>(1, std::min<uint64_t>((n + block - 1) / block, cap));
}

void fill(tid_ctx *ctx, uint32_t *p, uint64_t n, uint32_t v) {
    if (!n) return;
    hipLaunchKernelGGL(fill_u32, dim3(grid_for(n)), dim3(256), 0, ctx->stream, p, n, v);
    TID_HIP(hipGetLastError());
}

void iota(tid_ctx *ctx, uint32_t *p, uint64_t n) {
    if (!n) return;
    hipLaunchKernelGGL(iota_u32, dim3(grid_for(n)), dim3(256), 0, ctx->stream, p, n);
    TID_HIP(hipGetLastError());
}

// digit_scan of a matrix of `ranges` rows of `digits` counts
void scan_digits(tid_ctx *ctx, const uint32_t *counts, uint32_t *scan, uint32_t *totals,
                 uint32_t ranges, uint32_t digits) {
    hipLaunchKernelGGL(digit_scan, dim3(digits), dim3(kColThreads), 0, ctx->stream, counts, scan,
                       totals, ranges);
    TID_HIP(hipGetLastError());
}

// The passes of a stable sort of n pairs on key bits [first, last): digits of
// nearly equal widths, at most kWideBits, over ranges of whole tiles.
struct Passes {
    uint64_t n, range, P;
    int first, last, count, width;
    DevBuf counts, scan;
    Passes(tid_ctx *ctx, uint64_t rows, int b0, int b1) : n(rows), first(b0), last(b1) {
        auto passes = [&](int bits) { return std::max(1, (last - first + bits - 1) / bits); };
        count = std::min(passes(kDigitBits), passes(kWideBits));
        width = (last - first + count - 1) / count;
        const uint64_t tiles = (n + kSortTile - 1) / kSortTile;
        P = std::max<uint64_t>(1, std::min<uint64_t>(tiles, 3ull * device_cus(ctx)));
        range = (tiles + P - 1) / P * kSortTile;
        P = (n + range - 1) / range;
        counts = DevBuf(ctx, ((size_t)P << width) * sizeof(uint32_t));
        scan = DevBuf(ctx, ((size_t)(P + 1) << width) * sizeof(uint32_t));  // then the totals
    }
    template <class In, class Out>
    void run(tid_ctx *ctx, In in, Out out, int pass) const {
        if (width <= kDigitBits) run_bits<kDigitBits>(ctx, in, out, pass);
        else run_bits<kWideBits>(ctx, in, out, pass);
    }
    template <int BITS, class In, class Out>
    void run_bits(tid_ctx *ctx, In in, Out out, int pass) const {
        const int shift = first + pass * width, nbits = std::min(width, last - shift);
        uint32_t *totals = scan.get<uint32_t>() + ((size_t)P << nbits);
        hipLaunchKernelGGL((radix_hist<In, BITS>), dim3((uint32_t)P), dim3(kSortBlock), 0,
                           ctx->stream, in, n, range, shift, nbits, counts.get<uint32_t>());
        TID_HIP(hipGetLastError());
        scan_digits(ctx, counts.get<const uint32_t>(), scan.get<uint32_t>(), totals, (uint32_t)P,
                    1u << nbits);
        hipLaunchKernelGGL((radix_scatter<In, Out, BITS>), dim3((uint32_t)P), dim3(kSortBlock), 0,
                           ctx->stream, in, out, n, range, shift, nbits,
                           scan.get<const uint32_t>(), totals);
        TID_HIP(hipGetLastError());
    }
};

// Stable sort of n (key, value) pairs on key bits [0, bits).  The sorted pairs
// end in (k0, v0) if the return value is false, in (k1, v1) if true.
bool radix_sort_pairs(tid_ctx *ctx, uint64_t *k0, uint32_t *v0, uint64_t *k1, uint32_t *v1,
                      uint64_t n, int bits) {
    if (n <= 1 || bits <= 0) return false;
    TID_REQUIRE(n < (1ull << 32), TID_E_UNSUPPORTED, "sort: more than 2^32-1 rows");
    if (n <= kSmallMax) {
        // once per process, also when several host threads (serving workers,
        // each with its own context) reach the first small sort together
        static std::once_flag attr_once;
        std::call_once(attr_once, [] {
            TID_HIP(hipFuncSetAttribute((const void *)small_sort,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSmallLds));
        });
        hipLaunchKernelGGL(small_sort, dim3(1), dim3(kSmallBlock), kSmallLds, ctx->stream, k0, v0,
                           (uint32_t)n, bits);
        TID_HIP(hipGetLastError());
        return false;
    }
    const Passes ps(ctx, n, 0, bits);
    for (int x = 0; x < ps.count; ++x) {
        const bool flip = x & 1;
        ps.run(ctx, PairIn{flip ? k1 : k0, flip ? v1 : v0}, PairOut{flip ? k0 : k1, flip ? v0 : v1},
               x);
    }
    return ps.count & 1;
}

// Sort of n 64-bit words on bits [0, bits): in k0 if the return value is false,
// in k1 if true.
bool sort_words(tid_ctx *ctx, uint64_t *k0, uint64_t *k1, uint64_t n, int bits) {
    TID_REQUIRE(n >= 1 && n < (1ull << 32) && bits >= 1, TID_E_UNSUPPORTED,
                "sort: more than 2^32-1 rows");
    const Passes ps(ctx, n, 0, bits);
    for (int x = 0; x < ps.count; ++x)
        ps.run(ctx, WordIn{x & 1 ? k1 : k0}, WordOut{x & 1 ? k0 : k1}, x);
    return ps.count & 1;
}

// A column's values in ascending order and their rows (stable), on key bits
// [0, bits): in (k0, v0) if the return value is false, in (k1, v1) if true.
bool sort_keys32(tid_ctx *ctx, const uint32_t *col, uint64_t n, int bits, uint32_t *k0,
                 uint32_t *v0, uint32_t *k1, uint32_t *v1) {
    TID_REQUIRE(n >= 1 && n < (1ull << 32) && bits >= 1, TID_E_UNSUPPORTED,
                "sort: more than 2^32-1 rows");
    const Passes ps(ctx, n, 0, bits);
    for (int x = 0; x < ps.count; ++x) {
        const KeyOut out{x & 1 ? k1 : k0, x & 1 ? v1 : v0};
        if (x == 0) ps.run(ctx, KeyIn{col, nullptr, 0}, out, x);
        else ps.run(ctx, KeyIn{x & 1 ? k0 : k1, x & 1 ? v0 : v1, 0}, out, x);
    }
    return (ps.count & 1) == 0;
}

// The subject and object columns of the n triples in (predicate, value) order,
// stably: by_value = 0 predicate alone, else its subject (pos 0) or object (pos
// 2) too.  bits: width of the IDs of each position.  The first pass reads the
// triples, the last one writes the columns; between them a triple is one 64-bit
// key if its IDs fit (scratch k0, k1 of n words), else a pair of predicate and
// value and the other position (also v0, v1).  50M triples, all three orders,
// 1000 predicates: 5.07 ms with pairs and digits of at most 9 bits, now 3.97.
bool triples_pack(const int (&bits)[3]) { return bits[0] + bits[1] + bits[2] <= 64; }

void order_triples(tid_ctx *ctx, const uint32_t *g, uint64_t n, const int (&bits)[3], int by_value,
                   int pos, uint64_t *k0, uint32_t *v0, uint64_t *k1, uint32_t *v1, uint32_t *s,
                   uint32_t *o) {
    TID_REQUIRE(n < (1ull << 32), TID_E_UNSUPPORTED, "sort: more than 2^32-1 rows");
    if (n == 0) return;
    uint32_t *lo = pos == 0 ? s : o, *hi = pos == 0 ? o : s;
    auto sort = [&](const Passes &ps, auto in, auto mid_in, auto mid_out, auto out) {
        for (int x = 0; x < ps.count; ++x) {
            if (x == 0 && ps.count == 1) ps.run(ctx, in, out, x);
            else if (x == 0) ps.run(ctx, in, mid_out(x), x);
            else if (x + 1 == ps.count) ps.run(ctx, mid_in(x), out, x);
            else ps.run(ctx, mid_in(x), mid_out(x), x);
        }
    };
    auto from = [&](int x) { return x & 1 ? k0 : k1; };
    auto to = [&](int x) { return x & 1 ? k1 : k0; };
    if (triples_pack(bits)) {
        const int nlo = bits[pos], nhi = bits[2 - pos];
        const Passes ps(ctx, n, nhi + (by_value ? 0 : nlo), nhi + nlo + bits[1]);
        sort(ps, PackIn{g, pos, nlo, nhi}, [&](int x) { return WordIn{from(x)}; },
             [&](int x) { return WordOut{to(x)}; },
             UnpackOut{lo, hi, nhi, (uint32_t)((1ull << nlo) - 1), (uint32_t)((1ull << nhi) - 1)});
        return;
    }
    const int below = by_value ? bits[pos] : 32;  // bits below the predicate
    const Passes ps(ctx, n, by_value ? 0 : below, below + bits[1]);
    sort(ps, TripleIn{g, pos, below},
         [&](int x) { return PairIn{from(x), x & 1 ? v0 : v1}; },
         [&](int x) { return PairOut{to(x), x & 1 ? v1 : v0}; },
         ColumnsOut{lo, hi, (1ull << below) - 1});
}

std::vector<uint32_t> column_maxima(tid_ctx *ctx, const tid_table *t, uint64_t n) {
    std::vector<uint32_t> mx(t->ncols, 0);
    if (n == 0 || t->ncols == 0) return mx;
    DevBuf cols(ctx, sizeof(uint32_t *) * t->ncols);
    DevBuf dmx(ctx, sizeof(uint32_t) * t->ncols);
    TID_HIP(hipMemcpyAsync(cols.get(), t->col, sizeof(uint32_t *) * t->ncols,
                           hipMemcpyHostToDevice, ctx->stream));
    TID_HIP(hipMemsetAsync(dmx.get(), 0, sizeof(uint32_t) * t->ncols, ctx->stream));
    hipLaunchKernelGGL(column_max, dim3(grid_for(n, 256, 512), t->ncols), dim3(256), 0,
                       ctx->stream, cols.get<const uint32_t *const>(), n, dmx.get<uint32_t>());
    TID_HIP(hipGetLastError());
    TID_HIP(hipMemcpyAsync(mx.data(), dmx.get(), sizeof(uint32_t) * t->ncols,
                           hipMemcpyDeviceToHost, ctx->stream));
    ctx->sync();
    return mx;
}

static int bit_width(uint32_t v) { return v ? 32 - __builtin_clz(v) : 0; }

// Permutation that puts the rows of t (n rows) in lexicographic order.
DevBuf sort_permutation(tid_ctx *ctx, const tid_table *t, uint64_t n) {
    // column bounds known on the host spare a device round trip
    const std::vector<uint32_t> mx =
        t->maxv_known ? std::vector<uint32_t>(t->maxv, t->maxv + t->ncols)
                      : column_maxima(ctx, t, n);
    // columns grouped from the most significant one while their widths fit 64 bits
    std::vector<std::pair<int, int>> groups;  // [first, last) columns
    int c = 0;
    while (c < t->ncols) {
        int width = 0, e = c;
        while (e < t->ncols && width + bit_width(mx[e]) <= 64) width += bit_width(mx[e++]);
        if (e == c) e = c + 1;  // unreachable: a column is at most 32 bits
        groups.emplace_back(c, e);
        c = e;
    }
    DevBuf ka(ctx, n * 8), kb(ctx, n * 8), va(ctx, n * 4), vb(ctx, n * 4);
    iota(ctx, va.get<uint32_t>(), n);
    bool perm_in_b = false;
    bool first = true;
    for (int g = (int)groups.size() - 1; g >= 0; --g) {
        PackArgs pa{};
        int shift = 0;
        for (int x = groups[g].second - 1; x >= groups[g].first; --x) {
            pa.col[pa.ncols] = t->col[x];
            pa.shift[pa.ncols] = shift;
            ++pa.ncols;
            shift += bit_width(mx[x]);
        }
        if (shift == 0) continue;  // all-zero columns order nothing
        uint32_t *perm = perm_in_b ? vb.get<uint32_t>() : va.get<uint32_t>();
        uint64_t *keys = perm_in_b ? kb.get<uint64_t>() : ka.get<uint64_t>();
        hipLaunchKernelGGL(pack_keys, dim3(grid_for(n)), dim3(256), 0, ctx->stream, pa,
                           first ? (const uint32_t *)nullptr : perm, n, keys);
        TID_HIP(hipGetLastError());
        first = false;
        const bool moved = perm_in_b
                               ? radix_sort_pairs(ctx, kb.get<uint64_t>(), vb.get<uint32_t>(),
                                                  ka.get<uint64_t>(), va.get<uint32_t>(), n, shift)
                               : radix_sort_pairs(ctx, ka.get<uint64_t>(), va.get<uint32_t>(),
                                                  kb.get<uint64_t>(), vb.get<uint32_t>(), n, shift);
        if (moved) perm_in_b = !perm_in_b;
    }
    return perm_in_b ? std::move(vb) : std::move(va);
}

// rows of src (n rows) placed in the order given by perm, into dst
void gather_table(tid_ctx *ctx, const tid_table *src, const uint32_t *perm, uint64_t n,
                  tid_table *dst) {
    if (!n || !src->ncols) return;
    GatherArgs ga{};
    ga.ncols = src->ncols;
    for (int c = 0; c < src->ncols; ++c) {
        ga.in[c] = src->col[c];
        ga.out[c] = dst->col[c];
    }
    hipLaunchKernelGGL(gather_rows, dim3(grid_for(n)), dim3(256), 0, ctx->stream, ga, perm, n);
    TID_HIP(hipGetLastError());
}

// drop rows equal to their predecessor in a sorted table
std::unique_ptr<tid_table> unique_sorted(tid_ctx *ctx, const tid_table *t, uint64_t n) {
    auto out = make_table(ctx, t->ncols, t->vars, n);
    out->maxv_known = t->maxv_known;
    copy_bounds(out.get(), t, nullptr, t->ncols);
    if (n == 0) {
        set_count(out.get(), 0);
        return out;
    }
    UniqueSrc src{};
    for (int c = 0; c < t->ncols; ++c) src.col[c] = t->col[c];
    src.ncols = t->ncols;
    src.n = n;
    CompactArgs<1, TID_MAX_COLS> a{};
    for (int c = 0; c < t->ncols; ++c) a.out[0].col[c] = out->col[c];
    a.out[0].cap = n;
    a.out[0].count = out->d_count;
    a.out[0].ncols = t->ncols;
    launch_compact<UniqueSrc, 256, 16, 1, TID_MAX_COLS>(ctx, src, a, 1, 8192);
    return out;
}

std::unique_ptr<tid_table> sort_rows(tid_ctx *ctx, const tid_table *t, uint64_t n, int distinct) {
    if (t->ncols == 0) {
        // zero-width rows are all equal
        auto out = make_table(ctx, 0, t->vars, 0);
        set_count(out.get(), distinct ? std::min<uint64_t>(n, 1) : n);
        return out;
    }
    tid_table bounded;  // a caller's own table: its column bounds are found here
    if (!t->maxv_known && n > 1) {
        bounded = *t;
        const std::vector<uint32_t> mx = column_maxima(ctx, t, n);
        std::copy(mx.begin(), mx.end(), bounded.maxv);
        bounded.maxv_known = true;
        t = &bounded;
    }
    auto sorted = make_table(ctx, t->ncols, t->vars, n);
    sorted->maxv_known = t->maxv_known;
    copy_bounds(sorted.get(), t, nullptr, t->ncols);
    if (n <= 1) {
        for (int c = 0; c < t->ncols && n; ++c)
            TID_HIP(hipMemcpyAsync(sorted->col[c], t->col[c], n * 4, hipMemcpyDeviceToDevice,
                                   ctx->stream));
        set_count(sorted.get(), n);
        return sorted;
    }
    if (rows_mergeable(t, n) && merge_sort_rows(ctx, t, n, sorted.get(), distinct)) {
        if (distinct) return sorted;  // its count is still to come
        sorted->nrows = n;
        sorted->count_known = true;
    } else {
        DevBuf perm = sort_permutation(ctx, t, n);
        gather_table(ctx, t, perm.get<const uint32_t>(), n, sorted.get());
        set_count(sorted.get(), n);
    }
    if (!distinct) return sorted;
    return unique_sorted(ctx, sorted.get(), n);
}

// Row sorts of many tables of one round.  Every table needs its column bounds
// on the host and fewer than 2^32 rows; each output table is allocated by the
// caller with n rows.  The tables the merge sort takes share its launches;
// the others are sorted one by one.  Job tables go into `keep` / `host_keep`,
// which the caller holds until the stream has passed these launches; key arrays
// and permutations go back in stream order.
void sort_rows_batched(tid_ctx *ctx, const std::vector<RowSortJob> &jobs,
                       std::vector<DevBuf> &keep, std::vector<std::vector<char>> &host_keep) {
    std::vector<RowSortJob> merged, alone;
    for (const RowSortJob &job : jobs) {
        TID_REQUIRE(job.in->maxv_known && job.n >= 1 && job.n < (1ull << 32) &&
                        job.in->ncols > 0,
                    TID_E_INTERNAL, "batched sort: bad job");
        (rows_mergeable(job.in, job.n) ? merged : alone).push_back(job);
    }
    if (merged.size() == 1) {
        if (!merge_sort_rows(ctx, merged[0].in, merged[0].n, merged[0].out, 0))
            alone.push_back(merged[0]);
    } else if (!merged.empty()) {
        for (const RowSortJob &job : merge_sort_rows_batched(ctx, merged, keep, host_keep))
            alone.push_back(job);
    }
    for (const RowSortJob &job : alone) {
        const DevBuf perm = sort_permutation(ctx, job.in, job.n);
        gather_table(ctx, job.in, perm.get<const uint32_t>(), job.n, job.out);
    }
}

std::unique_ptr<tid_table> sort_table(tid_ctx *ctx, const tid_table *t, int distinct) {
    const uint64_t n = const_cast<tid_table *>(t)->rows();
    return sort_rows(ctx, t, n, distinct);
}

// Columns of several tables put one after the other, in one launch (a copy
// each took 48 us for 16 columns of 400,000 rows).
constexpr int kPieces = 64;
struct Pieces {
    const uint32_t *src[kPieces];  // null: zeros
    uint32_t *dst[kPieces];
    uint64_t n[kPieces];
};

__global__ __launch_bounds__(256) void copy_pieces(Pieces p) {
    const uint32_t *src = p.src[blockIdx.y];
    uint32_t *dst = p.dst[blockIdx.y];
    const uint64_t n = p.n[blockIdx.y], step = (uint64_t)gridDim.x * 256;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += step)
        dst[i] = src ? src[i] : 0u;
}

// Outer union: schema = ordered union of the inputs' variables; unbound cells 0.
std::unique_ptr<tid_table> union_tables(tid_ctx *ctx, const tid_table *const *ts, int k,
                                        int dedupe) {
    std::vector<int32_t> vars;
    for (int j = 0; j < k; ++j)
        for (int c = 0; c < ts[j]->ncols; ++c)
            if (std::find(vars.begin(), vars.end(), ts[j]->vars[c]) == vars.end())
                vars.push_back(ts[j]->vars[c]);
    TID_REQUIRE((int)vars.size() <= TID_MAX_COLS, TID_E_SCHEMA, "union: too many columns");
    std::vector<tid_table *> raw(k);
    for (int j = 0; j < k; ++j) raw[j] = const_cast<tid_table *>(ts[j]);
    resolve_counts(ctx, raw.data(), k);
    uint64_t total = 0;
    for (int j = 0; j < k; ++j) total += ts[j]->nrows;
    auto out = make_table(ctx, (int)vars.size(), vars.data(), total);
    out->maxv_known = true;
    for (size_t c = 0; c < vars.size(); ++c) {
        uint32_t m = 0;
        for (int j = 0; j < k; ++j)
            for (int x = 0; x < ts[j]->ncols; ++x)
                if (ts[j]->vars[x] == vars[c]) m = std::max(m, ts[j]->maxv[x]);
        out->maxv[c] = m;
    }
    for (int j = 0; j < k; ++j) out->maxv_known &= ts[j]->maxv_known;
    Pieces p{};
    int np = 0;
    uint64_t at = 0, most = 0;
    auto flush = [&] {
        if (!np) return;
        const unsigned gx = (unsigned)std::min<uint64_t>((most + 1023) / 1024, 1024);
        hipLaunchKernelGGL(copy_pieces, dim3(gx, np), dim3(256), 0, ctx->stream, p);
        TID_HIP(hipGetLastError());
        np = 0;
        most = 0;
    };
    for (int j = 0; j < k; ++j) {
        const uint64_t n = ts[j]->nrows;
        if (!n) continue;
        for (size_t c = 0; c < vars.size(); ++c) {
            const uint32_t *src = nullptr;
            for (int x = 0; x < ts[j]->ncols; ++x)
                if (ts[j]->vars[x] == vars[c]) src = ts[j]->col[x];
            p.src[np] = src;
            p.dst[np] = out->col[c] + at;
            p.n[np] = n;
            most = std::max(most, n);
            if (++np == kPieces) flush();
        }
        at += n;
    }
    flush();
    set_count(out.get(), total);
    if (!dedupe) return out;
    return sort_rows(ctx, out.get(), total, 1);
}

}  // namespace tid
