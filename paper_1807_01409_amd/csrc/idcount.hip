// idcount.hip -- how many triples have each ID at each position, for graphs of
// some million triples (the load statistics of runtime.hip).
//
// Adding every triple to a bin per ID in global memory is bound by the chip's
// rate of scattered atomics.  Here the IDs are split by their upper bits into
// buckets of kBucketIds consecutive IDs, and a bucket's bins fit in LDS:
//   buckets  a workgroup counts, over one contiguous range of the triples, the
//            IDs of each bucket; a position with few IDs (the predicates) is
//            counted in LDS bins directly;
//   (scan)   digit_scan of sort.hip finds where each range's IDs of a bucket go;
//   split    a workgroup puts the IDs of a tile in bucket order in LDS and
//            writes their lower bits, 16 a time, to the buckets' runs;
//   count    a workgroup counts equal shares of the split IDs, bucket by
//            bucket, in LDS bins, and adds the bins to the global ones (a
//            workgroup a bucket, its bins stored, took 488 us for 234: the
//            LDS atomics bound it, and equal shares balance them).
// IDs of more than kMaxBuckets buckets take several passes over the triples.
// Bound: the split, which reads 12 bytes a triple and writes 2 a position.
// 50M triples, 5M subject and object IDs: buckets 161 us, split 328, count 234;
// with global atomics, an LDS table for the hubs before them, 3653 us.
#include "compact.hpp"

#include <algorithm>

namespace tid {

int device_cus(tid_ctx *ctx);
int resident_blocks(const void *kernel, int block, size_t lds);
void scan_digits(tid_ctx *ctx, const uint32_t *counts, uint32_t *scan, uint32_t *totals,
                 uint32_t ranges, uint32_t digits);

namespace {

constexpr int kLowBits = 15;
constexpr uint32_t kBucketIds = 1u << kLowBits;  // 128 KB of bins
constexpr uint32_t kMaxBuckets = 512;            // of a pass
constexpr uint32_t kMaxPasses = 8;
constexpr uint64_t kPassRows = 1ull << 22;
constexpr uint32_t kDirectIds = 8192;            // counted without a split
constexpr int kBlock = 512;
constexpr int kIPT = 8;
constexpr uint32_t kTile = (uint32_t)kBlock * kIPT;
constexpr int kNW = kBlock / dev::kWave;
constexpr uint32_t kCopies = 8;                  // counters of a bucket, side by side
constexpr int kCountBlock = 1024;
constexpr uint32_t kShares = 256;

enum Mode : int32_t { kNone = 0, kDirect, kSplit };

struct IdArgs {
    const uint32_t *g;
    uint64_t n, range;
    Mode mode[3];
    uint32_t ids[3];       // IDs are below this
    uint32_t buckets[3];   // of the pass, from bucket `first` on
    uint32_t first[3];
    uint32_t lds[3];       // first word of the position's counters in LDS
    uint32_t lds_words;
    uint32_t *hist[3];
    uint32_t *counts[3], *scan[3], *totals[3];
    uint16_t *low[3];      // the split IDs' lower bits
};

__global__ __launch_bounds__(kBlock) void count_buckets(IdArgs a) {
    extern __shared__ uint32_t s_cnt[];
    const uint32_t tid = threadIdx.x, copy = tid % kCopies;
    for (uint32_t i = tid; i < a.lds_words; i += kBlock) s_cnt[i] = 0;
    __syncthreads();
    const uint64_t r0 = (uint64_t)blockIdx.x * a.range, r1 = min(a.n, r0 + a.range);
    auto add = [&](const uint32_t (&v)[3]) {
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            if (a.mode[x] == kDirect) atomicAdd(&s_cnt[a.lds[x] + v[x]], 1u);
            else if (a.mode[x] == kSplit) {
                const uint32_t b = (v[x] >> kLowBits) - a.first[x];
                if (b < a.buckets[x]) atomicAdd(&s_cnt[a.lds[x] + b * kCopies + copy], 1u);
            }
        }
    };
    for (uint64_t t0 = r0; t0 < r1; t0 += kTile) {
        if (r1 - t0 >= kTile) {
            uint32_t v[kIPT][3];
#pragma unroll
            for (int u = 0; u < kIPT; ++u)
#pragma unroll
                for (int x = 0; x < 3; ++x) v[u][x] = a.g[3 * (t0 + u * kBlock + tid) + x];
#pragma unroll
            for (int u = 0; u < kIPT; ++u) add(v[u]);
        } else {
            for (uint64_t i = t0 + tid; i < r1; i += kBlock) {
                const uint32_t v[3] = {a.g[3 * i], a.g[3 * i + 1], a.g[3 * i + 2]};
                add(v);
            }
        }
    }
    __syncthreads();
    for (int x = 0; x < 3; ++x) {
        const uint32_t *s = s_cnt + a.lds[x];
        if (a.mode[x] == kDirect) {
            for (uint32_t i = tid; i < a.ids[x]; i += kBlock)
                if (s[i]) atomicAdd(&a.hist[x][i], s[i]);
        } else if (a.mode[x] == kSplit) {
            const uint32_t B = a.buckets[x];
            for (uint32_t b = tid; b < B; b += kBlock) {
                uint32_t sum = 0;
#pragma unroll
                for (uint32_t c = 0; c < kCopies; ++c) sum += s[b * kCopies + c];
                a.counts[x][(size_t)blockIdx.x * B + b] = sum;
            }
        }
    }
}

// The order of a bucket's IDs does not matter, so an ID's place is what an LDS
// counter held before it (ballots that keep the triples' order took 489 us for
// 50M triples).
__global__ __launch_bounds__(kBlock) void split_ids(IdArgs a) {
    __shared__ uint32_t s_id[kTile];
    __shared__ uint32_t s_cnt[kMaxBuckets];     // the tile's IDs of a bucket
    __shared__ uint32_t s_run[3][kMaxBuckets];  // where the range's next ID of a bucket goes
    __shared__ uint32_t s_loc[kMaxBuckets];     // a bucket's first ID in the ordered tile
    __shared__ uint32_t s_off[kMaxBuckets];     // place of ordered ID i: s_off[bucket] + i
    __shared__ uint32_t s_w[kNW], s_all;
    const uint32_t tid = threadIdx.x, w = blockIdx.x;
    const int wave = tid / dev::kWave, lane = tid % dev::kWave;
    static_assert(kMaxBuckets <= kBlock, "a thread per bucket");
    auto prefix = [&](uint32_t v) {  // exclusive sum over the threads
        const uint32_t incl = dev::wave_inclusive_sum(v);
        __syncthreads();
        if (lane == dev::kWave - 1) s_w[wave] = incl;
        __syncthreads();
        uint32_t before = 0;
#pragma unroll
        for (int y = 0; y < kNW; ++y) before += y < wave ? s_w[y] : 0u;
        return before + incl - v;
    };
    if (tid < kMaxBuckets) s_cnt[tid] = 0;
#pragma unroll
    for (int x = 0; x < 3; ++x) {
        if (a.mode[x] != kSplit) continue;
        const bool in = tid < a.buckets[x];
        const uint32_t base = prefix(in ? a.totals[x][tid] : 0u);
        if (in) s_run[x][tid] = base + a.scan[x][(size_t)w * a.buckets[x] + tid];
    }
    __syncthreads();
    const uint64_t r0 = (uint64_t)w * a.range, r1 = min(a.n, r0 + a.range);
    for (uint64_t t0 = r0; t0 < r1; t0 += kTile) {
        const uint32_t cnt = (uint32_t)min((uint64_t)kTile, r1 - t0);
        uint32_t v[kIPT][3];
#pragma unroll
        for (int u = 0; u < kIPT; ++u) {
            const uint32_t i = u * kBlock + tid;
#pragma unroll
            for (int x = 0; x < 3; ++x) v[u][x] = i < cnt ? a.g[3 * (t0 + i) + x] : 0u;
        }
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            if (a.mode[x] != kSplit) continue;
            uint32_t rank[kIPT], bucket[kIPT];
#pragma unroll
            for (int u = 0; u < kIPT; ++u) {
                bucket[u] = (v[u][x] >> kLowBits) - a.first[x];
                if (u * kBlock + tid >= cnt) bucket[u] = kMaxBuckets;
                if (bucket[u] < a.buckets[x]) rank[u] = atomicAdd(&s_cnt[bucket[u]], 1u);
            }
            __syncthreads();
            const uint32_t tot = tid < a.buckets[x] ? s_cnt[tid] : 0u;
            const uint32_t loc = prefix(tot);
            if (tid == a.buckets[x] - 1) s_all = loc + tot;
            if (tid < a.buckets[x]) {
                const uint32_t run = s_run[x][tid];
                s_loc[tid] = loc;
                s_off[tid] = run - loc;
                s_run[x][tid] = run + tot;
                s_cnt[tid] = 0;
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < kIPT; ++u)
                if (bucket[u] < a.buckets[x]) s_id[s_loc[bucket[u]] + rank[u]] = v[u][x];
            __syncthreads();
            const uint32_t all = s_all;  // the tile's IDs in the pass's buckets
#pragma unroll
            for (int u = 0; u < kIPT; ++u) {
                const uint32_t i = u * kBlock + tid;
                if (i >= all) continue;
                const uint32_t id = s_id[i];
                a.low[x][s_off[(id >> kLowBits) - a.first[x]] + i] =
                    (uint16_t)(id & (kBucketIds - 1));
            }
            __syncthreads();
        }
    }
}

__global__ __launch_bounds__(kCountBlock) void count_split(IdArgs a) {
    extern __shared__ uint32_t s_cnt[];           // kBucketIds bins
    __shared__ uint32_t s_first[kMaxBuckets + 1];  // a bucket's first place
    const int x = blockIdx.y;
    if (a.mode[x] != kSplit) return;
    const uint32_t tid = threadIdx.x, B = a.buckets[x];
    if (tid < dev::kWave) {  // one wave: bucket totals to first places
        uint32_t run = 0;
        for (uint32_t b0 = 0; b0 < B; b0 += dev::kWave) {
            const uint32_t b = b0 + tid, c = b < B ? a.totals[x][b] : 0u;
            const uint32_t incl = dev::wave_inclusive_sum(c);
            if (b < B) s_first[b] = run + incl - c;
            run += __shfl(incl, dev::kWave - 1, dev::kWave);
        }
        if (tid == 0) s_first[B] = run;
    }
    __syncthreads();
    const uint64_t n = s_first[B], share = (n + kShares - 1) / kShares;
    uint64_t at = blockIdx.x * share;
    const uint64_t end = min(n, at + share);
    uint32_t b = 0;  // the bucket that holds place `at`
    for (uint32_t hi = B; b + 1 < hi;) {
        const uint32_t mid = (b + hi) / 2;
        if (s_first[mid] <= at) b = mid;
        else hi = mid;
    }
    const uint4 *low = reinterpret_cast<const uint4 *>(a.low[x]);  // eight IDs
    for (; at < end && b < B; ++b) {
        const uint64_t stop = min(end, (uint64_t)s_first[b + 1]);
        if (stop <= at) continue;
        const uint32_t id0 = (a.first[x] + b) << kLowBits, ids = min(kBucketIds, a.ids[x] - id0);
        for (uint32_t i = tid; i < ids; i += kCountBlock) s_cnt[i] = 0;
        __syncthreads();
        for (uint64_t c = at / 8 + tid; 8 * c < stop; c += kCountBlock) {
            const uint4 q = low[c];
            const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint64_t i = 8 * c + u;
                if (i >= at && i < stop) atomicAdd(&s_cnt[w[u / 2] >> (16 * (u & 1)) & 0xffff], 1u);
            }
        }
        __syncthreads();
        for (uint32_t i = tid; i < ids; i += kCountBlock)
            if (s_cnt[i]) atomicAdd(&a.hist[x][id0 + i], s_cnt[i]);
        __syncthreads();
        at = stop;
    }
}

}  // namespace

// Counts into hist[x][0 .. nbins[x]) (zeroed; null: not counted); false, and
// nothing done, where the atomics of runtime.hip are the better way (a whole
// load with them / with the split: 100,000 triples 171 / 198 us, 200,000 226 /
// 228, 300,000 275 / 250, 4M 591 / 394; IDs up to 16M at 1M triples 2621 /
// 2578), IDs would take more than kMaxPasses passes of kMaxBuckets buckets or a
// pass would have few triples (200M triples with 20M IDs 25.4 / 13.9 ms, with
// 130M 81.9 / 75.0; 20M triples with 20M IDs 11.0 / 10.3, with 130M 63.1 / 63.7),
// or there is no memory for the split.
constexpr uint64_t kSplitRows = 1ull << 18;
bool count_ids(tid_ctx *ctx, const uint32_t *g, uint64_t n, uint32_t *const *hist,
               const uint32_t *nbins) {
    if (n < kSplitRows || n >= (1ull << 32)) return false;
    IdArgs a{};
    a.g = g;
    a.n = n;
    uint32_t total[3] = {0, 0, 0}, most = 0;  // buckets
    for (int x = 0; x < 3; ++x) {
        a.hist[x] = hist[x];
        a.ids[x] = nbins[x];
        if (!hist[x]) continue;
        a.mode[x] = nbins[x] <= kDirectIds ? kDirect : kSplit;
        if (a.mode[x] == kSplit) total[x] = (nbins[x] + kBucketIds - 1) >> kLowBits;
        most = std::max(most, total[x]);
    }
    const uint64_t passes = (most + kMaxBuckets - 1) / kMaxBuckets;
    if (passes > kMaxPasses || (passes > 1 && n < passes * kPassRows)) return false;
    const uint64_t tiles = (n + kTile - 1) / kTile;
    uint64_t P = std::max<uint64_t>(1, std::min<uint64_t>(tiles, 3ull * device_cus(ctx)));
    a.range = (tiles + P - 1) / P * kTile;
    P = (n + a.range - 1) / a.range;
    DevBuf mem;
    if (most) {
        size_t bytes = 0;
        for (int step = 0; step < 2; ++step) {
            char *at = mem.get<char>();
            bytes = 0;
            auto take = [&](size_t len) {
                char *p = at + bytes;
                bytes += align_up(len);
                return p;
            };
            for (int x = 0; x < 3; ++x) {
                if (a.mode[x] != kSplit) continue;
                const uint32_t B = std::min(total[x], kMaxBuckets);
                const size_t cells = (size_t)P * B * 4;
                a.counts[x] = reinterpret_cast<uint32_t *>(take(cells));
                a.scan[x] = reinterpret_cast<uint32_t *>(take(cells));
                a.totals[x] = reinterpret_cast<uint32_t *>(take((size_t)B * 4));
                a.low[x] = reinterpret_cast<uint16_t *>(take((n + 8) * 2));
            }
            if (step) break;
            try {
                mem = DevBuf(ctx, bytes);
            } catch (const Error &) {
                return false;
            }
        }
    }
    for (uint32_t first = 0; first == 0 || first < most; first += kMaxBuckets) {
        a.lds_words = 0;
        for (int x = 0; x < 3; ++x) {
            if (first && a.mode[x] == kDirect) a.mode[x] = kNone;  // counted in the first pass
            if (a.mode[x] == kSplit && first >= total[x]) a.mode[x] = kNone;
            a.lds[x] = a.lds_words;
            a.first[x] = first;
            if (a.mode[x] == kDirect) a.lds_words += a.ids[x];
            if (a.mode[x] != kSplit) continue;
            a.buckets[x] = std::min(total[x] - first, kMaxBuckets);
            a.lds_words += kCopies * a.buckets[x];
        }
        const size_t lds = (size_t)a.lds_words * 4, bins = (size_t)kBucketIds * 4;
        // above 64 KB a kernel must be allowed its dynamic LDS first
        if (lds > (64u << 10)) (void)resident_blocks((const void *)count_buckets, kBlock, lds);
        hipLaunchKernelGGL(count_buckets, dim3((uint32_t)P), dim3(kBlock), lds, ctx->stream, a);
        TID_HIP(hipGetLastError());
        if (!most) return true;
        for (int x = 0; x < 3; ++x)
            if (a.mode[x] == kSplit)
                scan_digits(ctx, a.counts[x], a.scan[x], a.totals[x], (uint32_t)P, a.buckets[x]);
        hipLaunchKernelGGL(split_ids, dim3((uint32_t)P), dim3(kBlock), 0, ctx->stream, a);
        TID_HIP(hipGetLastError());
        (void)resident_blocks((const void *)count_split, kCountBlock, bins);
        hipLaunchKernelGGL(count_split, dim3(kShares, 3), dim3(kCountBlock), bins, ctx->stream, a);
        TID_HIP(hipGetLastError());
    }
    return true;
}

}  // namespace tid
