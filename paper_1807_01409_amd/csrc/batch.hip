// batch.hip -- the joins of many plans, in a few launches per round of a batch (the lockstep rounds of
// tid_query_batch): one workgroup per job, the job table in device memory.
// A plan's join whose sides both have at most kSmallRows rows does not launch
// its own hash build, scans, probe and expansion; it is a job of the round's
// one count launch, then of the next round's one expansion launch.  A job's
// hash table lives in the workgroup's LDS.  (The final sorts of a round are
// batched too: rowsort.hip.)
//
// Join job (Sec. 4.2: an equi-join on the shared variable, done here with a
// hash table in LDS): the R side's keys go into an open-addressing table
// (slot = key, count, first position of its rows in a per-slot row list);
// each L row finds its key's slot and pairs with the slot's R rows that also
// agree on every other shared variable (natural join).  The count launch
// writes each L row's exclusive output offset and the job's total.  Without
// other shared variables it also leaves its grouping of R's rows by key in
// device memory, and the expansion is one launch of output tiles over it;
// otherwise the expansion launch rebuilds the table and each L row's thread
// writes its pairs.  The order of rows within a join's output is not
// defined (a plan's result is always sorted at its end).
#include "batch.hpp"
#include "device_common.hpp"

#include <algorithm>

namespace tid {

namespace {

// Device-memory access through a pointer the compiler only knows as generic
// (one read from a job table): as a global access it is counted apart from
// LDS and scalar loads, so the waits those need do not also wait for it, as
// they would for a flat access.  p must point to device memory.
__device__ __forceinline__ uint32_t gload(const uint32_t *p) {
    return *(const __attribute__((address_space(1))) uint32_t *)p;
}
__device__ __forceinline__ void gstore(uint32_t *p, uint32_t v) {
    *(__attribute__((address_space(1))) uint32_t *)p = v;
}

__device__ __forceinline__ uint32_t pow2_at_least(uint32_t x) {
    uint32_t p = 64;
    while (p < x) p <<= 1;
    return p;
}

// exclusive scan of v over a block of BLOCK threads in thread order; returns
// this thread's prefix and leaves the total in *total
template <int BLOCK = kBatchBlock>
__device__ __forceinline__ uint32_t block_exclusive(uint32_t v, uint32_t *s_w, uint32_t *total) {
    constexpr int NW = BLOCK / dev::kWave;
    const int lane = threadIdx.x % dev::kWave, wave = threadIdx.x / dev::kWave;
    const uint32_t incl = dev::wave_inclusive_sum(v);
    if (lane == dev::kWave - 1) s_w[wave] = incl;
    __syncthreads();
    uint32_t before = 0, all = 0;
    for (int w = 0; w < NW; ++w) {
        if (w < wave) before += s_w[w];
        all += s_w[w];
    }
    __syncthreads();
    *total = all;
    return before + incl - v;
}

struct Table {
    uint32_t *key, *cnt, *start, *rows;
    uint32_t mask;
};

constexpr uint32_t kRowsPerThread = kSmallRows / kJoinBlock;  // 4

// R's keys into the LDS table: slot counts, slot starts, rows grouped by slot.
// The key equal to the empty marker (kEmptyKey, a valid ID) has a slot of its
// own past the probed ones, slot mask + 1, placed last.  Each thread loads its
// (up to kRowsPerThread) keys at once, then inserts them.  The lanes of a
// wave that share the key of its first row (a hub key fills whole waves)
// insert, count and reserve places through that row's lane: one LDS atomic
// for the group instead of one per lane on one word.
__device__ void build_table(const JoinJob &j, Table &t, uint32_t *s_w) {
    const uint32_t ts = pow2_at_least(2 * j.nr);
    t.mask = ts - 1;
    uint32_t rk[kRowsPerThread];
#pragma unroll
    for (uint32_t u = 0; u < kRowsPerThread; ++u) {
        const uint32_t r = u * kJoinBlock + threadIdx.x;
        rk[u] = r < j.nr ? gload(j.rkey + r) : kEmptyKey;
    }
    for (uint32_t s = threadIdx.x; s <= ts; s += kJoinBlock) {
        t.key[s] = kEmptyKey;
        t.cnt[s] = 0;
    }
    __syncthreads();
    const int lane = dev::lane_id();
#pragma unroll
    for (uint32_t u = 0; u < kRowsPerThread; ++u) {  // u is uniform: every lane takes the ballots
        const bool live = u * kJoinBlock + threadIdx.x < j.nr;
        const uint32_t k = rk[u];
        const uint64_t lv = dev::ballot(live);
        if (lv == 0) continue;  // the whole wave is past the end
        const int lead = __builtin_ctzll(lv);
        const uint32_t lk = __shfl(k, lead);
        const uint64_t same = dev::ballot(live && k == lk);
        if (live && (k != lk || lane == lead)) {
            uint32_t h = ts;
            if (k != kEmptyKey) {
                h = dev::hash32(k) & t.mask;
                for (;;) {  // ends: the table has more slots than keys
                    const uint32_t prev = atomicCAS(&t.key[h], kEmptyKey, k);
                    if (prev == kEmptyKey || prev == k) break;
                    h = (h + 1) & t.mask;
                }
            }
            atomicAdd(&t.cnt[h], k == lk ? (uint32_t)__popcll(same) : 1u);
        }
    }
    __syncthreads();
    // slot starts: each thread scans a contiguous run of ts / block slots
    const uint32_t per = ts / kJoinBlock > 0 ? ts / kJoinBlock : 1;
    const uint32_t s0 = threadIdx.x * per;
    uint32_t local = 0;
    for (uint32_t s = s0; s < s0 + per && s < ts; ++s) local += t.cnt[s];
    uint32_t all;
    uint32_t run = block_exclusive<kJoinBlock>(local, s_w, &all);
    for (uint32_t s = s0; s < s0 + per && s < ts; ++s) {
        t.start[s] = run;
        run += t.cnt[s];
        t.cnt[s] = 0;  // counts again while the rows are placed
    }
    if (threadIdx.x == 0) {  // the slot of kEmptyKey comes last
        t.start[ts] = all;
        t.cnt[ts] = 0;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t u = 0; u < kRowsPerThread; ++u) {
        const uint32_t r = u * kJoinBlock + threadIdx.x;
        const bool live = r < j.nr;
        const uint32_t k = rk[u];
        const uint64_t lv = dev::ballot(live);
        if (lv == 0) continue;
        const int lead = __builtin_ctzll(lv);
        const uint32_t lk = __shfl(k, lead);
        const uint64_t same = dev::ballot(live && k == lk);
        uint32_t at = 0;
        if (live && (k != lk || lane == lead)) {
            uint32_t h = ts;
            if (k != kEmptyKey) {
                h = dev::hash32(k) & t.mask;
                while (t.key[h] != k) h = (h + 1) & t.mask;
            }
            at = t.start[h] + atomicAdd(&t.cnt[h], k == lk ? (uint32_t)__popcll(same) : 1u);
        }
        const uint32_t group_at = __shfl(at, lead);
        if (live) t.rows[k == lk ? group_at + dev::rank_in_mask(same) : at] = r;
    }
    __syncthreads();
}

// the slot of key k, or kEmptyKey if R does not hold k
__device__ __forceinline__ uint32_t find_slot(const Table &t, uint32_t k) {
    if (k == kEmptyKey) return t.cnt[t.mask + 1] ? t.mask + 1 : kEmptyKey;
    uint32_t h = dev::hash32(k) & t.mask;
    for (;;) {
        const uint32_t x = t.key[h];
        if (x == k) return h;
        if (x == kEmptyKey) return kEmptyKey;
        h = (h + 1) & t.mask;
    }
}

__device__ __forceinline__ bool agree(const JoinJob &j, uint32_t l, uint32_t r) {
    bool ok = true;
    for (int e = 0; e < j.neq; ++e) ok &= gload(j.eq_l[e] + l) == gload(j.eq_r[e] + r);
    return ok;
}

__shared__ uint32_t s_key[kSmallSlots + 1], s_cnt[kSmallSlots + 1], s_start[kSmallSlots + 1];
__shared__ uint32_t s_rows[kSmallRows];
__shared__ uint32_t s_w[kJoinBlock / dev::kWave];

}  // namespace

__global__ __launch_bounds__(kJoinBlock) void batch_join_count(const JoinJob *jobs) {
    const JoinJob &j = jobs[blockIdx.x];
    Table t{s_key, s_cnt, s_start, s_rows, 0};
    build_table(j, t, s_w);
    // each thread a contiguous run of L rows, so offsets follow row order;
    // the keys are loaded at once, the offsets (and group starts) stored after
    uint32_t c[kRowsPerThread], lb[kRowsPerThread], lk[kRowsPerThread];
    const uint32_t i0 = threadIdx.x * kRowsPerThread;
#pragma unroll
    for (uint32_t u = 0; u < kRowsPerThread; ++u) lk[u] = i0 + u < j.nl ? gload(j.lkey + i0 + u) : 0u;
    uint32_t local = 0;
#pragma unroll
    for (uint32_t u = 0; u < kRowsPerThread; ++u) {
        c[u] = lb[u] = 0;  // a row without a match owns no output
        if (i0 + u >= j.nl) continue;
        const uint32_t h = find_slot(t, lk[u]);
        if (h == kEmptyKey) continue;
        const uint32_t a = t.start[h], b = a + t.cnt[h];
        lb[u] = a;
        if (j.neq == 0) {
            c[u] = b - a;
        } else {
            for (uint32_t m = a; m < b; ++m) c[u] += agree(j, i0 + u, t.rows[m]);
        }
        local += c[u];
    }
    uint32_t all;
    uint32_t run = block_exclusive<kJoinBlock>(local, s_w, &all);
#pragma unroll
    for (uint32_t u = 0; u < kRowsPerThread; ++u) {
        const uint32_t i = i0 + u;
        if (i < j.nl) {
            gstore(j.off + i, run);
            if (j.neq == 0) gstore(j.lbase + i, lb[u]);
        }
        run += c[u];
    }
    if (threadIdx.x == 0) {
        gstore(j.off + j.nl, all);
        *j.total = all;
    }
    if (j.neq == 0)  // the expansion pairs through this table's grouping
        for (uint32_t m = threadIdx.x; m < j.nr; m += kJoinBlock)
            gstore(j.grp + m, t.rows[m]);
}

// Expansion.  With no other shared variable, L row i owns the output rows
// [off[i], off[i+1]), paired in turn with the R rows of its key, so each
// output row is one thread's: its L row by a binary search of the offsets,
// its R row the matching entry of the key's group; consecutive threads write
// consecutive rows.  (Giving each L row to a thread instead makes the thread
// of a hub key walk hundreds of pairs, a global load after the other.)  With
// other shared variables, a row's pairs are those that also agree on them,
// and each L row's thread writes its pairs.
namespace {
__shared__ uint32_t s_off[kSmallRows], s_lb[kSmallRows];

// the last row i in [lo, hi] with off[i] <= o (off non-decreasing, off[lo] <= o)
__device__ __forceinline__ uint32_t owner_row(const uint32_t *off, uint32_t lo, uint32_t hi,
                                              uint32_t o) {
    uint32_t n = hi - lo + 1, a = lo;
    while (n > 1) {
        const uint32_t half = n / 2;
        if (off[a + half] <= o) a += half;
        n -= half;
    }
    return a;
}

constexpr int kUnroll = 4;

// Output rows [o0, o1) of a job without other shared variables, thread-
// parallel: the L rows i0 + k own [loff[k], loff[k+1]) (loff in LDS, i0..i1),
// each paired in turn with the entries of its key's group of R rows, which
// start at lb[k] in grp.  The loads of kUnroll rows are issued before their
// stores.
__device__ __forceinline__ void expand_rows(const JoinJob &j, const uint32_t *loff,
                                            const uint32_t *lb, const uint32_t *grp,
                                            uint32_t i0, uint32_t i1, uint32_t o0,
                                            uint32_t o1) {
    for (uint32_t base = o0; base < o1; base += kBatchBlock * kUnroll) {
        uint32_t li[kUnroll], ri[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const uint32_t o = base + u * kBatchBlock + threadIdx.x;
            li[u] = ri[u] = 0;
            if (o < o1) {
                const uint32_t k = owner_row(loff, 0, i1 - i0, o);
                li[u] = i0 + k;
                ri[u] = gload(grp + lb[k] + (o - loff[k]));
            }
        }
        for (int c = 0; c < j.nlc + j.nrc; ++c) {
            const bool left = c < j.nlc;
            const uint32_t *src = left ? j.lcol[c] : j.rcol[c - j.nlc];
            uint32_t v[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u)
                v[u] = base + u * kBatchBlock + threadIdx.x < o1
                           ? gload(src + (left ? li[u] : ri[u])) : 0u;
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const uint32_t o = base + u * kBatchBlock + threadIdx.x;
                if (o < o1) gstore(j.out[c] + o, v[u]);
            }
        }
    }
}
}  // namespace

// a job with other shared variables: each L row's thread writes its pairs
__global__ __launch_bounds__(kJoinBlock) void batch_join_expand(const JoinJob *jobs) {
    const JoinJob &j = jobs[blockIdx.x];
    Table t{s_key, s_cnt, s_start, s_rows, 0};
    build_table(j, t, s_w);
    for (uint32_t i = threadIdx.x; i < j.nl; i += kJoinBlock) {
        const uint32_t h = find_slot(t, gload(j.lkey + i));
        if (h == kEmptyKey) continue;
        uint32_t o = gload(j.off + i);
        const uint32_t a = t.start[h], b = a + t.cnt[h];
        for (uint32_t m = a; m < b; ++m) {
            const uint32_t r = t.rows[m];
            if (!agree(j, i, r)) continue;
            for (int c = 0; c < j.nlc; ++c) gstore(j.out[c] + o, gload(j.lcol[c] + i));
            for (int c = 0; c < j.nrc; ++c)
                gstore(j.out[j.nlc + c] + o, gload(j.rcol[c] + r));
            ++o;
        }
    }
}

// a job without other shared variables: tiles of kSplitTile output rows, a
// workgroup each, over the grouping the count launch left (lbase, grp); a
// tile stages the offsets and group starts of the L rows that own it
__global__ __launch_bounds__(kBatchBlock) void batch_join_split(const SplitJob *jobs, int nj,
                                                                uint32_t tile_base) {
    const uint32_t tile = tile_base + blockIdx.x;
    int lo = 0, hi = nj - 1;  // the job: the last one whose first tile is <= tile
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (jobs[mid].tile0 <= tile) lo = mid; else hi = mid - 1;
    }
    const SplitJob &x = jobs[lo];
    const JoinJob &j = x.j;
    const uint32_t o0 = (tile - x.tile0) * kSplitTile;
    const uint32_t o1 = min(o0 + kSplitTile, j.nout);
    // the L rows owning [o0, o1): i0..i1 (at most nl of them)
    const uint32_t i0 = owner_row(j.off, 0, j.nl - 1, o0);
    const uint32_t i1 = owner_row(j.off, i0, j.nl - 1, o1 - 1);
    for (uint32_t k = threadIdx.x; k <= i1 - i0; k += kBatchBlock) {
        s_off[k] = gload(j.off + i0 + k);
        s_lb[k] = gload(j.lbase + i0 + k);
    }
    __syncthreads();
    expand_rows(j, s_off, s_lb, j.grp, i0, i1, o0, o1);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

template <class Job>
static const Job *upload(tid_ctx *ctx, BatchState &bs, const std::vector<Job> &jobs) {
    const size_t bytes = jobs.size() * sizeof(Job);
    bs.host_keep.emplace_back(reinterpret_cast<const char *>(jobs.data()),
                              reinterpret_cast<const char *>(jobs.data()) + bytes);
    bs.keep.emplace_back(ctx, bytes);
    TID_HIP(hipMemcpyAsync(bs.keep.back().get(), bs.host_keep.back().data(), bytes,
                           hipMemcpyHostToDevice, ctx->stream));
    return bs.keep.back().get<const Job>();
}

// the expansions of jobs without other shared variables: one launch of
// output tiles; returns the other jobs
static std::vector<JoinJob> expand_split_jobs(tid_ctx *ctx, BatchState &bs,
                                              const std::vector<JoinJob> &jobs) {
    std::vector<JoinJob> rest;
    std::vector<SplitJob> split;
    uint64_t tiles = 0;
    for (const JoinJob &j : jobs) {
        if (j.neq != 0) {
            rest.push_back(j);
            continue;
        }
        SplitJob x{};
        x.j = j;
        x.tile0 = (uint32_t)tiles;
        tiles += (j.nout + kSplitTile - 1) / kSplitTile;
        split.push_back(x);
    }
    if (split.empty()) return rest;
    TID_REQUIRE(tiles < (1ull << 32), TID_E_UNSUPPORTED, "batched joins: output too large");
    const SplitJob *d = upload(ctx, bs, split);
    for (uint64_t t0 = 0; t0 < tiles; t0 += 1u << 20) {
        const unsigned g = (unsigned)std::min<uint64_t>(1u << 20, tiles - t0);
        hipLaunchKernelGGL(batch_join_split, dim3(g), dim3(kBatchBlock), 0, ctx->stream, d,
                           (int)split.size(), (uint32_t)t0);
        TID_HIP(hipGetLastError());
    }
    return rest;
}

void flush_join_jobs(tid_ctx *ctx, BatchState &bs, bool expand) {
    std::vector<JoinJob> &all = expand ? bs.expand_jobs : bs.count_jobs;
    if (all.empty()) return;
    std::vector<JoinJob> rest;
    if (expand) rest = expand_split_jobs(ctx, bs, all);
    std::vector<JoinJob> &jobs = expand ? rest : all;
    if (jobs.empty()) {
        all.clear();
        return;
    }
    const JoinJob *d = upload(ctx, bs, jobs);
    for (size_t j0 = 0; j0 < jobs.size(); j0 += 65535) {
        const unsigned g = (unsigned)std::min<size_t>(65535, jobs.size() - j0);
        if (expand)
            hipLaunchKernelGGL(batch_join_expand, dim3(g), dim3(kJoinBlock), 0, ctx->stream,
                               d + j0);
        else
            hipLaunchKernelGGL(batch_join_count, dim3(g), dim3(kJoinBlock), 0, ctx->stream,
                               d + j0);
        TID_HIP(hipGetLastError());
    }
    all.clear();
}

void flush_sort_jobs(tid_ctx *ctx, BatchState &bs) {
    if (bs.row_sorts.empty()) return;
    sort_rows_batched(ctx, bs.row_sorts, bs.keep, bs.host_keep);
    bs.row_sorts.clear();
}

}  // namespace tid

// ---------------------------------------------------------------------------
// larger joins of a batch
// ---------------------------------------------------------------------------

namespace tid {

void exclusive_scan_async(tid_ctx *ctx, const uint32_t *in, uint64_t n, uint64_t *out);
void scan_words_async(tid_ctx *ctx, const uint64_t *in, uint64_t n, uint64_t *out);
bool sort_keys32(tid_ctx *ctx, const uint32_t *col, uint64_t n, int bits, uint32_t *k0,
                 uint32_t *v0, uint32_t *k1, uint32_t *v1);
int device_cus(tid_ctx *ctx);

namespace {

constexpr int kBigBlock = 256;
constexpr int kBigIPT = 4, kProbeIPT = 8;  // build and probe rows of a thread,
constexpr int kFewIPT = 1, kFewProbeIPT = 2;  // and where that leaves the chip idle
constexpr uint64_t kFewBuildRows = 1ull << 14;
constexpr uint32_t kNoSlot32 = 0xFFFFFFFFu;

// index j with base[j] <= x < base[j + 1] (base non-decreasing, base[0] = 0)
__device__ __forceinline__ int job_of(const uint64_t *base, int J, uint64_t x) {
    int lo = 0, hi = J;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (base[mid] <= x) lo = mid;
        else hi = mid;
    }
    return lo;
}

// Build: R rows, tile by tile from a work counter (tiles of all joins
// concatenated; tbase = tile prefix per join).  Each row finds or claims its
// key's slot; ranks within a slot are reserved per tile through an LDS table
// (one global atomic per slot present in the tile, not per row).  IPT rows a
// thread: one where that leaves workgroups for the whole chip, since a thread
// claims its rows' slots one after the other (1,800 rows 18 us with four).
template <int IPT>
__global__ __launch_bounds__(kBigBlock) void big_insert(const BigCount *jobs, int J,
                                                        const uint64_t *tbase, uint64_t ntiles,
                                                        uint32_t *work, uint64_t *slots,
                                                        uint32_t *cnt, uint32_t *slot_of,
                                                        uint32_t *rank_of) {
    constexpr uint64_t kTile = (uint64_t)kBigBlock * IPT;
    constexpr int kBigLds = 2 * (int)kTile;  // rank table entries (> rows of a tile)
    __shared__ uint32_t s_slot[kBigLds], s_cnt[kBigLds], s_base[kBigLds];
    __shared__ uint64_t s_tile;
    for (int x = threadIdx.x; x < kBigLds; x += kBigBlock) {
        s_slot[x] = kNoSlot32;
        s_cnt[x] = 0;
    }
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) s_tile = atomicAdd(work, 1u);
        __syncthreads();
        const uint64_t t = s_tile;
        if (t >= ntiles) break;
        const int j = job_of(tbase, J, t);
        const BigCount &b = jobs[j];
        const uint64_t r0 = (t - tbase[j]) * kTile;
        uint32_t h[IPT], e[IPT], local[IPT];
#pragma unroll
        for (int u = 0; u < IPT; ++u) {
            const uint64_t r = r0 + (uint64_t)u * kBigBlock + threadIdx.x;
            if (r >= b.nr) continue;
            const uint32_t key = b.rkey[r];
            const uint64_t want = (uint64_t)key + 1ull;
            uint32_t hh = dev::hash32(key) & b.mask;
            for (uint32_t probe = 0; probe <= b.mask; ++probe) {  // ends: free slots remain
                unsigned long long *w = (unsigned long long *)&slots[b.sbase + hh];
                unsigned long long cur = *w;
                if (cur == 0ull) cur = atomicCAS(w, 0ull, (unsigned long long)want);
                if (cur == 0ull || cur == want) break;
                hh = (hh + 1) & b.mask;
            }
            const uint32_t gs = (uint32_t)(b.sbase + hh);
            uint32_t ee = gs & (kBigLds - 1);
            for (;;) {  // ends: fewer distinct slots per tile than entries
                const uint32_t prev = atomicCAS(&s_slot[ee], kNoSlot32, gs);
                if (prev == kNoSlot32 || prev == gs) break;
                ee = (ee + 1) & (kBigLds - 1);
            }
            h[u] = gs;
            e[u] = ee;
            local[u] = atomicAdd(&s_cnt[ee], 1u);
        }
        __syncthreads();
        for (int x = threadIdx.x; x < kBigLds; x += kBigBlock) {
            const uint32_t sl = s_slot[x];
            if (sl != kNoSlot32) {
                s_base[x] = atomicAdd(&cnt[sl], s_cnt[x]);
                s_slot[x] = kNoSlot32;
                s_cnt[x] = 0;
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < IPT; ++u) {
            const uint64_t r = r0 + (uint64_t)u * kBigBlock + threadIdx.x;
            if (r >= b.nr) continue;
            slot_of[b.rbase + r] = h[u];
            rank_of[b.rbase + r] = s_base[e[u]] + local[u];
        }
    }
}

__global__ void big_fill(const BigCount *jobs, int J, const uint64_t *rbase, uint64_t nrows,
                         const uint32_t *slot_of, const uint32_t *rank_of, const uint64_t *start,
                         uint32_t *rows) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; g < nrows; g += stride) {
        const int j = job_of(rbase, J, g);
        rows[start[slot_of[g]] + rank_of[g]] = (uint32_t)(g - jobs[j].rbase);
    }
}

__device__ __forceinline__ bool big_agree(const uint32_t *const *el, const uint32_t *const *er,
                                          int neq, uint64_t l, uint32_t r) {
    bool ok = true;
    for (int e = 0; e < neq; ++e) ok &= el[e][l] == er[e][r];
    return ok;
}

// Index of a sorted build side: for every present key, or group of keys that
// share key >> shift, where its run starts and ends in the sorted rows.
__global__ void index_runs(const uint32_t *__restrict__ key, uint64_t n, int shift, uint2 *index) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const uint32_t h = key[i] >> shift;
        if (i == 0 || key[i - 1] >> shift != h) index[h].x = (uint32_t)i;
        if (i + 1 == n || key[i + 1] >> shift != h) index[h].y = (uint32_t)(i + 1);
    }
}

// The build rows of key k: `len` of them from `at` on in the job's rows.
__device__ __forceinline__ void find_run(const BigCount &b, const uint64_t *slots,
                                         const uint32_t *cnt, const uint64_t *start, uint32_t k,
                                         uint32_t &at, uint32_t &len) {
    at = len = 0;
    if (b.index) {
        if (k > b.max_key) return;
        const uint2 run = b.index[k >> b.shift];
        if (run.x >= run.y) return;  // absent (both words are ~0)
        if (b.shift == 0) {
            at = run.x;
            len = run.y - run.x;
            return;
        }
        uint32_t lo = run.x, hi = run.y;  // first row with key >= k
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (b.skey[mid] < k) lo = mid + 1;
            else hi = mid;
        }
        at = lo;
        hi = run.y;
        while (lo < hi) {  // first row with key > k
            const uint32_t mid = (lo + hi) >> 1;
            if (b.skey[mid] <= k) lo = mid + 1;
            else hi = mid;
        }
        len = lo - at;
        return;
    }
    const uint64_t want = (uint64_t)k + 1ull;
    uint32_t h = dev::hash32(k) & b.mask;
    for (uint32_t probe = 0; probe <= b.mask; ++probe) {
        const uint64_t cur = slots[b.sbase + h];
        if (cur == want) {
            len = cnt[b.sbase + h];
            at = (uint32_t)start[b.sbase + h];
            return;
        }
        if (cur == 0ull) return;
        h = (h + 1) & b.mask;
    }
}

// A tile of a job's probe rows: the rows that put out anything become entries
// (row, first build row, output rows before it in the tile), packed at the
// tile's start in `entries`; their number and the tile's output rows are left
// for the expansion.  Only rows with output are written, and only the tiles'
// sums are scanned afterwards: with an offset kept and scanned for every probe
// row, joins of millions of rows and few matches spent as long on those.  IPT
// rows a thread, as for big_insert.
template <int IPT>
__global__ __launch_bounds__(kBigBlock) void big_probe(const BigCount *jobs, int J,
                                                       const uint64_t *ltile,
                                                       const uint64_t *slots, const uint32_t *cnt,
                                                       const uint64_t *start, BigEntry *entries,
                                                       uint32_t *tcount, uint64_t *ttotal) {
    constexpr int NW = kBigBlock / dev::kWave;
    constexpr uint64_t kTile = (uint64_t)kBigBlock * IPT;
    __shared__ uint32_t s_m[NW];
    __shared__ uint64_t s_s[NW];
    const uint64_t tile = blockIdx.x;
    const int j = job_of(ltile, J, tile);
    const BigCount &b = jobs[j];
    const uint64_t l0 = (tile - ltile[j]) * kTile;
    uint32_t key[IPT], at[IPT], len[IPT];
#pragma unroll
    for (int u = 0; u < IPT; ++u) {
        const uint64_t l = l0 + (uint64_t)u * kBigBlock + threadIdx.x;
        key[u] = l < b.nl ? b.lkey[l] : 0u;
    }
    uint32_t mine = 0;
    uint64_t sum = 0;
#pragma unroll
    for (int u = 0; u < IPT; ++u) {
        const uint64_t l = l0 + (uint64_t)u * kBigBlock + threadIdx.x;
        at[u] = len[u] = 0;
        if (l >= b.nl) continue;
        find_run(b, slots, cnt, start, key[u], at[u], len[u]);
        if (b.neq) {
            uint32_t c = 0;
            for (uint32_t m = 0; m < len[u]; ++m)
                c += big_agree(b.eq_l, b.eq_r, b.neq, l, b.rows[at[u] + m]);
            len[u] = c;
        }
        if (len[u]) {
            if (!b.matched) len[u] = 0;
        } else if (b.unmatched) {
            at[u] = kNoSlot32;  // one output row, without a build row
            len[u] = 1;
        }
        mine += len[u] != 0;
        sum += len[u];
    }
    const int lane = dev::lane_id(), wave = threadIdx.x / dev::kWave;
    const uint32_t mi = dev::wave_inclusive_sum(mine);
    const uint64_t si = dev::wave_inclusive_sum(sum);
    if (lane == dev::kWave - 1) {
        s_m[wave] = mi;
        s_s[wave] = si;
    }
    __syncthreads();
    uint32_t m = mi - mine, all_m = 0;
    uint64_t s = si - sum, all_s = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        if (w < wave) {
            m += s_m[w];
            s += s_s[w];
        }
        all_m += s_m[w];
        all_s += s_s[w];
    }
    BigEntry *e = entries + tile * kTile;
#pragma unroll
    for (int u = 0; u < IPT; ++u) {
        if (!len[u]) continue;
        e[m++] = BigEntry{(uint32_t)(l0 + (uint64_t)u * kBigBlock + threadIdx.x), at[u], s};
        s += len[u];
    }
    if (threadIdx.x == 0) {
        tcount[tile] = all_m;
        ttotal[tile] = all_s;
    }
}

__global__ void big_totals(const uint64_t *ltile, int J, const uint64_t *toff, uint64_t *tot) {
    for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < J; j += gridDim.x * blockDim.x)
        tot[j] = toff[ltile[j + 1]] - toff[ltile[j]];
}

// the last i of [lo, hi) with v(i) <= x (v does not fall; v(lo) <= x): the 64
// lanes of a wave probe evenly spaced places, a ballot keeps the part that
// holds it
template <class V>
__device__ __forceinline__ uint64_t wave_last(uint64_t lo, uint64_t hi, uint64_t x, const V &v) {
    while (hi - lo > 1) {  // the same for every lane
        const uint64_t step = (hi - lo + dev::kWave - 1) / dev::kWave;
        const uint64_t m = lo + (uint64_t)dev::lane_id() * step;
        const uint64_t c = (uint64_t)__popcll(dev::ballot(m < hi && v(m) <= x));
        lo += (c - 1) * step;
        hi = min(hi, lo + step);
    }
    return lo;
}

// One output row per thread.  A wave finds the join, the probe tile and the
// entry of its first row with 64-way searches; its other rows in that tile are
// of the next 63 entries at most, one of which a lane loads, and a row finds its
// entry among the lanes.  Rows of later tiles search by themselves, as all do
// where tiles put out few rows (DENSE false).  With every row searching, 24
// dependent reads, the seven expansions of a batch of 256 queries took 595 us,
// now 418.
template <bool DENSE>
__global__ __launch_bounds__(256) void big_expand(const BigExpand *jobs, int J,
                                                  const uint64_t *obase, uint64_t ntotal,
                                                  const uint64_t *toff, const uint32_t *tcount,
                                                  const BigEntry *entries, uint32_t tile) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    const uint32_t lane = (uint32_t)dev::lane_id();
    for (uint64_t g0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x - lane; g0 < ntotal;
         g0 += stride) {
        const uint64_t g = g0 + lane;
        uint32_t j = 0, a = 0;
        uint64_t rows = 0, l = 0, k = 0;  // rows: how many of the wave's are found here
        if (DENSE) {
            j = (uint32_t)wave_last(0, J, g0, [&](uint64_t i) { return obase[i]; });
            const uint64_t x0 = toff[jobs[j].tile0] + (g0 - jobs[j].obase);
            const uint64_t t = wave_last(jobs[j].tile0, jobs[j].tile1, x0,
                                         [&](uint64_t i) { return toff[i]; });
            const uint64_t in0 = x0 - toff[t];
            rows = toff[t + 1] - x0;
            const BigEntry *e = entries + t * tile;
            const uint32_t n = tcount[t];
            const uint32_t p0 =
                (uint32_t)wave_last(0, n, in0, [&](uint64_t i) { return e[i].pre; });
            BigEntry mine{0, 0, 0};
            uint32_t first = dev::kWave;  // the entry's first output row, from the wave's
            if (p0 + lane < n) {
                mine = e[p0 + lane];
                first = mine.pre <= in0 ? 0u : (uint32_t)min(mine.pre - in0, (uint64_t)dev::kWave);
            }
            uint32_t from = 0;  // the last lane whose entry starts at or before this row
#pragma unroll
            for (uint32_t step = dev::kWave / 2; step; step >>= 1) {
                const uint32_t s = __shfl(first, (int)(from + step), dev::kWave);
                if (s <= lane) from += step;
            }
            l = __shfl(mine.row, (int)from, dev::kWave);
            a = __shfl(mine.at, (int)from, dev::kWave);
            k = in0 + lane - __shfl(mine.pre, (int)from, dev::kWave);
        }
        if (g >= ntotal) continue;
        if (lane >= rows) {
            j = (uint32_t)job_of(obase, J, g);
            const uint64_t x = toff[jobs[j].tile0] + (g - jobs[j].obase);
            uint64_t lo = jobs[j].tile0, hi = jobs[j].tile1;  // last tile with toff <= x
            while (hi - lo > 1) {
                const uint64_t mid = (lo + hi) >> 1;
                if (toff[mid] <= x) lo = mid;
                else hi = mid;
            }
            const uint64_t in = x - toff[lo];
            const BigEntry *f = entries + lo * tile;
            uint32_t p = 0, q = tcount[lo];  // last entry with pre <= in
            while (q - p > 1) {
                const uint32_t mid = (p + q) >> 1;
                if (f[mid].pre <= in) p = mid;
                else q = mid;
            }
            l = f[p].row;
            a = f[p].at;
            k = in - f[p].pre;
        }
        const BigExpand &b = jobs[j];
        const uint64_t o = g - b.obase;
        const bool paired = a != kNoSlot32;
        uint32_t r = 0;
        if (paired && b.neq == 0) {
            r = b.rows[a + k];
        } else if (paired) {  // the k-th partner that also agrees on the other shared variables
            for (uint32_t m = 0;; ++m) {
                r = b.rows[a + m];
                if (big_agree(b.eq_l, b.eq_r, b.neq, l, r)) {
                    if (k == 0) break;
                    --k;
                }
            }
        }
        for (int c = 0; c < b.ncols; ++c) {
            uint32_t v = 0;
            if (b.side[c] == kFromProbe) v = b.col[c][l];
            else if (b.side[c] == kFromBuild && paired) v = b.col[c][r];
            b.out[c][o] = v;
        }
    }
}

unsigned grid_cap(uint64_t n, uint64_t cap = 16384) {
    return (unsigned)std::max<uint64_t>(1, std::min<uint64_t>((n + 255) / 256, cap));
}

}  // namespace

// A large build side is sorted by key instead of hashed: its insertions are two
// device atomics a row, which this chip does at about 15e9 a second (3M rows:
// 392 us), against three or four radix passes and an index of plain stores
// (3M rows: 130 us).  Below kSortBuildRows the passes' launches cost more.
constexpr uint64_t kSortBuildRows = 1ull << 19;
// Largest build side of one join: a table of two slots a row has then 2^31,
// and every row number and slot fits 32 bits.
constexpr uint64_t kMostBuildRows = 1ull << 30;

static void sort_build_side(tid_ctx *ctx, BigCount &b, BigArena &arena) {
    // direct by key while that takes at most four index entries a row; else
    // by the key's upper bits, about two entries a row
    b.shift = 0;
    if ((uint64_t)b.max_key + 1 > 4 * b.nr)
        while (((uint64_t)b.max_key >> b.shift) + 1 > 2 * b.nr) ++b.shift;
    const uint64_t n_index = ((uint64_t)b.max_key >> b.shift) + 1;
    int bits = 1;
    while (bits < 32 && b.max_key >> bits) ++bits;
    DevBuf k0(ctx, b.nr * 4), k1(ctx, b.nr * 4), v0(ctx, b.nr * 4), v1(ctx, b.nr * 4);
    const bool moved = sort_keys32(ctx, b.rkey, b.nr, bits, k0.get<uint32_t>(), v0.get<uint32_t>(),
                                   k1.get<uint32_t>(), v1.get<uint32_t>());
    DevBuf index(ctx, n_index * sizeof(uint2));
    TID_HIP(hipMemsetAsync(index.get(), 0xFF, n_index * sizeof(uint2), ctx->stream));
    DevBuf &key = moved ? k1 : k0, &row = moved ? v1 : v0;
    hipLaunchKernelGGL(index_runs, dim3(grid_cap(b.nr)), dim3(256), 0, ctx->stream,
                       key.get<const uint32_t>(), b.nr, b.shift, index.get<uint2>());
    TID_HIP(hipGetLastError());
    b.index = index.get<const uint2>();
    b.skey = key.get<const uint32_t>();
    b.rows = row.get<const uint32_t>();
    arena.builds.push_back(std::move(index));
    arena.builds.push_back(std::move(key));
    arena.builds.push_back(std::move(row));
}

void flush_big_count(tid_ctx *ctx, std::vector<BigJoinReq> &reqs,
                     std::shared_ptr<BigArena> *arena_out) {
    if (reqs.empty()) return;
    const int J = (int)reqs.size();
    std::vector<BigCount> jobs(J);
    std::vector<uint64_t> tbase(J + 1, 0), rbase(J + 1, 0), ltile(J + 1, 0);
    auto arena = std::make_shared<BigArena>();
    uint64_t S = 0, build = 0, probe = 0;
    for (const BigJoinReq &r : reqs) {
        TID_REQUIRE(r.c.nr <= kMostBuildRows, TID_E_UNSUPPORTED,
                    "join: the build side has more than 2^30 rows");
        if (r.c.nr < kSortBuildRows) build += r.c.nr;
        probe += r.c.nl;
    }
    // fewer rows a thread: for builds of up to kFewBuildRows (18 us with four
    // rows a thread, 9 with one, for some thousand rows; for 60,000 24 and 35),
    // for probes as long as four workgroups a CU take them all
    const bool few_build = build <= kFewBuildRows;
    const bool few_probe =
        probe <= 4ull * (uint64_t)device_cus(ctx) * kBigBlock * kFewProbeIPT;
    const uint64_t btile = (uint64_t)kBigBlock * (few_build ? kFewIPT : kBigIPT);
    const uint64_t ptile = (uint64_t)kBigBlock * (few_probe ? kFewProbeIPT : kProbeIPT);
    arena->tile = (uint32_t)ptile;
    for (int j = 0; j < J; ++j) {
        BigCount &b = jobs[j];
        b = reqs[j].c;
        ltile[j + 1] = ltile[j] + (b.nl + ptile - 1) / ptile;
        rbase[j + 1] = rbase[j];
        tbase[j + 1] = tbase[j];
        if (b.nr >= kSortBuildRows) {
            sort_build_side(ctx, b, *arena);
            continue;
        }
        uint64_t cap = 64;
        while (cap < 2 * b.nr) cap <<= 1;
        b.mask = (uint32_t)(cap - 1);
        b.sbase = S;
        S += cap;
        b.rbase = rbase[j];
        rbase[j + 1] += b.nr;
        tbase[j + 1] += (b.nr + btile - 1) / btile;
    }
    const uint64_t NR = rbase[J], LT = ltile[J], T = tbase[J];
    TID_REQUIRE(S < (1ull << 32) && NR < (1ull << 32), TID_E_UNSUPPORTED,
                "batched joins: too many build rows in one round");
    TID_REQUIRE(LT < (1ull << 31), TID_E_UNSUPPORTED, "batched joins: too many probe rows");
    // one arena: job table and prefixes, then the per-slot and per-row arrays
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += align_up(std::max<size_t>(bytes, 8));
        return at;
    };
    const size_t o_jobs = take(J * sizeof(BigCount)), o_tb = take((J + 1) * 8),
                 o_rb = take((J + 1) * 8), o_lt = take((J + 1) * 8), o_work = take(8),
                 o_slots = take(S * 8), o_cnt = take(S * 4), o_start = take((S + 1) * 8),
                 o_slotof = take(NR * 4), o_rank = take(NR * 4), o_rows = take(NR * 4),
                 o_entries = take(LT * ptile * sizeof(BigEntry)), o_tcount = take(LT * 4),
                 o_ttotal = take(LT * 8), o_toff = take((LT + 1) * 8), o_tot = take(J * 8);
    arena->buf = DevBuf(ctx, off);
    char *base = arena->buf.get<char>();
    uint64_t *slots = reinterpret_cast<uint64_t *>(base + o_slots);
    uint32_t *cnt = reinterpret_cast<uint32_t *>(base + o_cnt);
    uint64_t *start = reinterpret_cast<uint64_t *>(base + o_start);
    uint32_t *rows = reinterpret_cast<uint32_t *>(base + o_rows);
    uint64_t *ttotal = reinterpret_cast<uint64_t *>(base + o_ttotal);
    arena->entries = reinterpret_cast<BigEntry *>(base + o_entries);
    arena->tcount = reinterpret_cast<uint32_t *>(base + o_tcount);
    arena->toff = reinterpret_cast<uint64_t *>(base + o_toff);
    uint64_t *tot = reinterpret_cast<uint64_t *>(base + o_tot);
    for (BigCount &b : jobs)
        if (!b.index) b.rows = rows;
    // host tables: one staging copy, then one upload
    std::vector<char> host(o_slots);
    std::memcpy(host.data() + o_jobs, jobs.data(), J * sizeof(BigCount));
    std::memcpy(host.data() + o_tb, tbase.data(), (J + 1) * 8);
    std::memcpy(host.data() + o_rb, rbase.data(), (J + 1) * 8);
    std::memcpy(host.data() + o_lt, ltile.data(), (J + 1) * 8);
    std::memset(host.data() + o_work, 0, 8);
    ctx->uploads.push_back(std::move(host));
    TID_HIP(hipMemcpyAsync(base, ctx->uploads.back().data(), o_slots, hipMemcpyHostToDevice,
                           ctx->stream));
    const BigCount *dj = reinterpret_cast<const BigCount *>(base + o_jobs);
    const uint64_t *dtb = reinterpret_cast<const uint64_t *>(base + o_tb);
    const uint64_t *drb = reinterpret_cast<const uint64_t *>(base + o_rb);
    const uint64_t *dlt = reinterpret_cast<const uint64_t *>(base + o_lt);
    uint32_t *slot_of = reinterpret_cast<uint32_t *>(base + o_slotof);
    uint32_t *rank_of = reinterpret_cast<uint32_t *>(base + o_rank);
    if (S)  // slot words and counts start at zero (one clear of the contiguous run)
        TID_HIP(hipMemsetAsync(base + o_slots, 0, o_start - o_slots, ctx->stream));
    if (NR) {
        const unsigned workers = (unsigned)std::max<uint64_t>(
            1, std::min<uint64_t>(T, 4ull * (uint64_t)device_cus(ctx)));
        hipLaunchKernelGGL(few_build ? big_insert<kFewIPT> : big_insert<kBigIPT>, dim3(workers),
                           dim3(kBigBlock), 0, ctx->stream, dj, J, dtb, T,
                           reinterpret_cast<uint32_t *>(base + o_work), slots, cnt, slot_of,
                           rank_of);
        TID_HIP(hipGetLastError());
        exclusive_scan_async(ctx, cnt, S, start);
        hipLaunchKernelGGL(big_fill, dim3(grid_cap(NR)), dim3(256), 0, ctx->stream, dj, J, drb,
                           NR, slot_of, rank_of, start, rows);
        TID_HIP(hipGetLastError());
    }
    if (LT) {
        hipLaunchKernelGGL(few_probe ? big_probe<kFewProbeIPT> : big_probe<kProbeIPT>,
                           dim3((unsigned)LT), dim3(kBigBlock), 0, ctx->stream, dj, J, dlt, slots,
                           cnt, start, arena->entries, arena->tcount, ttotal);
        TID_HIP(hipGetLastError());
    }
    scan_words_async(ctx, ttotal, LT, arena->toff);
    hipLaunchKernelGGL(big_totals, dim3(grid_cap(J)), dim3(256), 0, ctx->stream, dlt, J,
                       arena->toff, tot);
    TID_HIP(hipGetLastError());
    for (int j = 0; j < J; ++j) {
        PendingJoin *pj = reqs[j].pj;
        pj->total_ptr = tot + j;
        pj->big_tile0 = ltile[j];
        pj->big_tile1 = ltile[j + 1];
        pj->big_rows = jobs[j].rows;
        pj->big_arena = arena;
    }
    reqs.clear();
    *arena_out = arena;
}

void flush_big_expand(tid_ctx *ctx, const BigArena &arena, std::vector<BigExpand> &jobs,
                      BatchState &bs) {
    if (jobs.empty()) return;
    const int J = (int)jobs.size();
    // jobs arrive with obase = their output's first row in the concatenated
    // output space; bs.big_out_total is that space's size
    std::vector<uint64_t> obase(J + 1, 0);
    for (int j = 0; j < J; ++j) obase[j] = jobs[j].obase;
    const uint64_t total = bs.big_out_total;
    obase[J] = total;
    const size_t bytes_jobs = align_up(J * sizeof(BigExpand));
    std::vector<char> host(bytes_jobs + (J + 1) * 8);
    std::memcpy(host.data(), jobs.data(), J * sizeof(BigExpand));
    std::memcpy(host.data() + bytes_jobs, obase.data(), (J + 1) * 8);
    ctx->uploads.push_back(std::move(host));
    const std::vector<char> &table = ctx->uploads.back();
    bs.keep.emplace_back(ctx, table.size());
    char *d = bs.keep.back().get<char>();
    TID_HIP(hipMemcpyAsync(d, table.data(), table.size(), hipMemcpyHostToDevice, ctx->stream));
    uint64_t tiles = 0;
    for (const BigExpand &b : jobs) tiles += b.tile1 - b.tile0;
    if (total)
        hipLaunchKernelGGL(total >= 256 * tiles ? big_expand<true> : big_expand<false>,
                           dim3(grid_cap(total)), dim3(256), 0, ctx->stream,
                           reinterpret_cast<const BigExpand *>(d), J,
                           reinterpret_cast<const uint64_t *>(d + bytes_jobs), total, arena.toff,
                           arena.tcount, arena.entries, arena.tile);
    TID_HIP(hipGetLastError());
    jobs.clear();
    bs.big_out_total = 0;
}

}  // namespace tid

namespace tid {

namespace {
__global__ void batch_copy_kernel(const CopyJob *jobs, const uint64_t *base, int J,
                                  uint64_t total) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; g < total; g += stride) {
        const int j = job_of(base, J, g);
        const uint64_t i = g - base[j];
        jobs[j].dst[i] = jobs[j].src[i];
    }
}
}  // namespace

void batch_copy(tid_ctx *ctx, const std::vector<CopyJob> &jobs, BatchState &bs) {
    std::vector<CopyJob> nz;
    for (const CopyJob &c : jobs)
        if (c.n) nz.push_back(c);
    if (nz.empty()) return;
    const int J = (int)nz.size();
    std::vector<uint64_t> base(J + 1, 0);
    for (int j = 0; j < J; ++j) base[j + 1] = base[j] + nz[j].n;
    const size_t bj = align_up(J * sizeof(CopyJob));
    std::vector<char> host(bj + (J + 1) * 8);
    std::memcpy(host.data(), nz.data(), J * sizeof(CopyJob));
    std::memcpy(host.data() + bj, base.data(), (J + 1) * 8);
    bs.host_keep.push_back(std::move(host));
    bs.keep.emplace_back(ctx, bs.host_keep.back().size());
    char *d = bs.keep.back().get<char>();
    TID_HIP(hipMemcpyAsync(d, bs.host_keep.back().data(), bs.host_keep.back().size(),
                           hipMemcpyHostToDevice, ctx->stream));
    hipLaunchKernelGGL(batch_copy_kernel, dim3(grid_cap(base[J])), dim3(256), 0, ctx->stream,
                       reinterpret_cast<const CopyJob *>(d),
                       reinterpret_cast<const uint64_t *>(d + bj), J, base[J]);
    TID_HIP(hipGetLastError());
}

}  // namespace tid
