// runtime.hip -- context, device memory, tables, graph load and load-time
// statistics of libtid.
#include "device_common.hpp"
#include "internal.hpp"

#include <algorithm>
#include <cstdio>

namespace tid {

// ---------------------------------------------------------------------------
// caching pool
// ---------------------------------------------------------------------------

size_t Pool::size_class(size_t bytes) {
    if (bytes <= 4096) return 4096;
    size_t p = 1;
    while (p < bytes) p <<= 1;
    // Up to 256 MiB a block is the next power of two, so that blocks of the
    // many intermediate tables of varying size are reused rather than
    // allocated again; above, 1/8 of the next power of two (at most 12.5%
    // slack) keeps large tables and graphs tight.
    if (p <= (size_t(256) << 20)) return p;
    const size_t step = p / 8;
    return (bytes + step - 1) / step * step;
}

void *Pool::alloc(size_t bytes) {
    const size_t sz = size_class(bytes);
    auto it = free_.lower_bound(sz);
    if (it != free_.end() && it->first <= sz + sz / 4) {
        void *p = it->second;
        live_[p] = it->first;
        free_.erase(it);
        return p;
    }
    void *p = nullptr;
    if (hipMalloc(&p, sz) != hipSuccess) {
        (void)hipGetLastError();
        release_all();  // give cached blocks back and try once more
        if (hipMalloc(&p, sz) != hipSuccess) {
            (void)hipGetLastError();
            return nullptr;
        }
    }
    live_[p] = sz;
    return p;
}

void Pool::free(void *p, size_t) {
    auto it = live_.find(p);
    if (it == live_.end()) return;
    free_.emplace(it->second, p);
    live_.erase(it);
}

void Pool::release_all() {
    for (auto &kv : free_) (void)hipFree(kv.second);
    free_.clear();
}

Pool::~Pool() {
    release_all();
    for (auto &kv : live_) (void)hipFree(kv.first);
    live_.clear();
}

// ---------------------------------------------------------------------------
// tables
// ---------------------------------------------------------------------------

HostWords::~HostWords() {
    for (uint64_t *s : slabs_) (void)hipHostFree(s);
}

void HostWords::grow() {
    uint64_t *s = nullptr;
    TID_HIP(hipHostMalloc((void **)&s, kSlab * 8, hipHostMallocCoherent));
    slabs_.push_back(s);
    for (size_t i = kSlab; i-- > 0;) free_.push_back(s + i);
}

uint64_t *HostWords::keep(size_t n) {
    grow();
    free_.resize(free_.size() - n);  // the slab's first words are its last to be listed
    return slabs_.back();
}

uint64_t *HostWords::take() {
    if (free_.empty()) grow();
    uint64_t *w = free_.back();
    free_.pop_back();
    return w;
}

std::unique_ptr<tid_table> make_table(tid_ctx *ctx, int32_t ncols, const int32_t *vars,
                                      uint64_t cap) {
    TID_REQUIRE(ncols >= 0 && ncols <= TID_MAX_COLS, TID_E_SCHEMA, "table: too many columns");
    auto t = std::make_unique<tid_table>();
    t->ctx = ctx;
    t->ncols = ncols;
    for (int c = 0; c < ncols; ++c) t->vars[c] = vars[c];
    t->cap = cap;
    const size_t stride = align_up(std::max<uint64_t>(cap, 1) * sizeof(uint32_t));
    t->block = std::make_shared<TableMem>(ctx, stride * (size_t)ncols);
    char *base = t->block->buf.get<char>();
    for (int c = 0; c < ncols; ++c) t->col[c] = reinterpret_cast<uint32_t *>(base + stride * c);
    t->d_count = t->block->count;
    return t;
}

void copy_bounds(tid_table *dst, const tid_table *src, const int *map, int n, int dst_off) {
    if (!src->maxv_known) {
        dst->maxv_known = false;
        return;
    }
    for (int c = 0; c < n; ++c) dst->maxv[dst_off + c] = src->maxv[map ? map[c] : c];
}

// n device words to pinned host memory, which the host reads after its wait
constexpr int kReadWords = 256;
struct WordList {
    const uint64_t *p[kReadWords];
};

__global__ __launch_bounds__(kReadWords) void gather_words(WordList src, uint64_t *dst, int n) {
    if ((int)threadIdx.x < n) dst[threadIdx.x] = *src.p[threadIdx.x];
}

// at least n words at ctx->rw_host
static void grow_host_words(tid_ctx *ctx, size_t n) {
    if (ctx->rw_cap >= n) return;
    if (ctx->rw_host) (void)hipHostFree(ctx->rw_host);
    ctx->rw_host = nullptr;
    const size_t cap = std::max<size_t>({n, 2 * ctx->rw_cap, 1024});
    ctx->rw_cap = 0;
    TID_HIP(hipHostMalloc((void **)&ctx->rw_host, cap * 8, hipHostMallocCoherent));
    ctx->rw_cap = cap;
}

void read_words(tid_ctx *ctx, const std::vector<const uint64_t *> &src, uint64_t *dst) {
    const size_t n = src.size();
    if (n == 0) return;
    grow_host_words(ctx, n);
    for (size_t i = 0; i < n; i += kReadWords) {
        WordList w{};
        const int m = (int)std::min<size_t>(kReadWords, n - i);
        for (int j = 0; j < m; ++j) w.p[j] = src[i + j];
        hipLaunchKernelGGL(gather_words, dim3(1), dim3(kReadWords), 0, ctx->stream, w,
                           ctx->rw_host + i, m);
        TID_HIP(hipGetLastError());
    }
    ctx->sync();
    ctx->check_flags();
    for (size_t i = 0; i < n; ++i) dst[i] = ctx->rw_host[i];
}

void resolve_counts(tid_ctx *ctx, tid_table *const *ts, int k) {
    bool waited = false;
    for (int j = 0; j < k; ++j) {
        if (ts[j]->count_known) continue;
        if (!waited) {  // the kernels that write the counts have then run
            ctx->sync();
            ctx->check_flags();
            waited = true;
        }
        set_count(ts[j], *static_cast<const volatile uint64_t *>(ts[j]->d_count));
    }
}

std::unique_ptr<tid_table> copy_columns(tid_ctx *ctx, const uint32_t *const *cols, int32_t ncols,
                                        const int32_t *vars, uint64_t nrows, int on_device) {
    auto t = make_table(ctx, ncols, vars, nrows);
    for (int c = 0; c < ncols; ++c) {
        TID_REQUIRE(nrows == 0 || cols[c], TID_E_INVALID_ARG, "null column");
        if (nrows)
            TID_HIP(hipMemcpyAsync(t->col[c], cols[c], nrows * sizeof(uint32_t),
                                   on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice,
                                   ctx->stream));
    }
    set_count(t.get(), nrows);
    return t;
}

// ---------------------------------------------------------------------------
// load-time checks and statistics
// ---------------------------------------------------------------------------

// Per position minimum and maximum ID (mm[0..2] = min, mm[3..5] = max).  A
// workgroup reduces in LDS before its six atomics: with six a wave, the
// atomics on the six words took most of 1186 us for 50M triples; now 142 us.
constexpr int kMinMaxBlock = 256;
__global__ __launch_bounds__(kMinMaxBlock) void minmax_kernel(const uint32_t *__restrict__ g,
                                                              uint64_t n, uint32_t *mm) {
    __shared__ uint32_t s_mm[6];
    constexpr int kU = 4;  // triples a thread has in flight
    uint32_t lo[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, hi[3] = {0, 0, 0};
    if (threadIdx.x < 6) s_mm[threadIdx.x] = threadIdx.x < 3 ? 0xFFFFFFFFu : 0u;
    __syncthreads();
    const uint64_t stride = (uint64_t)gridDim.x * kMinMaxBlock;
    uint64_t i = (uint64_t)blockIdx.x * kMinMaxBlock + threadIdx.x;
    for (; i + (kU - 1) * stride < n; i += kU * stride) {
        uint32_t v[kU][3];
#pragma unroll
        for (int u = 0; u < kU; ++u)
#pragma unroll
            for (int x = 0; x < 3; ++x) v[u][x] = g[3 * (i + u * stride) + x];
#pragma unroll
        for (int u = 0; u < kU; ++u)
#pragma unroll
            for (int x = 0; x < 3; ++x) {
                lo[x] = min(lo[x], v[u][x]);
                hi[x] = max(hi[x], v[u][x]);
            }
    }
    for (; i < n; i += stride)
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            lo[x] = min(lo[x], g[3 * i + x]);
            hi[x] = max(hi[x], g[3 * i + x]);
        }
#pragma unroll
    for (int x = 0; x < 3; ++x) {
        for (int d = 32; d >= 1; d >>= 1) {
            lo[x] = min(lo[x], (uint32_t)__shfl_xor((int)lo[x], d, 64));
            hi[x] = max(hi[x], (uint32_t)__shfl_xor((int)hi[x], d, 64));
        }
        if (dev::lane_id() == 0) {
            atomicMin(&s_mm[x], lo[x]);
            atomicMax(&s_mm[3 + x], hi[x]);
        }
    }
    __syncthreads();
    if (threadIdx.x < 3) atomicMin(&mm[threadIdx.x], s_mm[threadIdx.x]);
    else if (threadIdx.x < 6) atomicMax(&mm[threadIdx.x], s_mm[threadIdx.x]);
}

// The same while the triples are copied: one read of them instead of two.  A
// thread's 16-byte words are a multiple of three words apart, so that each of
// their four IDs always has the same position.  50M triples: copy 226 us and
// minmax 142, together 240.
__global__ __launch_bounds__(kMinMaxBlock) void copy_minmax(const uint4 *__restrict__ src,
                                                            uint4 *__restrict__ dst, uint64_t n,
                                                            uint32_t *mm) {
    __shared__ uint32_t s_mm[6];
    constexpr int kU = 4;  // words a thread has in flight
    if (threadIdx.x < 6) s_mm[threadIdx.x] = threadIdx.x < 3 ? 0xFFFFFFFFu : 0u;
    __syncthreads();
    uint32_t lo4[4] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, hi4[4] = {0, 0, 0, 0};
    auto add = [&](const uint4 &q) {
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int y = 0; y < 4; ++y) {
            lo4[y] = min(lo4[y], w[y]);
            hi4[y] = max(hi4[y], w[y]);
        }
    };
    const uint64_t words = 3 * n, nv = words / 4;
    const uint64_t stride = (uint64_t)gridDim.x * kMinMaxBlock;  // gridDim: a multiple of 3
    const uint64_t i0 = (uint64_t)blockIdx.x * kMinMaxBlock + threadIdx.x;
    uint64_t i = i0;
    for (; i + (kU - 1) * stride < nv; i += kU * stride) {
        uint4 q[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) q[u] = src[i + u * stride];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            dst[i + u * stride] = q[u];
            add(q[u]);
        }
    }
    for (; i < nv; i += stride) {
        const uint4 q = src[i];
        dst[i] = q;
        add(q);
    }
    uint32_t lo[3] = {0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu}, hi[3] = {0, 0, 0};
    auto put = [&](uint32_t pos, uint32_t l, uint32_t h) {
#pragma unroll
        for (uint32_t x = 0; x < 3; ++x)
            if (x == pos) {
                lo[x] = min(lo[x], l);
                hi[x] = max(hi[x], h);
            }
    };
#pragma unroll
    for (int y = 0; y < 4; ++y) put((uint32_t)((i0 + y) % 3), lo4[y], hi4[y]);  // 4 i + y mod 3
    if (i0 < words - 4 * nv) {  // up to three IDs past the last whole word
        const uint64_t w = 4 * nv + i0;
        const uint32_t v = reinterpret_cast<const uint32_t *>(src)[w];
        reinterpret_cast<uint32_t *>(dst)[w] = v;
        put((uint32_t)(w % 3), v, v);
    }
#pragma unroll
    for (int x = 0; x < 3; ++x) {
        for (int d = 32; d >= 1; d >>= 1) {
            lo[x] = min(lo[x], (uint32_t)__shfl_xor((int)lo[x], d, 64));
            hi[x] = max(hi[x], (uint32_t)__shfl_xor((int)hi[x], d, 64));
        }
        if (dev::lane_id() == 0) {
            atomicMin(&s_mm[x], lo[x]);
            atomicMax(&s_mm[3 + x], hi[x]);
        }
    }
    __syncthreads();
    if (threadIdx.x < 3) atomicMin(&mm[threadIdx.x], s_mm[threadIdx.x]);
    else if (threadIdx.x < 6) atomicMax(&mm[threadIdx.x], s_mm[threadIdx.x]);
}

__global__ void init_minmax(uint32_t *mm) {
    if (threadIdx.x < 3) mm[threadIdx.x] = 0xFFFFFFFFu;
    else if (threadIdx.x < 6) mm[threadIdx.x] = 0u;
}

// Per-position ID histograms in one pass over the graph, where count_ids does
// not take them (small graphs, few triples to many IDs).  Each workgroup
// counts in LDS first and adds its counts to the global bins at the end:
//  - a position whose IDs fit kDirectBins bins (the predicates) is counted
//    in LDS bins directly;
//  - any other position goes through a small open-addressing LDS table of
//    kHashEntries (ID, count) entries, so the hubs of a skewed position
//    (Zipf subjects and objects) cost one global atomic per workgroup
//    instead of one per triple; an ID that finds no free entry within
//    kHashProbes steps is added to its global bin directly.
// IDs are >= 1 here (checked before), so key 0 marks an empty entry.
int device_cus(tid_ctx *ctx);
bool count_ids(tid_ctx *ctx, const uint32_t *g, uint64_t n, uint32_t *const *hist,
               const uint32_t *nbins);

constexpr uint32_t kDirectBins = 8192;
constexpr uint32_t kHashEntries = 2048;
constexpr int kHashProbes = 16;
constexpr int kHistBlock = 1024;

struct HistArgs {
    uint32_t *hist[3];   // global bins per position (null: not counted)
    uint32_t nbins[3];
};

__global__ __launch_bounds__(kHistBlock) void hist3_kernel(const uint32_t *__restrict__ g,
                                                           uint64_t n, HistArgs a) {
    // per position a region of kDirectBins words: direct bins, or hash keys
    // (first kHashEntries words) and their counts (next kHashEntries words)
    __shared__ uint32_t s[3][kDirectBins];
    for (int x = 0; x < 3; ++x)
        for (uint32_t b = threadIdx.x; b < kDirectBins; b += kHistBlock) s[x][b] = 0;
    __syncthreads();
    bool direct[3];
#pragma unroll
    for (int x = 0; x < 3; ++x) direct[x] = a.nbins[x] <= kDirectBins;
    const uint64_t stride = (uint64_t)gridDim.x * kHistBlock;
    for (uint64_t i = (uint64_t)blockIdx.x * kHistBlock + threadIdx.x; i < n; i += stride) {
        uint32_t v[3];
        v[0] = __builtin_nontemporal_load(g + 3 * i);
        v[1] = __builtin_nontemporal_load(g + 3 * i + 1);
        v[2] = __builtin_nontemporal_load(g + 3 * i + 2);
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            if (!a.hist[x]) continue;
            if (direct[x]) {
                atomicAdd(&s[x][v[x]], 1u);
                continue;
            }
            uint32_t h = dev::hash32(v[x]) & (kHashEntries - 1);
            bool done = false;
            for (int probe = 0; probe < kHashProbes && !done; ++probe) {
                uint32_t k = s[x][h];
                if (k == 0) k = atomicCAS(&s[x][h], 0u, v[x]);
                if (k == 0 || k == v[x]) {
                    atomicAdd(&s[x][kHashEntries + h], 1u);
                    done = true;
                }
                h = (h + 1) & (kHashEntries - 1);
            }
            if (!done) atomicAdd(&a.hist[x][v[x]], 1u);
        }
    }
    __syncthreads();
    for (int x = 0; x < 3; ++x) {
        if (!a.hist[x]) continue;
        if (direct[x]) {
            for (uint32_t b = threadIdx.x; b < a.nbins[x]; b += kHistBlock)
                if (s[x][b]) atomicAdd(&a.hist[x][b], s[x][b]);
        } else {
            for (uint32_t e = threadIdx.x; e < kHashEntries; e += kHistBlock) {
                const uint32_t k = s[x][e], c = s[x][kHashEntries + e];
                if (k && c) atomicAdd(&a.hist[x][k], c);
            }
        }
    }
}

// One byte a count (kBig: the count goes to the list of large ones), and per
// block of IDs (a wave each) its triples and its large counts.
constexpr uint32_t kBlockWaves = IdCounts::kBlock / dev::kWave;  // steps of a wave

__global__ void pack_counts(const uint32_t *__restrict__ bins, uint64_t nblocks, uint8_t *bytes,
                            uint32_t *rows, uint32_t *nbig) {
    const int lane = dev::lane_id();
    const uint64_t waves = (uint64_t)gridDim.x * blockDim.x / dev::kWave;
    for (uint64_t b = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / dev::kWave; b < nblocks;
         b += waves) {
        uint32_t sum = 0, big = 0;
#pragma unroll
        for (uint32_t u = 0; u < kBlockWaves; ++u) {
            const uint64_t i = b * IdCounts::kBlock + u * dev::kWave + lane;
            const uint32_t c = bins[i];
            bytes[i] = (uint8_t)min(c, IdCounts::kBig);
            sum += c;
            big += (uint32_t)__popcll(dev::ballot(c >= IdCounts::kBig));
        }
        sum = dev::wave_sum(sum);
        if (lane == 0) {
            rows[b] = sum;
            nbig[b] = big;
        }
    }
}

// the large counts in ID order (at: exclusive sums of nbig)
__global__ void list_big(const uint32_t *__restrict__ bins, uint64_t nblocks,
                         const uint64_t *__restrict__ at, uint32_t *big) {
    const int lane = dev::lane_id();
    const uint64_t waves = (uint64_t)gridDim.x * blockDim.x / dev::kWave;
    for (uint64_t b = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / dev::kWave; b < nblocks;
         b += waves) {
        if (at[b + 1] == at[b]) continue;
        uint64_t to = at[b];
#pragma unroll
        for (uint32_t u = 0; u < kBlockWaves; ++u) {
            const uint32_t c = bins[b * IdCounts::kBlock + u * dev::kWave + lane];
            const uint64_t m = dev::ballot(c >= IdCounts::kBig);
            if (c >= IdCounts::kBig) big[to + dev::rank_in_mask(m)] = c;
            to += (uint64_t)__popcll(m);
        }
    }
}

void exclusive_scan_async(tid_ctx *ctx, const uint32_t *in, uint64_t n, uint64_t *out);

// Up to so many blocks of bins (1 MB) go to the host as they are: one copy, through
// the context's pinned words, where the packed ones take five launches, two waits
// and four copies.  A load of 1000 triples with 2,000 / 120,000 / 200,000 / 240,000
// IDs in all, packed: 103 / 120 / 124 / 128 us, summed on the host: 58 / 88 / 106 /
// 117 us.  (To pageable memory: 58 / 98 / 122 / 134, and 8 us more in the first
// scan after it.)
constexpr uint64_t kHostBlocks = 1024;

// Device bins (nblocks blocks) to the host, packed on the device (counts below 2^32
// in all per block).
static std::shared_ptr<IdCounts::Mem> packed_counts(tid_ctx *ctx, const uint32_t *bins,
                                                    uint64_t nblocks) {
    DevBuf bytes(ctx, nblocks * IdCounts::kBlock), rows(ctx, nblocks * 4), nbig(ctx, nblocks * 4),
        offs(ctx, 2 * (nblocks + 1) * 8);
    uint64_t *r = offs.get<uint64_t>(), *b = r + nblocks + 1;
    const unsigned grid = (unsigned)std::min<uint64_t>((nblocks + 3) / 4, 8192);
    hipLaunchKernelGGL(pack_counts, dim3(grid), dim3(256), 0, ctx->stream, bins, nblocks,
                       bytes.get<uint8_t>(), rows.get<uint32_t>(), nbig.get<uint32_t>());
    TID_HIP(hipGetLastError());
    exclusive_scan_async(ctx, rows.get<const uint32_t>(), nblocks, r);
    exclusive_scan_async(ctx, nbig.get<const uint32_t>(), nblocks, b);
    uint64_t nlarge = 0;
    read_words(ctx, {b + nblocks}, &nlarge);
    DevBuf big(ctx, std::max<uint64_t>(nlarge, 1) * 4);
    hipLaunchKernelGGL(list_big, dim3(grid), dim3(256), 0, ctx->stream, bins, nblocks, b,
                       big.get<uint32_t>());
    TID_HIP(hipGetLastError());
    auto m = std::make_shared<IdCounts::Mem>();
    m->bytes.reset(new uint8_t[nblocks * IdCounts::kBlock]);
    m->rows.reset(new uint64_t[nblocks + 1]);
    m->nbig.reset(new uint64_t[nblocks + 1]);
    m->big.reset(new uint32_t[std::max<uint64_t>(nlarge, 1)]);
    auto get = [&](void *dst, const void *src, size_t len) {
        if (len) TID_HIP(hipMemcpyAsync(dst, src, len, hipMemcpyDeviceToHost, ctx->stream));
    };
    get(m->bytes.get(), bytes.get(), nblocks * IdCounts::kBlock);
    get(m->rows.get(), r, (nblocks + 1) * 8);
    get(m->nbig.get(), b, (nblocks + 1) * 8);
    get(m->big.get(), big.get(), nlarge * 4);
    ctx->sync();
    return m;
}

// The same from the bins as they are, summed on the host.
static std::shared_ptr<IdCounts::Mem> summed_counts(tid_ctx *ctx, const uint32_t *bins,
                                                    uint64_t nblocks) {
    const uint64_t nbins = nblocks * IdCounts::kBlock;
    std::unique_ptr<uint32_t[]> pageable;
    uint32_t *host;
    if (nblocks <= kHostBlocks) {
        grow_host_words(ctx, kHostBlocks * IdCounts::kBlock / 2);
        host = reinterpret_cast<uint32_t *>(ctx->rw_host);
    } else {
        pageable.reset(host = new uint32_t[nbins]);
    }
    TID_HIP(hipMemcpyAsync(host, bins, nbins * sizeof(uint32_t), hipMemcpyDeviceToHost,
                           ctx->stream));
    ctx->sync();
    return counts_of_bins(host, nblocks);
}

// The bins of n triples: packed, unless they are few, a block's sum could pass 32
// bits or there is no memory for it.
static std::shared_ptr<IdCounts::Mem> counts_to_host(tid_ctx *ctx, const uint32_t *bins,
                                                     uint64_t nblocks, uint64_t n) {
    if (n < (1ull << 32) && nblocks > kHostBlocks) {
        try {
            return packed_counts(ctx, bins, nblocks);
        } catch (const Error &e) {
            if (e.code != TID_E_OOM) throw;
        }
    }
    return summed_counts(ctx, bins, nblocks);
}

// bytes of `ids` bins: whole blocks, so that every position starts on one
static size_t bin_bytes(uint64_t ids) {
    return (size_t)((ids + IdCounts::kBlock - 1) / IdCounts::kBlock) * IdCounts::kBlock *
           sizeof(uint32_t);
}

constexpr size_t kGraphPad = 64;        // zeros past a graph's triples
constexpr uint32_t kMaxHistIds = 1u << 28;  // 1 GiB of uint32 counts per position

// Whether p is memory of the context's own device, which its kernels may read
// without a copy.
bool on_this_device(tid_ctx *ctx, const void *p) {
    hipPointerAttribute_t at{};
    if (hipPointerGetAttributes(&at, p) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return at.type == hipMemoryTypeDevice && at.device == ctx->device;
}

// The triples of `from` (on the device if on_device) to the graph's memory, and
// its statistics.
void load_triples(tid_ctx *ctx, tid_graph *g, const uint32_t *from, int on_device) {
    g->data = DevBuf(ctx, (size_t)g->n * 12 + kGraphPad);
    if (g->n == 0) return;
    const size_t bytes = (size_t)g->n * 12;
    const bool fused =
        on_device && (uintptr_t)from % sizeof(uint4) == 0 && on_this_device(ctx, from);
    if (!fused)  // before any launch: a copy of host memory waits for those
        TID_HIP(hipMemcpyAsync(g->data.get(), from, bytes,
                               on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice,
                               ctx->stream));
    TID_HIP(hipMemsetAsync(g->data.get<char>() + bytes, 0, kGraphPad, ctx->stream));
    DevBuf mm(ctx, 6 * sizeof(uint32_t));
    hipLaunchKernelGGL(init_minmax, dim3(1), dim3(64), 0, ctx->stream, mm.get<uint32_t>());
    const int blocks = (int)std::min<uint64_t>((g->n + kMinMaxBlock - 1) / kMinMaxBlock, 2048);
    if (fused)
        hipLaunchKernelGGL(copy_minmax, dim3((blocks + 2) / 3 * 3), dim3(kMinMaxBlock), 0,
                           ctx->stream, reinterpret_cast<const uint4 *>(from),
                           g->data.get<uint4>(), g->n, mm.get<uint32_t>());
    else
        hipLaunchKernelGGL(minmax_kernel, dim3(blocks), dim3(kMinMaxBlock), 0, ctx->stream,
                           g->data.get<const uint32_t>(), g->n, mm.get<uint32_t>());
    TID_HIP(hipGetLastError());
    uint32_t h[6];
    TID_HIP(hipMemcpyAsync(h, mm.get(), sizeof(h), hipMemcpyDeviceToHost, ctx->stream));
    TID_HIP(hipStreamSynchronize(ctx->stream));
    for (int x = 0; x < 3; ++x) {
        TID_REQUIRE(h[x] != 0, TID_E_INVALID_ARG,
                    "load: ID 0 is reserved for the free variable and may not appear in a triple");
        g->max_id[x] = h[3 + x];
    }
    if (g->n >= (1ull << 32)) return;  // counts would not fit the uint32 bins
    // bins of the counted positions, one allocation, one clear
    HistArgs a{};
    size_t off[3] = {0, 0, 0}, total = 0;
    for (int x = 0; x < 3; ++x) {
        if (h[3 + x] >= kMaxHistIds) continue;
        a.nbins[x] = h[3 + x] + 1;
        off[x] = total;
        total += bin_bytes(a.nbins[x]);
    }
    if (total == 0) return;
    DevBuf hist(ctx, total);
    TID_HIP(hipMemsetAsync(hist.get(), 0, total, ctx->stream));
    for (int x = 0; x < 3; ++x)
        if (a.nbins[x]) a.hist[x] = reinterpret_cast<uint32_t *>(hist.get<char>() + off[x]);
    if (!count_ids(ctx, g->data.get<const uint32_t>(), g->n, a.hist, a.nbins)) {
        const int hb = (int)std::min<uint64_t>((g->n + kHistBlock - 1) / kHistBlock,
                                               2ull * (uint64_t)device_cus(ctx));
        hipLaunchKernelGGL(hist3_kernel, dim3(hb), dim3(kHistBlock), 0, ctx->stream,
                           g->data.get<const uint32_t>(), g->n, a);
        TID_HIP(hipGetLastError());
    }
    const auto mem = counts_to_host(ctx, hist.get<const uint32_t>(),
                                    total / sizeof(uint32_t) / IdCounts::kBlock, g->n);
    for (int x = 0; x < 3; ++x) {
        if (!a.nbins[x]) continue;
        g->counts[x].mem = mem;
        g->counts[x].first = off[x] / sizeof(uint32_t) / IdCounts::kBlock;
        g->counts[x].ids = a.nbins[x];
        g->counts[x].total = g->n;
    }
}

}  // namespace tid

// ---------------------------------------------------------------------------
// context
// ---------------------------------------------------------------------------

void *tid_ctx::alloc(size_t bytes) {
    void *p = alloc_fn ? alloc_fn(user, bytes, (void *)stream) : pool.alloc(bytes);
    if (!p) throw tid::Error(TID_E_OOM, "device allocation of " + std::to_string(bytes) +
                                            " bytes failed");
    return p;
}

void tid_ctx::free(void *p, size_t bytes) {
    if (!p) return;
    if (free_fn)
        free_fn(user, p, bytes, (void *)stream);
    else
        pool.free(p, bytes);
}

// Look-back state shared by the context's kernels (one stream, so launches
// never overlap).  Kernels leave it all zero when they finish; a new buffer is
// cleared here once.
uint32_t tid_ctx::next_epoch(size_t bytes, uint64_t **state) {
    bool zero = false;
    if (ep_bytes < bytes) {
        const size_t want = tid::align_up(std::max(bytes, ep_bytes + ep_bytes / 2), 1 << 16);
        if (ep_state) free(ep_state, ep_bytes);
        ep_state = nullptr;
        ep_bytes = 0;
        ep_state = alloc(want);
        ep_bytes = want;
        zero = true;
    }
    if (++epoch > tid::kEpochMax) {
        epoch = 1;
        zero = true;
    }
    if (zero) TID_HIP(hipMemsetAsync(ep_state, 0, ep_bytes, stream));
    *state = static_cast<uint64_t *>(ep_state);
    return epoch;
}

void tid_ctx::sync() {
    TID_HIP(hipStreamSynchronize(stream));
    uploads.clear();
}

void tid_ctx::check_flags() const {
    TID_REQUIRE(*static_cast<const volatile uint32_t *>(d_flags) == 0, TID_E_INTERNAL,
                "a cross-workgroup wait exceeded its spin bound (device state inconsistent)");
}

namespace tid {

// The predicate histogram of a chunk view (its other positions take their
// bounds from the whole graph's histograms).
void chunk_stats(tid_ctx *ctx, tid_graph *v) {
    if (v->n == 0 || v->max_id[1] >= kMaxHistIds) return;
    HistArgs a{};
    a.nbins[1] = v->max_id[1] + 1;
    const size_t bytes = bin_bytes(a.nbins[1]);
    DevBuf hist(ctx, bytes);
    TID_HIP(hipMemsetAsync(hist.get(), 0, bytes, ctx->stream));
    a.hist[1] = hist.get<uint32_t>();
    const int hb = (int)std::min<uint64_t>((v->n + kHistBlock - 1) / kHistBlock,
                                           2ull * (uint64_t)device_cus(ctx));
    hipLaunchKernelGGL(hist3_kernel, dim3(hb), dim3(kHistBlock), 0, ctx->stream, v->triples(),
                       v->n, a);
    TID_HIP(hipGetLastError());
    const uint64_t blocks = bytes / sizeof(uint32_t) / IdCounts::kBlock;
    auto mem = counts_to_host(ctx, hist.get<const uint32_t>(), blocks, v->n);
    // a predicate of 2^32 triples or more wraps in its bin: no counts then, and
    // every bound is the view's triples
    if (mem->rows[blocks] != v->n) return;
    IdCounts &c = v->counts[1];
    c.mem = std::move(mem);
    c.ids = a.nbins[1];
    c.total = v->n;
}

}  // namespace tid

uint64_t tid_graph::count_in(int pos, uint64_t lo, uint64_t hi) const {
    if (hi <= lo) return 0;
    const tid::IdCounts &c = counts[pos];
    if (c.empty()) return bounds_from ? std::min(n, bounds_from->count_in(pos, lo, hi)) : n;
    return c.below(hi) - c.below(lo);
}

#include <mutex>

namespace tid {
int resident_blocks(const void *kernel, int block, size_t lds) {
    static std::mutex mu;
    static std::map<std::pair<const void *, size_t>, int> cache;
    static std::map<const void *, size_t> allowed;
    std::lock_guard<std::mutex> lock(mu);
    // above 64 KB of dynamic LDS a kernel must be allowed that much first
    // (its static LDS counts against the same 160 KB)
    if (lds > 65536 && lds > allowed[kernel]) {
        TID_HIP(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        allowed[kernel] = lds;
    }
    auto key = std::make_pair(kernel, lds);
    auto it = cache.find(key);
    if (it != cache.end()) return it->second;
    int nb = 0;
    TID_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, kernel, block, lds));
    nb = std::max(nb, 1);
    cache[key] = nb;
    return nb;
}

int device_cus(tid_ctx *ctx) {
    if (ctx->num_cus <= 0) {
        int n = 0;
        TID_HIP(hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, ctx->device));
        ctx->num_cus = n > 0 ? n : 1;
    }
    return ctx->num_cus;
}
}  // namespace tid

uint64_t tid_table::rows() {
    if (!count_known) {
        tid_table *self = this;
        tid::resolve_counts(ctx, &self, 1);
    }
    return nrows;
}
