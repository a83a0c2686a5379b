// dict.hip -- dictionary encoding of string triples into TripleID rows, and
// decoding of IDs back to strings (Sec. 3: the conversion of an RDF file into
// ID dictionaries and rows of three 32-bit IDs, done there in one linear pass
// with hash tables on the host).
//
// Encoding on the GPU, one shared dictionary, IDs from 1 in order of first
// appearance when the terms are read s, p, o, triple by triple:
//   1. hash every term (64-bit FNV-1a over its bytes) and find its hash's slot
//      in a table, which keeps the smallest term index of each hash: the
//      term's first appearance;
//   2. check that every term is byte-equal to the first one of its hash (a
//      64-bit collision between different strings is reported as an error,
//      never silently merged);
//   3. prefix sums over the terms, of the first appearances and of their
//      lengths: a first appearance's rank is its ID - 1, its bytes' place is
//      known, and both are written with every term's ID in one pass.
// Bound: the random accesses of step 1 (78 us of 150 us on the device for
// 200,000 triples); a host between the steps and two radix sorts (eleven
// passes) in place of the table took 1088 us for 200,000 triples and a page of
// 5,000 decoded, now 272 us.
// Decoding gathers the strings of a column of IDs (lengths, offsets by an
// exclusive scan, bytes).
#include "compact.hpp"

#include <algorithm>

namespace tid {

bool on_this_device(tid_ctx *ctx, const void *p);
void exclusive_scan_async(tid_ctx *ctx, const uint32_t *in, uint64_t n, uint64_t *out);
void read_words(tid_ctx *ctx, const std::vector<const uint64_t *> &src, uint64_t *dst);

namespace {

unsigned grid_of(uint64_t n) {
    return (unsigned)std::max<uint64_t>(1, std::min<uint64_t>((n + 255) / 256, 16384));
}

#define TID_GRID_LOOP(i, n)                                                              \
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < (n);          \
         i += (uint64_t)gridDim.x * blockDim.x)

__device__ __forceinline__ uint64_t eight_bytes(const uint8_t *p) {
    uint64_t w;
    __builtin_memcpy(&w, p, 8);  // one load, at any alignment
    return w;
}

// The bytes of a string in words of eight (the last one shorter, its bytes
// alone): f(word, bytes) until it returns false.  No byte outside the string
// is read.
template <class F>
__device__ __forceinline__ void each_word(const uint8_t *p, uint64_t len, const F &f) {
    uint64_t k = 0;
    for (; k + 8 <= len; k += 8)
        if (!f(k, eight_bytes(p + k), 8)) return;
    const int rest = (int)(len - k);
    if (rest == 0) return;
    uint64_t w = 0;
    if (len >= 8) {
        w = eight_bytes(p + len - 8) >> (64 - 8 * rest);
    } else {
        for (int x = 0; x < rest; ++x) w |= (uint64_t)p[k + x] << (8 * x);
    }
    f(k, w, rest);
}

__device__ __forceinline__ void copy_string(uint8_t *dst, const uint8_t *src, uint64_t len) {
    each_word(src, len, [&](uint64_t k, uint64_t w, int n) {
        if (n == 8) {
            __builtin_memcpy(dst + k, &w, 8);
        } else {
            for (int x = 0; x < n; ++x) dst[k + x] = (uint8_t)(w >> (8 * x));
        }
        return true;
    });
}

struct Terms {
    const uint8_t *bytes;
    const uint64_t *off;
    uint64_t nbytes, m;
    uint32_t *falls, *past;  // offsets that fall, or reach past the bytes
    uint32_t *wide;          // a term of 2^32 bytes or more: lengths are summed as 32-bit words
    // length of term t; 0 if it is refused
    __device__ __forceinline__ uint32_t length(uint64_t t, uint64_t &at) const {
        at = off[t];
        const uint64_t end = off[t + 1], len = end - at;
        if ((end >= at) & (end <= nbytes) & (len >> 32 == 0)) return (uint32_t)len;
        dev::raise(end < at ? falls : end > nbytes ? past : wide);
        return 0;
    }
};

// Table of hashes: key[cap] (0: free) and, for each, ~(its smallest term
// index).  The hash 0 has the slot cap, past the others.
struct TermTable {
    uint64_t *key;
    uint32_t *lead;
    uint64_t cap;
    __device__ __forceinline__ uint64_t find(uint64_t h) const {
        if (h == 0) return cap;
        uint64_t x = h ^ h >> 32;  // FNV's high bits vary little over short strings
        x *= 0x9e3779b97f4a7c15ull;
        uint64_t s = __umul64hi(x, cap);
        for (uint64_t probes = 0; probes < cap; ++probes) {  // cap > distinct hashes
            uint64_t cur = dev::peek(key + s);
            if (cur == 0)
                cur = atomicCAS((unsigned long long *)(key + s), 0ull, (unsigned long long)h);
            if (cur == 0 || cur == h) return s;
            if (++s == cap) s = 0;
        }
        return cap;  // not reached
    }
};

// Slot of every term.  The lanes of a wave that hold the same term are found
// first and the lowest one goes to the table for all of them: a predicate
// stands in many triples.
__global__ __launch_bounds__(256) void insert_terms(Terms in, TermTable tab, uint32_t *slot,
                                                    uint32_t *slot_hi) {
    const int lane = dev::lane_id();
    for (uint64_t t0 = (uint64_t)blockIdx.x * blockDim.x; t0 < in.m;
         t0 += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t t = t0 + threadIdx.x;
        const bool valid = t < in.m;
        uint64_t h = 0xcbf29ce484222325ull;  // FNV-1a, 64 bits (Fowler, Noll, Vo)
        if (valid) {
            uint64_t at;
            const uint64_t len = in.length(t, at);
            each_word(in.bytes + at, len, [&](uint64_t, uint64_t w, int n) {
                for (int x = 0; x < n; ++x) {
                    h ^= w >> (8 * x) & 0xff;
                    h *= 0x100000001b3ull;
                }
                return true;
            });
        }
        int leader = lane;
        for (uint64_t rem = dev::ballot(valid); rem;) {
            const int first = __builtin_ctzll(rem);
            const uint64_t same = dev::ballot(h == __shfl(h, first, dev::kWave)) & rem;
            if (same >> lane & 1) leader = first;
            rem &= ~same;
        }
        uint64_t s = 0;
        if (valid && leader == lane) {
            s = tab.find(h);
            const uint32_t mine = ~(uint32_t)t;
            if (__hip_atomic_load(tab.lead + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < mine)
                atomicMax(tab.lead + s, mine);
        }
        s = __shfl(s, leader, dev::kWave);
        if (valid) {
            slot[t] = (uint32_t)s;
            slot_hi[t] = (uint32_t)(s >> 32);
        }
    }
}

// lead[t] (in place of t's slot, whose upper half is in first[t]) = the first term of t's hash; first[t] = 1
// and len[t] = its length if that is t itself (else 0); the flag raised if the
// two terms differ.
__global__ __launch_bounds__(256) void check_terms(Terms in, TermTable tab, uint32_t *lead,
                                                   uint32_t *first, uint32_t *len,
                                                   uint32_t *differ) {
    TID_GRID_LOOP(t, in.m) {
        const uint32_t a = ~tab.lead[(uint64_t)first[t] << 32 | lead[t]];
        uint64_t at, at_a;
        const uint64_t l = in.length(t, at);
        bool eq = true;
        if (a != t) {
            eq = in.length(a, at_a) == l;
            if (eq)
                each_word(in.bytes + at, l, [&](uint64_t k, uint64_t w, int n) {
                    const uint8_t *q = in.bytes + at_a;
                    uint64_t v = 0;
                    if (n == 8) v = eight_bytes(q + k);
                    else if (l >= 8) v = eight_bytes(q + l - 8) >> (64 - 8 * n);
                    else for (int x = 0; x < n; ++x) v |= (uint64_t)q[k + x] << (8 * x);
                    eq = v == w;
                    return eq;
                });
        }
        if (!eq) dev::raise(differ);
        lead[t] = a;
        first[t] = a == t ? 1u : 0u;
        len[t] = a == t ? (uint32_t)l : 0u;
    }
}

// Every term's ID; a first appearance also writes its string to the dictionary.
__global__ __launch_bounds__(256) void write_terms(Terms in, const uint32_t *lead,
                                                   const uint64_t *rank, const uint64_t *place,
                                                   uint32_t *rows, uint64_t *doff,
                                                   uint8_t *dbytes) {
    TID_GRID_LOOP(t, in.m) {
        const uint32_t a = lead[t];
        const uint64_t r = rank[a];
        rows[t] = (uint32_t)(r + 1);
        if (a != t) continue;
        uint64_t at;
        const uint64_t l = in.length(t, at), to = place[t];
        doff[r + 1] = to + l;
        if (r == 0) doff[0] = 0;
        copy_string(dbytes + to, in.bytes + at, l);
    }
}

__global__ void decode_lengths(const uint32_t *ids, uint64_t n, const uint64_t *doff,
                               uint64_t nterms, uint32_t *len, uint32_t *bad) {
    TID_GRID_LOOP(i, n) {
        const uint32_t id = ids[i];
        if (id == 0 || id > nterms) {
            dev::raise(bad);
            len[i] = 0;
        } else {
            len[i] = (uint32_t)(doff[id] - doff[id - 1]);
        }
    }
}

__global__ void decode_copy(const uint32_t *ids, uint64_t n, const uint64_t *doff,
                            const uint8_t *dbytes, uint64_t nterms, const uint64_t *out_off,
                            uint8_t *out) {
    TID_GRID_LOOP(i, n) {
        const uint32_t id = ids[i];
        if (id == 0 || id > nterms) continue;
        const uint64_t a = doff[id - 1], l = doff[id] - a;
        copy_string(out + out_off[i], dbytes + a, l);
    }
}

// The context's four pinned flags of a dictionary call.  Their kernels have
// run when the call ends, however it ends, so the next call may clear them.
struct Flags {
    tid_ctx *ctx;
    explicit Flags(tid_ctx *c) : ctx(c) {
        for (int x = 0; x < 4; ++x) at(x)[0] = 0;
    }
    Flags(const Flags &) = delete;
    Flags &operator=(const Flags &) = delete;
    ~Flags() { (void)hipStreamSynchronize(ctx->stream); }
    uint32_t *at(int x) const { return ctx->d_flags + 4 + x; }
    bool raised(int x) const { return *static_cast<const volatile uint32_t *>(at(x)) != 0; }
};

bool overlap(const void *a, uint64_t na, const void *b, uint64_t nb) {
    const auto x = (uintptr_t)a, y = (uintptr_t)b;
    return x < y + nb && y < x + na;
}

}  // namespace

std::unique_ptr<tid_dict> encode(tid_ctx *ctx, const uint8_t *bytes, uint64_t nbytes,
                                 const uint64_t *offsets, uint64_t n, int on_device,
                                 uint32_t *rows) {
    TID_REQUIRE(n < (1ull << 32) / 3, TID_E_UNSUPPORTED, "encode: too many triples");
    TID_REQUIRE(n == 0 || (offsets && rows), TID_E_INVALID_ARG, "encode: null argument");
    TID_REQUIRE(nbytes == 0 || bytes, TID_E_INVALID_ARG, "encode: null bytes");
    const uint64_t m = 3 * n;
    auto dict = std::make_unique<tid_dict>();
    dict->ctx = ctx;
    if (m == 0) {
        dict->offsets = DevBuf(ctx, 8);
        TID_HIP(hipMemsetAsync(dict->offsets.get(), 0, 8, ctx->stream));
        TID_HIP(hipStreamSynchronize(ctx->stream));
        return dict;
    }
    // Inputs on the device: buffers on the context's device are read where they
    // are, unless rows would be written over them or the offsets are misaligned.
    DevBuf bytes_in, off_in;
    Terms in{bytes, offsets, nbytes, m, nullptr, nullptr, nullptr};
    const auto kind = on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice;
    if (nbytes && (!on_device || overlap(bytes, nbytes, rows, m * 4) ||
                   !on_this_device(ctx, bytes))) {
        bytes_in = DevBuf(ctx, nbytes);
        TID_HIP(hipMemcpyAsync(bytes_in.get(), bytes, nbytes, kind, ctx->stream));
        in.bytes = bytes_in.get<const uint8_t>();
    }
    if (!on_device || (uintptr_t)offsets % 8 != 0 ||
        overlap(offsets, (m + 1) * 8, rows, m * 4) || !on_this_device(ctx, offsets)) {
        off_in = DevBuf(ctx, (m + 1) * 8);
        TID_HIP(hipMemcpyAsync(off_in.get(), offsets, (m + 1) * 8, kind, ctx->stream));
        in.off = off_in.get<const uint64_t>();
    }
    const Flags flags(ctx);
    in.falls = flags.at(0);
    in.past = flags.at(1);
    in.wide = flags.at(3);
    // 1-2: the first appearance of every term.  The table is 2/3 full if no
    // term repeats, and is given back before the prefix sums.
    DevBuf lead(ctx, m * 4), first(ctx, m * 4), len(ctx, m * 4);
    {
        const uint64_t cap = m + m / 2 + 1;
        DevBuf table(ctx, (cap + 1) * 12);
        TermTable tab{table.get<uint64_t>(), nullptr, cap};
        tab.lead = reinterpret_cast<uint32_t *>(tab.key + cap + 1);
        TID_HIP(hipMemsetAsync(table.get(), 0, (cap + 1) * 12, ctx->stream));
        hipLaunchKernelGGL(insert_terms, dim3(grid_of(m)), dim3(256), 0, ctx->stream, in, tab,
                           lead.get<uint32_t>(), first.get<uint32_t>());
        TID_HIP(hipGetLastError());
        hipLaunchKernelGGL(check_terms, dim3(grid_of(m)), dim3(256), 0, ctx->stream, in, tab,
                           lead.get<uint32_t>(), first.get<uint32_t>(), len.get<uint32_t>(),
                           flags.at(2));
        TID_HIP(hipGetLastError());
    }
    // 3: ranks and places
    DevBuf rank(ctx, (m + 1) * 8), place(ctx, (m + 1) * 8);
    exclusive_scan_async(ctx, first.get<const uint32_t>(), m, rank.get<uint64_t>());
    exclusive_scan_async(ctx, len.get<const uint32_t>(), m, place.get<uint64_t>());
    uint64_t sums[2];
    read_words(ctx, {rank.get<const uint64_t>() + m, place.get<const uint64_t>() + m}, sums);
    TID_REQUIRE(!flags.raised(0), TID_E_INVALID_ARG, "encode: offsets must not fall");
    TID_REQUIRE(!flags.raised(1), TID_E_INVALID_ARG, "encode: offsets past the bytes");
    TID_REQUIRE(!flags.raised(3), TID_E_UNSUPPORTED, "encode: a term of 2^32 bytes or more");
    TID_REQUIRE(!flags.raised(2), TID_E_UNSUPPORTED,
                "encode: two different terms share a 64-bit hash; not encoded");
    const uint64_t d = sums[0], total = sums[1];
    dict->offsets = DevBuf(ctx, (d + 1) * 8);
    dict->bytes = DevBuf(ctx, std::max<uint64_t>(total, 1));
    hipLaunchKernelGGL(write_terms, dim3(grid_of(m)), dim3(256), 0, ctx->stream, in,
                       lead.get<const uint32_t>(), rank.get<const uint64_t>(),
                       place.get<const uint64_t>(), rows, dict->offsets.get<uint64_t>(),
                       dict->bytes.get<uint8_t>());
    TID_HIP(hipGetLastError());
    TID_HIP(hipStreamSynchronize(ctx->stream));
    dict->n_terms = d;
    dict->n_bytes = total;
    return dict;
}

// Strings of n IDs, to host buffers: out_off gets n + 1 offsets (always);
// the bytes only if they fit cap_bytes (else TID_E_CAPACITY, the total in
// out_off[n]).  An ID of 0 or above the dictionary's size is refused.
void decode(tid_ctx *ctx, const tid_dict *dict, const uint32_t *ids, uint64_t n, int on_device,
            uint64_t *out_off, uint8_t *out, uint64_t cap_bytes) {
    TID_REQUIRE(out_off, TID_E_INVALID_ARG, "decode: null offsets");
    if (n == 0) {
        out_off[0] = 0;
        return;
    }
    TID_REQUIRE(ids, TID_E_INVALID_ARG, "decode: null ids");
    DevBuf did;
    const uint32_t *I = ids;
    if (!on_device) {
        did = DevBuf(ctx, n * 4);
        TID_HIP(hipMemcpyAsync(did.get(), ids, n * 4, hipMemcpyHostToDevice, ctx->stream));
        I = did.get<const uint32_t>();
    }
    DevBuf len(ctx, n * 4), off(ctx, (n + 1) * 8);
    const Flags flags(ctx);
    hipLaunchKernelGGL(decode_lengths, dim3(grid_of(n)), dim3(256), 0, ctx->stream, I, n,
                       dict->offsets.get<const uint64_t>(), dict->n_terms, len.get<uint32_t>(),
                       flags.at(0));
    TID_HIP(hipGetLastError());
    exclusive_scan_async(ctx, len.get<const uint32_t>(), n, off.get<uint64_t>());
    TID_HIP(hipMemcpyAsync(out_off, off.get(), (n + 1) * 8, hipMemcpyDeviceToHost, ctx->stream));
    TID_HIP(hipStreamSynchronize(ctx->stream));
    TID_REQUIRE(!flags.raised(0), TID_E_INVALID_ARG, "decode: an ID is 0 or not in the dictionary");
    const uint64_t total = out_off[n];
    TID_REQUIRE(total <= cap_bytes, TID_E_CAPACITY, "decode: the strings need more bytes");
    if (total == 0) return;
    TID_REQUIRE(out, TID_E_INVALID_ARG, "decode: null output bytes");
    DevBuf dout(ctx, total);
    hipLaunchKernelGGL(decode_copy, dim3(grid_of(n)), dim3(256), 0, ctx->stream, I, n,
                       dict->offsets.get<const uint64_t>(), dict->bytes.get<const uint8_t>(),
                       dict->n_terms, off.get<const uint64_t>(), dout.get<uint8_t>());
    TID_HIP(hipGetLastError());
    TID_HIP(hipMemcpyAsync(out, dout.get(), total, hipMemcpyDeviceToHost, ctx->stream));
    TID_HIP(hipStreamSynchronize(ctx->stream));
}

}  // namespace tid
