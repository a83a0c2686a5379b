// idcounts.hpp -- how many triples of a graph hold each ID at one position, on
// the host (load-time statistics: they bound scan outputs).  Host code alone.
#pragma once

#include <algorithm>
#include <cstdint>
#include <memory>
#include <vector>

namespace tid {

// How many triples hold each ID at one position, on the host: one byte an ID
// (255: the count is in `big`), and per block of 256 IDs the triples and the
// `big` entries of all IDs before it.  Eight and a half bits an ID instead of the
// 64 of a cumulative count, which is what loading a graph waits for: the copy to
// the host and the first touch of its pages.
struct IdCounts {
    static constexpr uint32_t kBlock = 256;
    static constexpr uint32_t kBig = 255;
    struct Mem {
        std::unique_ptr<uint8_t[]> bytes;   // of every position
        std::unique_ptr<uint64_t[]> rows;   // per block: triples before it
        std::unique_ptr<uint64_t[]> nbig;   // per block: `big` entries before it
        std::unique_ptr<uint32_t[]> big;
    };
    std::shared_ptr<Mem> mem;               // shared by a graph's positions
    uint64_t first = 0;                     // the position's first block in `mem`
    uint64_t ids = 0;                       // IDs 0 .. ids - 1 (0: not counted)
    uint64_t total = 0;                     // triples
    bool empty() const { return ids == 0; }
    // triples whose position holds an ID below `id`
    uint64_t below(uint64_t id) const {
        if (id >= ids) return total;
        const uint64_t b = first + id / kBlock;
        uint64_t s = mem->rows[b] - mem->rows[first];
        const uint8_t *c = mem->bytes.get() + b * kBlock;
        uint32_t sum = 0, nbig = 0;
        for (uint32_t i = 0; i < id % kBlock; ++i) {
            sum += c[i];
            nbig += c[i] == kBig;
        }
        s += sum;
        const uint32_t *big = mem->big.get() + mem->nbig[b];
        for (uint32_t i = 0; i < nbig; ++i) s += big[i] - kBig;
        return s;
    }
};

// The counts of whole blocks of bins (as many bins as `blocks` blocks hold), in
// 64-bit sums.
inline std::shared_ptr<IdCounts::Mem> counts_of_bins(const uint32_t *bins, uint64_t blocks) {
    auto m = std::make_shared<IdCounts::Mem>();
    m->bytes.reset(new uint8_t[blocks * IdCounts::kBlock]);
    m->rows.reset(new uint64_t[blocks + 1]);
    m->nbig.reset(new uint64_t[blocks + 1]);
    std::vector<uint32_t> big;
    uint64_t rows = 0;
    for (uint64_t b = 0; b < blocks; ++b) {
        m->rows[b] = rows;
        m->nbig[b] = big.size();
        const uint32_t *in = bins + b * IdCounts::kBlock;
        uint8_t *out = m->bytes.get() + b * IdCounts::kBlock;
        uint32_t any = 0;
        for (uint32_t i = 0; i < IdCounts::kBlock; ++i) any |= in[i];
        if (any < IdCounts::kBig) {  // most blocks: vector code, sums of 32 bits
            uint32_t sum = 0;
            for (uint32_t i = 0; i < IdCounts::kBlock; ++i) sum += in[i];
            for (uint32_t i = 0; i < IdCounts::kBlock; ++i) out[i] = (uint8_t)in[i];
            rows += sum;
            continue;
        }
        for (uint32_t i = 0; i < IdCounts::kBlock; ++i) {
            out[i] = (uint8_t)std::min(in[i], IdCounts::kBig);
            if (in[i] >= IdCounts::kBig) big.push_back(in[i]);
            rows += in[i];
        }
    }
    m->rows[blocks] = rows;
    m->nbig[blocks] = big.size();
    m->big.reset(new uint32_t[std::max<size_t>(big.size(), 1)]);
    std::copy(big.begin(), big.end(), m->big.get());
    return m;
}

}  // namespace tid
