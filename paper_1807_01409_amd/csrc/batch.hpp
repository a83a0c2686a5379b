// batch.hpp -- job descriptors of the batched small joins and sorts
// (batch.hip): one workgroup per job, many plans' jobs in one launch.
#pragma once

#include "internal.hpp"

namespace tid {

constexpr int kBatchBlock = 256;
constexpr int kJoinBlock = 1024;             // threads of a small join's count or expansion (LDS table)
constexpr uint32_t kSmallRows = 4096;       // rows per side of a batched join
constexpr uint32_t kSmallSlots = 8192;      // LDS hash slots (>= 2 * kSmallRows)
constexpr int kSmallCols = 8;               // columns per side of a batched join
constexpr int kSmallEq = 4;                 // other shared variables of a batched join
constexpr uint32_t kEmptyKey = 0xFFFFFFFFu;  // empty LDS hash slot (the ID itself has its own slot)
// A join job without other shared variables is expanded in tiles of
// kSplitTile output rows, a workgroup each.
constexpr uint32_t kSplitTile = 2048;

struct JoinJob {
    const uint32_t *lkey, *rkey;
    uint32_t nl, nr;
    int32_t neq, nlc, nrc;
    const uint32_t *eq_l[kSmallEq], *eq_r[kSmallEq];
    const uint32_t *lcol[kSmallCols], *rcol[kSmallCols];
    uint32_t *out[2 * kSmallCols];
    uint32_t *off;     // nl + 1 entries
    uint32_t *lbase;   // neq == 0: nl entries, where each L row's key group starts in grp
    uint32_t *grp;     // neq == 0: nr entries, R row indices grouped by key
    uint64_t *total;
    uint32_t nout;     // output rows (set on the host for the expansion)
};

// A join job expanded in tiles (neq == 0), with its first tile in the
// expansion launch.
struct SplitJob {
    JoinJob j;
    uint32_t tile0;
};

// A table to put in lexicographic row order with the round's other sorts
// (sort_rows_batched, sort.hip): input, output (n rows allocated).
struct RowSortJob {
    const tid_table *in;
    tid_table *out;
    uint64_t n;
};
void sort_rows_batched(tid_ctx *ctx, const std::vector<RowSortJob> &jobs,
                       std::vector<DevBuf> &keep, std::vector<std::vector<char>> &host_keep);

// Jobs of one round of a batch, launched together; the device job tables
// and the host copies they came from (some in tid_ctx::uploads) are kept until
// the round's wait.
struct BatchState {
    std::vector<JoinJob> count_jobs, expand_jobs;
    std::vector<RowSortJob> row_sorts;
    std::vector<DevBuf> keep;
    std::vector<std::vector<char>> host_keep;
    std::vector<std::unique_ptr<tid_table>> keep_tables;  // inputs of queued sorts
    uint64_t big_out_total = 0;   // rows of the queued larger-join expansions
    std::vector<struct BigJoinReq> big_reqs;
    std::vector<struct BigExpand> big_expand_jobs;
};
// launch and clear the queued jobs of one kind
void flush_join_jobs(tid_ctx *ctx, BatchState &bs, bool expand);
void flush_sort_jobs(tid_ctx *ctx, BatchState &bs);

}  // namespace tid

namespace tid {

// Larger hash joins of a batch (sides above kSmallRows rows): every join of
// a round in the same few launches over the concatenation of all the joins'
// rows.  Count phase: build (insert with per-workgroup rank reservation in LDS,
// slot scan, fill; large build sides are sorted instead), probe into entries
// per tile, scan of the tiles' output rows, per-join totals; expansion phase
// (next round): one output-row-parallel launch for all joins.
constexpr int kBigCols = TID_MAX_COLS;
// largest build side of a batched larger join (as the automatic choice of
// tid_join: 2^23 rows, 2^24 slots)
constexpr uint64_t kBigBuildMax = 1ull << 23;

// "l" is the probe side and "r" the build side here (the build is the
// smaller table, which may be the join's L or R); eq_l / eq_r are columns of
// the probe / build side that must agree (the join's other shared variables).
// matched, unmatched: whether probe rows with, without a partner put out rows
// (inner join 1 0, left outer 1 1, the rest of a full outer join 0 1).
struct BigCount {
    const uint32_t *lkey, *rkey;
    uint64_t nl, nr;
    uint64_t rbase;            // offset in the concatenated hashed build rows
    uint64_t sbase;            // first slot in the concatenated slot arrays
    uint32_t mask;             // slots - 1 (a power of two minus one)
    uint32_t max_key;          // bound of the build keys
    int32_t neq;
    int32_t matched, unmatched;
    const uint32_t *eq_l[kSmallEq], *eq_r[kSmallEq];
    // a sorted build side: run of each key >> shift (null: hashed), sorted keys
    const uint2 *index;
    const uint32_t *skey;
    int32_t shift;
    const uint32_t *rows;      // build rows grouped by key
};

// A probe row with output: its first build row (~0u: none), and the output
// rows of its tile before it.
struct BigEntry {
    uint32_t row, at;
    uint64_t pre;
};

constexpr uint8_t kFromProbe = 0, kFromBuild = 1, kFromNone = 2;
struct BigExpand {
    uint64_t tile0, tile1, obase;   // probe tiles, first output row
    const uint32_t *rows;           // build rows grouped by key
    int32_t neq, ncols;
    const uint32_t *eq_l[kSmallEq], *eq_r[kSmallEq];
    const uint32_t *col[kBigCols];  // output column c: this column of the side, or zeros
    uint32_t *out[kBigCols];
    uint8_t side[kBigCols];
};

// The device state of one round's larger joins, kept until their expansion.
struct BigArena {
    DevBuf buf;
    BigEntry *entries = nullptr;   // `tile` per probe tile
    uint32_t tile = 0;             // probe rows of a workgroup
    uint32_t *tcount = nullptr;    // entries of each tile
    uint64_t *toff = nullptr;      // per tile: output rows of all tiles before it
    std::vector<DevBuf> builds;    // sorted build sides
};

struct BigJoinReq {
    BigCount c;
    PendingJoin *pj;
};

// Count phase of the queued larger joins: launches, and points each
// PendingJoin's total at its word in the new arena.
void flush_big_count(tid_ctx *ctx, std::vector<BigJoinReq> &reqs,
                     std::shared_ptr<BigArena> *arena_out);
// Expansion of larger joins whose totals are known (each job's tiles refer to
// `arena`).
void flush_big_expand(tid_ctx *ctx, const BigArena &arena, std::vector<BigExpand> &jobs,
                      BatchState &bs);

}  // namespace tid

namespace tid {

// Many device-to-device copies of uint32 runs in one launch.
struct CopyJob {
    const uint32_t *src;
    uint32_t *dst;
    uint64_t n;
};
void batch_copy(tid_ctx *ctx, const std::vector<CopyJob> &jobs, BatchState &bs);

}  // namespace tid
