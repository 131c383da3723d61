// reduce.hpp -- launch interface of the reductions of groups of PCFs
// (reduce.hip): the tree levels, the standard deviation's sums and the
// root's row rule.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace pcf {

// Reductions of groups of PCFs (reduce.hip). Ops as in pcf_reduce_op.
// RO_SUB, RO_MUL and RO_SQDIFF (a - b, ab, (a - b)^2) are combinations of two
// PCFs only: not associative, so never reduced over more than a pair.
enum { RO_SUM = 0, RO_MEAN = 1, RO_MAX = 2, RO_MIN = 3, RO_STD = 4, RO_SUB = 5, RO_MUL = 6, RO_SQDIFF = 7 };
struct RedLevelArgs {
    const int64_t *offsets;  // the set's CSR offsets (device, n+1)
    const int64_t *groups;   // group offsets (device, B+1)
    const int32_t *row_pcf;  // the PCF of every row (device, P)
    int64_t n;
    int32_t B;
    int level;               // inputs are items of 2^level PCFs
    const void *tin, *vin;
    void *tout, *vout;
};
// Several levels in one pass (red_fuse): bundles of at most kFuseLists items.
constexpr int kFuseLevels = 4;
constexpr int kFuseLists = 1 << kFuseLevels;
constexpr int kFuseSpacing = 48;  // rows between a list's samples
constexpr int kFuseRanks = 24;    // samples between tile starts
constexpr int kFuseTile = kFuseRanks * kFuseSpacing + kFuseLists * kFuseSpacing;
constexpr int kFuseSplit = kFuseLists + 1;
// The fused passes are taken for at most kFuseFew bundles in the first one or
// from kFuseRows rows a bundle on average: a bundle takes a workgroup of its own
// at least, and its entry of the host's table. Means, FP64, whole calls, single
// levels / fused, us: 33,333 groups of 3 PCFs, 60 rows a bundle 491 / 865; 8,032
// of 3, 249 rows 212 / 265; 5,000 of 16, 400 rows 326 / 314; 1,893 of 33 (3
// bundles each), 512 rows 345 / 356; 2,861 of 3, 699 rows 168 / 168; 1,818 of 4,
// 1,100 rows 178 / 159; 100 of 16, 192 rows 133 / 81; 3,000 of 16, 192 rows 229 /
// 207; 1,000 of 60 (4,000 bundles), 192 rows 245 / 278.
constexpr int64_t kFuseRows = 512, kFuseFew = 3000;
struct RedBundle {
    int64_t p0, pend;       // its PCFs (one output item)
    int64_t sample0, tile0; // its first sample and tile
};
struct RedFuseArgs {
    const int64_t *offsets;  // the set's CSR offsets (device, n+1)
    const RedBundle *bundles;
    int64_t nbundles, nsamples, ntiles;
    int level, depth;        // inputs are items of 2^level PCFs, outputs of 2^(level + depth)
    const void *tin, *vin;
    void *tout, *vout;
    int64_t *split;          // scratch, kFuseSplit a tile: where its lists begin, its bundle
};
struct RedStdArgs {
    const int64_t *offsets, *groups;
    int32_t B;
    int64_t rows;            // the set's total rows
    const void *t, *v;       // the set
    const void *rt, *rv;     // the sum tree's roots
    void *q;                 // out: sum of squared deviations per root row
    int64_t nchunks;         // the root pass's chunks (red_std_small)
    const int64_t *chunk_row, *chunk_grp;
    int64_t *chunk_first;    // scratch, 64 per chunk: PCF i's row at or before
                             // the chunk's first time
};
struct RedScanArgs {
    int64_t nchunks;
    int32_t B;
    const int64_t *chunk_cnt, *chunk_grp;
    int64_t *chunk_off;      // out: the output row of every chunk
    int64_t *offsets_out;    // out: the B groups' offsets
};
struct RedEmitArgs {
    const int64_t *offsets, *groups;
    int op;
    const void *rt, *rv;     // roots: times, and the values the rule compares
    int64_t nchunks;         // chunks of at most 1024 rows of one group
    const int64_t *chunk_row, *chunk_grp;
    int fill;                // 0: chunk_cnt[c] = kept rows; 1: write them
    int64_t *chunk_cnt;
    const int64_t *chunk_off;
    const int64_t *out_end;  // device: the output's total rows (fill)
    void *t_out, *v_out;
};
hipError_t launch_red_level(bool f64, int op, const RedLevelArgs &a, int64_t rows,
                            hipStream_t s);
// Levels a.level .. a.level + a.depth - 1 (ops of a tree: sum, max, min).
hipError_t launch_red_fuse(bool f64, int op, const RedFuseArgs &a, hipStream_t s);
hipError_t launch_red_interleave(bool f64, int64_t n, const int64_t *xo, const void *xt,
                                 const void *xv, const int64_t *yo, const void *yt,
                                 const void *yv, const int64_t *zo, void *zt, void *zv,
                                 hipStream_t s);
hipError_t launch_red_rowmap(const int64_t *offsets, int64_t n, int32_t *row_pcf, hipStream_t s);
// groups of more than 64 PCFs (a search per PCF and root row)
hipError_t launch_red_std(bool f64, const RedStdArgs &a, hipStream_t s);
// groups of at most 64 PCFs (a block per chunk of root rows, the PCF rows
// it selects staged in LDS)
hipError_t launch_red_std_small(bool f64, const RedStdArgs &a, hipStream_t s);
hipError_t launch_red_scan(const RedScanArgs &a, hipStream_t s);
hipError_t launch_red_emit(bool f64, const RedEmitArgs &a, hipStream_t s);

}  // namespace pcf
