// Convolution of many output positions with its input rows resident in LDS (gemm_conv_plane.hip).
#pragma once
#include <cstdint>

#include <hip/hip_runtime.h>

#include "gemm_conv.h"

namespace nt {

// c: the output side (Y, syn, syf, filters N, positions M, out_dtype), positions numbered n * PQ8 + pq with PQ8 = P * Q rounded up
// to 8 (conv_store_rows16 sees images of one row), and mt / mt_a / nt tiles.
struct ConvPlaneArgs {
    ConvArgs c;
    const uint16_t *x, *w;         // x: planes (n, c) of H * W contiguous elements; w: [filter][block of 32 channels][tap][32]
    int64_t xs1;                   // elements between channels
    uint32_t xs0, ldb;             // elements between images, filters
    int32_t blocks, R, S;
    int32_t H, W, P, Q, PQ;
    int32_t sh, sw, ph, pw;
    int32_t span, image, row, last_h, units;      // as in ConvPatchArgs; units: runs of eight elements
    uint32_t tap_col, tap_row;     // bytes in a plane from a tap to the next in its row, in its column
    uint32_t plane;                // bytes of a plane (8 channels)
    float inv_pq8, inv_q, inv_w, inv_units;
};

// the kernels that are built: heights of the tile in 32 positions, width in 32 filters, runs per lane and block, taps (0: any)
#define NT_PLANE_TILES(X) \
    X(8, 7, 8, 2, 9) X(7, 6, 8, 2, 9) X(6, 5, 8, 2, 9) X(5, 4, 8, 2, 9) X(4, 3, 8, 2, 9) X(4, 3, 8, 3, 9) \
    X(8, 7, 4, 2, 9) X(7, 6, 4, 2, 9) X(6, 5, 4, 2, 9) X(5, 4, 4, 2, 9) X(4, 3, 4, 2, 9) X(4, 3, 4, 3, 9) \
    X(6, 5, 8, 2, 0) X(4, 3, 8, 2, 0) X(8, 7, 8, 3, 0) X(6, 5, 8, 3, 0) X(4, 3, 8, 3, 0) X(8, 7, 4, 2, 0) X(4, 3, 4, 2, 0) X(8, 7, 4, 3, 0)

struct ConvPlanePlan { int tile; int64_t mt_a, mt; };      // tile heights, tiles of the first height, of both
// geometry, tile and estimated time (us); false: its input rows do not fit
bool conv_plane_plan(const ConvHint &h, ConvPlaneArgs *a, ConvPlanePlan *p, double *cost);
nt_conv_plan conv_plane_describe(const ConvPlanePlan &p);
nt_status launch_conv_plane(const ConvPlaneArgs &a, const ConvPlanePlan &p, bool bf16, hipStream_t s);
// loader trace: one workgroup, one slice of one operand to a.c.trace_out (gemm_conv_plane_trace.hip)
nt_status launch_conv_plane_trace(const ConvPlaneArgs &a, const ConvPlanePlan &p, hipStream_t s);
// filter [F][C][RS] (row pitch ldb) -> [F][C / 32][RS][32]
nt_status launch_conv_plane_filter(const uint16_t *w, int64_t ldb, uint16_t *out, int32_t F, int32_t C, int32_t RS, hipStream_t s);

}  // namespace nt
