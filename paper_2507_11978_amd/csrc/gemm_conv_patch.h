// Convolution of few output positions in one launch, straight from the caller's tensors (gemm_conv_patch.hip).
#pragma once
#include <cstdint>

#include <hip/hip_runtime.h>

#include "kernels.h"

namespace nt {

constexpr int kPatchMaxTaps = 25;

// x: planes (n, c) of H * W contiguous elements; w: rows of C * RS contiguous elements, 16-byte aligned; y: planes of P * Q.
struct ConvPatchArgs {
    const uint16_t *x, *w;
    void *Y;
    int64_t xs1, syn, syf;         // elements between channels of x, images and filters of Y
    uint32_t xs0, ldb;             // elements between images of x, filters of w (offsets below 2^31 bytes)
    int32_t F, M, blocks;          // filters, positions N * P * Q, blocks of 32 channels
    int32_t H, W, P, Q, PQ;
    int32_t sh, sw, ph, pw;
    int32_t ft, pt, f_major;       // tiles of filters and positions; whether consecutive programs share a filter tile
    // the patch in LDS: slots of one input position each, `row` slots per input row, zero where the padding lies
    int32_t span;                  // input rows under a filter: (R - 1) dh + 1
    int32_t image;                 // ... under an image's output
    int32_t row;
    int32_t last_h;                // last input row that an image's output reads
    int32_t units;                 // runs of four elements that this takes
    uint32_t plane, region;        // bytes of a plane (8 channels), of a wavefront's whole region
    int32_t inner;                 // tiles of the operand that changes from program to program
    float inv_inner, inv_pq, inv_q, inv_w, inv_units;       // reciprocals
    int32_t tap[kPatchMaxTaps];    // byte offset of each tap in a plane
    int out_dtype;
    // loader trace (nullptr otherwise): 32 k of one tap of one block of channels, as the matrix instructions read them
    uint16_t *trace_out;
    int32_t trace_program, trace_slice, trace_operand;
};

struct ConvPatchPlan { int tile, waves; };     // wavefronts per program: the parts of the reduction
// geometry, tile and estimated time (us) for a convolution; false: not built for it
bool conv_patch_plan(const ConvHint &h, ConvPatchArgs *a, ConvPatchPlan *p, double *cost);
nt_conv_plan conv_patch_describe(const ConvPatchArgs &a, const ConvPatchPlan &p);
// (trace: one workgroup, one slice of one operand to a.trace_out)
nt_status launch_conv_patch_trace(const ConvPatchArgs &a, const ConvPatchPlan &p, hipStream_t s);
nt_status launch_conv_patch(const ConvPatchArgs &a, const ConvPatchPlan &p, bool bf16, hipStream_t s);

}  // namespace nt
