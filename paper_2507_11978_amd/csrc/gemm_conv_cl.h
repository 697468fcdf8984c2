// Convolution on a channels-last copy of its input (gemm_conv_cl.hip).
#pragma once
#include <cstdint>

#include <hip/hip_runtime.h>

#include "kernels.h"

namespace nt {

struct ConvClArgs {
    const uint16_t *P;             // the copy, [n][Hc][Wc][C], dense, zero where the padding lies
    const uint16_t *Wt;            // filter, tap-major: [f][r][s][c], dense
    void *Y;                       // output: element (f, n, pq) at n * syn + f * syf + pq
    int64_t syn, syf;
    int32_t F, M, C, K;            // filters, output positions N * P * Q, channels (a multiple of 32), C * R * S
    int32_t PQ, Q, Hc, Wc;
    int32_t S, sp, sq, dh, dw;     // filter columns; step of an output row / column and of a filter row / column in the copy
    int32_t mt, nt;                // tiles of filters and of positions
    int32_t ksplit, per;           // parts of the reduction, 32-k slices per part (ksplit 1: all of them)
    float *ws;                     // ksplit > 1: the parts, fp32, [part][f][m]
    int out_dtype;
    uint16_t *trace_out;           // loader trace (gemm_direct16.h): program i * mt + j for tile i of positions and j of filters
    int64_t trace_program;
    int32_t trace_slice, trace_operand;
};

// What the copies are made from.  Copy position (hc, wc) is input position (hc * eh - ph, wc * ew - pw).
struct ConvClCopy {
    const uint16_t *x;
    uint16_t *P;
    int64_t xs[4];
    int32_t N, C, H, W, Hc, Wc, ph, pw, eh, ew;
    const uint16_t *w;             // filter [F][C][R * S], row pitch ldb; nullptr: no filter copy
    uint16_t *Wt;
    int64_t ldb;
    int32_t F, RS;
};

nt_status launch_conv_cl_copy(const ConvClCopy &c, hipStream_t s);
// tile: 64 (x 64) or 128 (x 128)
nt_status launch_conv_cl(const ConvClArgs &a, int tile, bool bf16, hipStream_t s);
// the loader trace of the same kernel: one workgroup
nt_status launch_conv_cl_trace(const ConvClArgs &a, int tile, hipStream_t s);

}  // namespace nt
