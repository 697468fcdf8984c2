// The filter's copy for the convolution kernel whose input rows stay in LDS, the choice of its tile and its launch.
#include "gemm_conv_plane.h"

#include <cmath>

#include "gemm_direct.h"

namespace nt {

// filter [F][C][RS] (row pitch ldb) -> [F][C / 32][RS][32]: one workgroup per filter, the row read and written 16 bytes per
// thread, permuted on its way through LDS
__global__ __launch_bounds__(256) void conv_plane_filter_kernel(const uint16_t *w, int64_t ldb, uint16_t *out, int32_t C, int32_t RS)
{
    extern __shared__ __attribute__((aligned(16))) uint16_t row[];
    const int32_t K = C * RS, B = 32 * RS;
    const uint16_t *src = w + (int64_t)blockIdx.x * ldb;
    uint16_t *dst = out + (int64_t)blockIdx.x * K;
    for (int32_t i = threadIdx.x * 8; i < K; i += 2048) {
        u32x4 v;
        __builtin_memcpy(&v, src + i, 16);
        *reinterpret_cast<u32x4 *>(row + i) = v;
    }
    __syncthreads();
    for (int32_t j = threadIdx.x * 8; j < K; j += 2048) {
        const int32_t block = j / B, in = j - block * B, tap = in >> 5, c = block * 32 + (in & 31);
        uint32_t e[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) e[i] = row[(c + i) * RS + tap];
        *reinterpret_cast<u32x4 *>(dst + j) = u32x4{e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
    }
}

nt_status launch_conv_plane_filter(const uint16_t *w, int64_t ldb, uint16_t *out, int32_t F, int32_t C, int32_t RS, hipStream_t s)
{
    // (at most 32768 elements per filter: a row fits LDS)
    hipLaunchKernelGGL(conv_plane_filter_kernel, dim3((unsigned)F), dim3(256), (size_t)C * RS * sizeof(uint16_t), s, w, ldb, out, C, RS);
    return check_launch("conv_plane_filter_kernel");
}

template <int TMA, int TMB, int TN, int U, int TAPS> nt_status launch_conv_plane_t(const ConvPlaneArgs &a, bool bf16, hipStream_t s);
#define NT_PLANE_ENTRY(TMA, TMB, TN, U, TAPS) extern template nt_status launch_conv_plane_t<TMA, TMB, TN, U, TAPS>(const ConvPlaneArgs &, bool, hipStream_t);
NT_PLANE_TILES(NT_PLANE_ENTRY)
#undef NT_PLANE_ENTRY
struct PlaneTile { int tma, tmb, tn, u, taps; nt_status (*launch)(const ConvPlaneArgs &, bool, hipStream_t); };
#define NT_PLANE_ENTRY(TMA, TMB, TN, U, TAPS) {TMA, TMB, TN, U, TAPS, launch_conv_plane_t<TMA, TMB, TN, U, TAPS>},
static const PlaneTile kPlaneTiles[] = {NT_PLANE_TILES(NT_PLANE_ENTRY)};
#undef NT_PLANE_ENTRY

nt_conv_plan conv_plane_describe(const ConvPlanePlan &p)
{
    const PlaneTile &t = kPlaneTiles[p.tile];
    return nt_conv_plan{2, {32 * t.tma, 32 * t.tmb}, 32 * t.tn, {(int32_t)p.mt_a, (int32_t)(p.mt - p.mt_a)}, kThreads / 64, t.u};
}
nt_status launch_conv_plane(const ConvPlaneArgs &a, const ConvPlanePlan &p, bool bf16, hipStream_t s) { return kPlaneTiles[p.tile].launch(a, bf16, s); }

// Tile heights and widths by an estimate (us): the filter's copy, then rounds of one program per unit.  A program costs a fixed
// part, its epilogue, and its trips: the matrix instructions, or the LDS reads, or (taps in a loop) the bookkeeping between
// them; rows that start off 16 bytes keep the loads of a block longer.  Fits; 57 drawn convolutions that it sends here
// take 1.09 times its figure in the mean, with a spread of 8 % (four sets of operands in turn, graph replays).
bool conv_plane_plan(const ConvHint &h, ConvPlaneArgs *a, ConvPlanePlan *best, double *cost_out)
{
    const int64_t PQ = h.P * h.Q, PQ8 = (PQ + 7) / 8 * 8, M = h.N * PQ8, RS = h.R * h.S;
    const int64_t span = (h.R - 1) * h.dh + 1, row = (h.Q - 1) * h.sw + (h.S - 1) * h.dw + 1;
    const int64_t last_h = std::min<int64_t>(h.H - 1, (h.P - 1) * h.sh + span - 1 - h.ph);
    const int64_t below = std::max<int64_t>((h.P - 1) * h.sh + span - 1 - h.ph - (h.H - 1), 0);
    double cost = 0;
    int64_t best_plane = 0;
    int i = -1;
    for (const PlaneTile &t : kPlaneTiles) {
        ++i;
        if (t.taps != (RS == 9 ? 9 : 0)) continue;
        // the most output rows and images that a tile touches, the most input rows under them, the most real ones (where images meet,
        // the padding below one and above the next is none), the most runs of eight elements (an image's may begin and end inside one)
        const int64_t BM = 32 * t.tma, out_rows = std::min<int64_t>((BM + h.Q - 2) / h.Q + 1, h.N * h.P);
        const int64_t images = std::min<int64_t>(std::min<int64_t>((BM + PQ8 - 2) / PQ8 + 1, h.N), out_rows);
        const int64_t rows = std::max((out_rows - 1) * h.sh + span, (out_rows - images) * h.sh + images * span);
        int64_t real = 0;
        for (int64_t n = 1; n <= images; ++n) real = std::max(real, (out_rows - n) * h.sh + n * span - (n - 1) * (h.ph + below));
        real = std::min(real, images * std::max<int64_t>(last_h + 1, 0));
        const int64_t runs = (real * h.W + 7) / 8 + (h.W % 8 ? images + 1 : 0), plane = (rows * row * 16 + 16 + 255) / 256 * 256;
        if (2 * runs > 64 * t.u || 3 * 32 * t.tn * 64 + t.u * 16384 + (t.u == 2 ? 8 : 4) * plane > (160 << 10)) continue;
        const int64_t nt_ = (h.K + 32 * t.tn - 1) / (32 * t.tn), units = 256, blocks = (M + 31) / 32;
        const double off16 = (h.H * h.W % 8 ? 0.4 : 0.0) + (h.W % 2 ? 0.16 : 0.0);
        auto program = [&](int height) {
            const double mm = height * t.tn, trip = std::max(0.129 + 0.0061 * mm, 0.02 + 0.015 * (height + t.tn)) + (t.taps ? 0.0 : 0.058);
            return 9.5 + (0.031 + (PQ % 2 ? 0.17 : 0.0)) * mm + (double)(h.C / 32) * ((double)RS * trip + (t.u == 3 ? 0.42 : 0.0) + off16 * t.u);
        };
        auto consider = [&](int64_t mt_a) {
            const int64_t left = std::max<int64_t>(blocks - mt_a * t.tma, 0), mt_b = (left + t.tmb - 1) / t.tmb;
            const int64_t ra = (mt_a * nt_ + units - 1) / units, rb = (mt_b * nt_ + units - 1) / units;
            const double c = 0.3 + (double)ra * program(t.tma) + (double)rb * program(t.tmb);
            if (cost == 0 || c < cost) { cost = c; best->tile = i; best->mt_a = mt_a; best->mt = mt_a + mt_b; best_plane = plane; }
        };
        const int64_t per_round = std::max<int64_t>(units / nt_, 1), all = (blocks + t.tma - 1) / t.tma;
        consider(0);
        for (int64_t mt_a = per_round; mt_a < all; mt_a += per_round) consider(mt_a);
        consider(all);
    }
    if (cost == 0) return false;
    const PlaneTile &t = kPlaneTiles[best->tile];
    a->c.M = (int32_t)M; a->c.N = (int32_t)h.K; a->c.Q8 = a->c.PQ8 = (int32_t)PQ8; a->c.Q = (int32_t)PQ;
    a->c.mt = best->mt; a->c.mt_a = (int32_t)best->mt_a; a->c.nt = (h.K + 32 * t.tn - 1) / (32 * t.tn);
    a->c.syn = h.ys[0]; a->c.syf = h.ys[1]; a->c.slice = 0;
    a->xs1 = h.xs[1]; a->xs0 = (uint32_t)h.xs[0];
    a->blocks = (int32_t)(h.C / 32); a->R = (int32_t)h.R; a->S = (int32_t)h.S;
    a->H = (int32_t)h.H; a->W = (int32_t)h.W; a->P = (int32_t)h.P; a->Q = (int32_t)h.Q; a->PQ = (int32_t)PQ;
    a->sh = (int32_t)h.sh; a->sw = (int32_t)h.sw; a->ph = (int32_t)h.ph; a->pw = (int32_t)h.pw;
    a->span = (int32_t)span; a->image = (int32_t)((h.P - 1) * h.sh + span); a->row = (int32_t)row; a->last_h = (int32_t)last_h;
    a->units = (int32_t)(last_h >= 0 ? ((last_h + 1) * h.W + 7) / 8 : 1);
    a->tap_col = (uint32_t)(h.dw * 16);
    a->tap_row = (uint32_t)(h.dh * row * 16);
    a->plane = (uint32_t)best_plane;
    a->inv_pq8 = 1.f / (float)PQ8; a->inv_q = 1.f / (float)h.Q; a->inv_w = 1.f / (float)h.W; a->inv_units = 1.f / (float)a->units;
    *cost_out = cost;
    return true;
}

}  // namespace nt
