// Dispatch between the kernels, plus the small auxiliary kernels (zero fill, address trace).
#include <mutex>

#include "gemm_conv_cl.h"
#include "gemm_conv_direct.h"
#include "gemm_conv_patch.h"
#include "gemm_conv_plane.h"
#include "gemm_conv_tap.h"
#include "gemm_direct.h"
#include "gemm_direct16.h"
#include "gemm_skinny.h"
#include "kept.h"

namespace nt {

// ------------------------------------------------------------- auxiliary kernels
__global__ void fill_zero_kernel(void *C, const OperandMap mc, int64_t batch, int64_t sc_batch, int out_dtype)
{
    const int64_t total = mc.rows * mc.cols;
    for (int64_t b = blockIdx.y; b < batch; b += gridDim.y)
        for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
            const int64_t row = e / mc.cols, col = e % mc.cols;
            int64_t off;
            if (element_at(mc, row, col, row_part(mc, row), col_part(mc, col), &off))
                store_out(C, b * sc_batch + off, 0.f, out_dtype);
        }
}

__global__ void trace_tile_kernel(const OperandMap m, int64_t batch_off, int64_t row0, int64_t col0,
                                  int32_t rows, int32_t cols, int64_t *offsets_out, uint8_t *mask_out)
{
    const int64_t total = (int64_t)rows * cols;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t row = row0 + e / cols, col = col0 + e % cols;
        int64_t off;
        const bool ok = element_at(m, row, col, row_part(m, row), col_part(m, col), &off);
        offsets_out[e] = ok ? batch_off + off : -1;
        mask_out[e] = ok ? 1 : 0;
    }
}

struct TileEntry { int bm, bn, bk; };
static const TileEntry kTiles[] = {{64, 64, 32}, {128, 128, 64}, {256, 128, 64}, {128, 256, 64}, {256, 256, 64}};

// A compute unit works through p = ceil(programs / 256) programs; a program costs kt steps of `step` microseconds
// (time of one 64-wide k tile with the whole unit's matrix rate) plus a fixed `fixed` microseconds of launch, prologue and
// epilogue, which `resident` co-resident workgroups overlap with each other's multiplications.  The constants are fits to
// measurements on 8192 x 8192 x K and batched 2048 x 2048 x K problems.
static int gemm_ksplit(int64_t programs, int64_t kt, int64_t M, int64_t N, bool small, double *cost_out, bool uneven = false);
static bool beyond_l2(int64_t M, int64_t N, int64_t kt) { return (M + N) * kt * 64 * 2 > (32 << 20); }

nt_tile_cfg pick_gemm_tile(int64_t batch, int64_t M, int64_t N, int64_t K, bool narrow)
{
    struct Cand { int bm, bn; double fixed, step; int resident; };
    // (fits to 8192 x 8192 x K, 4096 x 4096 x K and 32 x 2048 x 2048 x K for K = 256 .. 8192 on a chip with every unit busy;
    // the 256 x 256 figures are those of the persistent kernel)
    const Cand cands[] = {{256, 256, 8.5, 1.42, 1}, {128, 256, 7.0, 0.82, 2}, {256, 128, 6.5, 0.915, 2}, {128, 128, 4.5, 0.51, 2}};
    const double kt = (double)((K + 63) / 64);
    // Products of at most two 64 x 64 tiles per unit leave a wider tile's matrix pipes waiting for its loads: the narrow tile
    // has four times the programs and an eighth of the reduction in flight per program.  Measured against 128 x 128, us:
    // 256 tiles 4.5 / 5.8 (K = 256), 7.3 / 10.7 (1024), 11.0 / 18.4 (2048); 512 tiles 5.8 / 6.2, 10.0 / 11.1, 16.9 / 18.6 and
    // 33.1 / 32.2 (4096); 576 tiles 7.6 / 6.1, 14.4 / 11.2.
    const int64_t small = batch * ((M + 63) / 64) * ((N + 63) / 64);
    // Not where a strip of a tile or two (M or N up to 128) fills more than a round of them (operands from memory, 128 x 128 / this:
    // 64 x 19712 x 960 14.2 / 18.5, 64 x 31936 x 704 12.9 / 14.9; unaligned rows 77 x 14309 x 2717 56 / 40), and not where the wider
    // tile's k split is estimated to be ahead of this one's (448 x 1280 x 7168 27.6 / 35.7, 192 x 5376 x 7488 43 / 58).
    const bool strip = (M <= 128 || N <= 128) && K % 8 == 0;
    bool take = narrow && (small <= 256 || (small <= 512 && kt <= (strip ? 8 : 48)));
    if (take && batch == 1 && K % 64 == 0) {
        double cost = 0, wide = 0;
        gemm_ksplit(small, K / 64, M, N, true, &cost);
        // (its estimate is 2 us on the safe side where the operands stay in the L2s: 320 x 1152 x 4928 23 for 18.7)
        if (gemm_ksplit(((M + 127) / 128) * ((N + 127) / 128), K / 64, M, N, false, &wide) > 1 && wide - (beyond_l2(M, N, K / 64) ? 0 : 2) < cost) take = false;
    }
    if (take) return nt_tile_cfg{64, 64, 32};
    nt_tile_cfg best{128, 128, 64};
    double best_cost = 0;
    for (const Cand &c : cands) {
        const int64_t programs = batch * ((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn);
        const int64_t p = (programs + 255) / 256;
        // (the range-checked kernels for overhanging tiles and ragged or unaligned operands fit two workgroups per unit like the others:
        // with one assumed for them, 27 x 1344 x 1800 x 656 ran on 256 x 256 in 181 us for 142 on 128 x 256, 30 x 856 x 1472 x 320
        // 61.8 / 51.7, 31 x 304 x 704 x 64 14.1 / 10.4, 14 x 1640 x 960 x 299 31.9 / 27.9)
        const bool full = M % c.bm == 0 && N % c.bn == 0 && K % 64 == 0;
        // (the persistent kernel staggers short programs: a program's fixed part then overlaps other units' multiplications)
        const bool staggered = c.bm == 256 && c.bn == 256 && full && programs >= 512 && kt <= 16;
        double cost = staggered ? 4.0 + (double)p * (6.0 + kt * c.step)
                                : (double)((p + c.resident - 1) / c.resident) * c.fixed + (double)p * kt * c.step;
        // (an overhanging 256 x 128 not on a tie with 128 x 128: 27 x 1184 x 448 x 114 19.8 us for 19.0)
        if (c.bm == 256 && c.bn == 128 && !full) cost *= 1.02;
        if (best_cost == 0 || cost < best_cost) { best_cost = cost; best = nt_tile_cfg{c.bm, c.bn, 64}; }
    }
    return best;
}

// Dense zero-padded copy of a convolution's input: P[n][c][h'][w'] = x[n, c, h' - ph, w' - pw] (zero outside the image),
// rows Wp = W + 2 pw long (the caller rounds nothing: the copy is as dense as a tensor).  For unit-stride convolutions
// that the implicit kernels do not take as they are (more than one column of padding, channels-last or otherwise strided
// input): on the copy they are convolutions without padding.  One thread: 8 consecutive elements of the copy, offsets
// first, the eight loads back to back (see conv_unfold_kernel).  The workspace holds total rounded up to 8 elements.
struct PadArgs {
    const uint16_t *x;
    uint16_t *P;
    int64_t xs[4];
    int64_t total;                 // N * C * Hp * Wp
    int32_t C, H, W, Hp, Wp, ph, pw;
};

__global__ __launch_bounds__(256) void conv_pad_kernel(const PadArgs g)
{
    const int64_t groups = (g.total + 7) / 8;
    const int32_t xs2 = (int32_t)g.xs[2], xs3 = (int32_t)g.xs[3];
    for (int64_t grp = (int64_t)blockIdx.x * 256 + threadIdx.x; grp < groups; grp += (int64_t)gridDim.x * 256) {
        const int64_t e0 = grp * 8;
        const int64_t plane = e0 / ((int64_t)g.Hp * g.Wp);                  // (n, c)
        const int32_t rem = (int32_t)(e0 - plane * ((int64_t)g.Hp * g.Wp));
        const int64_t n = plane / g.C, c = plane - n * g.C;
        const int64_t n2 = c + 1 == g.C ? n + 1 : n, c2 = c + 1 == g.C ? 0 : c + 1;     // the plane after it (a group may run into it)
        const int64_t base = n * g.xs[0] + c * g.xs[1], base2 = n2 * g.xs[0] + c2 * g.xs[1];
        int32_t h = rem / g.Wp, w = rem - h * g.Wp;
        int64_t off[8];
        uint32_t keep = 0;
        bool next = false;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const bool in = e0 + e < g.total && (uint32_t)(h - g.ph) < (uint32_t)g.H && (uint32_t)(w - g.pw) < (uint32_t)g.W;
            off[e] = in ? (next ? base2 : base) + (h - g.ph) * xs2 + (w - g.pw) * xs3 : 0;
            keep |= (in ? 1u : 0u) << e;
            const bool row_end = ++w == g.Wp;
            w = row_end ? 0 : w;
            h += row_end ? 1 : 0;
            const bool plane_end = h == g.Hp;
            h = plane_end ? 0 : h;
            next = next || plane_end;
        }
        uint32_t v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = g.x[off[e]];
        uint32_t o[4];
#pragma unroll
        for (int e = 0; e < 8; e += 2)
            o[e >> 1] = ((keep >> e) & 1u ? v[e] : 0u) | (((keep >> (e + 1)) & 1u ? v[e + 1] : 0u) << 16);
        const u32x4 ov{o[0], o[1], o[2], o[3]};
        __builtin_memcpy(g.P + e0, &ov, 16);
    }
}

// The same copy for a dense channels-last input (x[n][h][w][c]): a transposition.  One workgroup: 64 channels x 32
// positions of one padded row, read along c (128 contiguous bytes per wavefront), turned in LDS, written along w.
// (conv_pad_kernel reads such an input with its lanes C elements apart: 70 us for 51 MB.)
__global__ __launch_bounds__(256) void conv_pad_nhwc_kernel(const PadArgs g)
{
    __shared__ uint16_t tile[32][66];
    const int32_t ctiles = (g.C + 63) / 64;
    const int32_t n = blockIdx.z / ctiles, c0 = (blockIdx.z - n * ctiles) * 64;
    const int32_t hp = blockIdx.y, w0 = blockIdx.x * 32, h = hp - g.ph;
    const int tid = threadIdx.x;
    {
        const int c = tid & 63, wl = tid >> 6;
        const uint16_t *row = g.x + (((int64_t)n * g.H + h) * g.W) * g.C + c0 + c;
        const bool hc_ok = (uint32_t)h < (uint32_t)g.H && c0 + c < g.C;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int32_t w = w0 + wl + 4 * i - g.pw;
            const bool in = hc_ok && (uint32_t)w < (uint32_t)g.W;
            tile[wl + 4 * i][c] = in ? row[(int64_t)w * g.C] : (uint16_t)0;
        }
    }
    __syncthreads();
    {
        const int w = tid & 31, cl = tid >> 5;
        if (w0 + w < g.Wp) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int c = cl + 8 * i;
                if (c0 + c < g.C) g.P[(((int64_t)n * g.C + c0 + c) * g.Hp + hp) * g.Wp + w0 + w] = tile[w][c];
            }
        }
    }
}

// Unfolded input of a convolution (Section 4.3: A[m, kk] = x[n, c, p sh + r - ph, q sw + s - pw], zero outside the
// image), written out for the convolutions the implicit kernels do not take (strided, widely padded, channels-last):
// U[kk][m] with m = (n, p, q) contiguous and the row pitch Mp (a multiple of 8; the surplus columns are zeros);
// x has any strides.
struct UnfoldArgs {
    const uint16_t *x;
    uint16_t *U;
    int64_t xs[4];
    int64_t M, Mp, K;
    int32_t C, H, W, R, S, P, Q, sh, sw, ph, pw, dh, dw;
};

__global__ __launch_bounds__(256) void conv_unfold_kernel(const UnfoldArgs g)
{
    // blockIdx.y: the line kk = (c, r, s), taken apart once per workgroup in scalar registers; x: groups of 8 positions.
    // Element offsets are 32-bit (the host admits inputs whose offsets stay below 2^31).
    const uint32_t kk = blockIdx.y;
    const uint32_t c = kk / (uint32_t)(g.R * g.S), rs = kk - c * (uint32_t)(g.R * g.S);
    const uint32_t r = rs / (uint32_t)g.S, sx = rs - r * (uint32_t)g.S;
    const uint16_t *xc = g.x + (int64_t)c * g.xs[1];
    const int32_t xs0 = (int32_t)g.xs[0], xs2 = (int32_t)g.xs[2], xs3 = (int32_t)g.xs[3];
    const uint32_t groups = (uint32_t)(g.Mp / 8), pq = (uint32_t)(g.P * g.Q);
    for (uint32_t grp = blockIdx.x * 256 + threadIdx.x; grp < groups; grp += gridDim.x * 256) {
        const uint32_t m0 = grp * 8;
        uint32_t n = m0 / pq;
        const uint32_t rem = m0 - n * pq;
        int32_t p = (int32_t)(rem / (uint32_t)g.Q), q = (int32_t)(rem - (uint32_t)p * (uint32_t)g.Q);
        // A group that lies in one output row and reads 8 (conv stride 1) or 16 (stride 2) consecutive elements of one
        // input row, all inside the image: one or two 16-byte loads (2-byte aligned), every second element picked for
        // stride 2.  (Input contiguous along w only.)
        if (xs3 == 1 && g.sw <= 2 && q + 8 <= g.Q && m0 + 8 <= (uint32_t)g.M) {
            const int32_t h = p * g.sh + (int32_t)r * g.dh - g.ph, col = q * g.sw + (int32_t)sx * g.dw - g.pw;
            if ((uint32_t)h < (uint32_t)g.H && col >= 0 && col + 8 * g.sw <= g.W) {
                const uint16_t *src = xc + ((int32_t)n * xs0 + h * xs2 + col);
                u32x4 a;
                __builtin_memcpy(&a, src, 16);
                if (g.sw == 2) {
                    u32x4 b;
                    __builtin_memcpy(&b, src + 8, 16);
                    a = u32x4{__builtin_amdgcn_perm(a[1], a[0], 0x05040100u), __builtin_amdgcn_perm(a[3], a[2], 0x05040100u),
                              __builtin_amdgcn_perm(b[1], b[0], 0x05040100u), __builtin_amdgcn_perm(b[3], b[2], 0x05040100u)};
                }
                __builtin_memcpy(g.U + (int64_t)kk * g.Mp + m0, &a, 16);
                continue;
            }
        }
        // Otherwise all eight offsets first (an element outside the image or past M points at element 0 and is dropped),
        // then the eight loads back to back, with no branch between them: this part is bound by the latency of its loads
        int32_t off[8];
        uint32_t keep = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int32_t h = p * g.sh + (int32_t)r * g.dh - g.ph, col = q * g.sw + (int32_t)sx * g.dw - g.pw;
            const bool in = m0 + e < (uint32_t)g.M && (uint32_t)h < (uint32_t)g.H && (uint32_t)col < (uint32_t)g.W;
            off[e] = in ? (int32_t)n * xs0 + h * xs2 + col * xs3 : 0;
            keep |= (in ? 1u : 0u) << e;
            const bool row_end = ++q == g.Q;
            q = row_end ? 0 : q;
            p += row_end ? 1 : 0;
            const bool image_end = p == g.P;
            p = image_end ? 0 : p;
            n += image_end ? 1 : 0;
        }
        uint32_t v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = xc[off[e]];
        uint32_t w[4];
#pragma unroll
        for (int e = 0; e < 8; e += 2)
            w[e >> 1] = ((keep >> e) & 1u ? v[e] : 0u) | (((keep >> (e + 1)) & 1u ? v[e + 1] : 0u) << 16);
        const u32x4 o{w[0], w[1], w[2], w[3]};
        __builtin_memcpy(g.U + (int64_t)kk * g.Mp + m0, &o, 16);
    }
}

// k split of a GEMM, second step: C[m, n] = act(alpha * sum_i ws[i][m][n] + beta * D[m, n]) with the slices added in slice
// order (reproducible), converted once.  C and D are plain strided matrices.
__global__ __launch_bounds__(256) void splitk_sum_kernel(const float *ws, int ksplit, int64_t M, int64_t N, void *C, int64_t scm, int64_t scn, int out_dtype,
                                                         const void *D, int64_t sdm, int64_t sdn, float alpha, float beta, int act)
{
    const ActParams ap = act_params(act);
    const int64_t total = M * N;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
        // (eight slices' loads in flight, added in slice order: one after the other they took 4 us for 8 slices of 16 x 4096)
        float sum = 0.f;
        for (int j = 0; j < ksplit; j += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = j + u < ksplit ? ws[(j + u) * total + i] : 0.f;
#pragma unroll
            for (int u = 0; u < 8; ++u) sum += v[u];
        }
        const int64_t m = i / N, n = i - m * N;
        const float x = combine(sum, D ? load_as_f32(D, m * sdm + n * sdn, out_dtype) : 0.f, alpha, beta);
        store_out(C, m * scm + n * scn, act ? activate(x, ap) : x, out_dtype);
    }
}

bool tile_is_built(nt_tile_cfg cfg)
{
    for (const TileEntry &t : kTiles)
        if (t.bm == cfg.bm && t.bn == cfg.bn && t.bk == cfg.bk) return true;
    return false;
}

// The dense convolution that the convolution kernels handle: contiguous NCHW input, conv stride 1, at
// most one element of left / right padding, a filter whose (c, r, s) are contiguous, an output with
// contiguous (p, q).  Everything else runs on the operand-map kernel.
static bool conv_tap_ok(const GemmLaunch &g, const ConvArgs &c, size_t *repack_bytes);

static bool match_conv(const GemmLaunch &g, ConvArgs *a)
{
    const ConvHint &h = g.conv;
    if (!h.valid || g.batch != 1 || g.tile.bm != 256 || g.tile.bk != 64 || (g.tile.bn != 128 && g.tile.bn != 256)) return false;
    if (h.sh != 1 || h.sw != 1 || h.dh != 1 || h.dw != 1 || h.ph < 0 || h.pw < 0 || h.pw > 1 || h.R > 31 || h.S > 31 || h.P <= 0 || h.Q <= 0) return false;
    if (h.xs[3] != 1 || h.xs[2] != h.W || h.xs[1] != h.H * h.W || h.xs[0] != h.C * h.H * h.W) return false;
    // filter rows contiguous in (c, r, s), or in (r, s, c) (a channels-last filter, which is the tap-major kernel's own order)
    const bool krsc = h.ws[1] == 1 && h.ws[3] == h.C && h.ws[2] == h.S * h.C && (h.C > 1 || h.R * h.S == 1);
    if (!krsc && (h.ws[3] != 1 || h.ws[2] != h.S || h.ws[1] != h.R * h.S)) return false;
    if (h.ws[0] <= 0 || h.ws[0] >= (1 << 22)) return false;
    if (h.ys[3] != 1 || h.ys[2] != h.Q) return false;
    // the kernel numbers the output positions with the row pitch rounded up to a multiple of 8
    const int64_t Q8 = (h.Q + 7) / 8 * 8;
    const int64_t CRS = h.C * h.R * h.S, NPQ = h.N * h.P * Q8, numel = h.N * h.C * h.H * h.W;
    if (numel >= (1LL << 31) || numel < 8 || NPQ >= (1LL << 31) - 256 || CRS >= (1 << 16) - 128 || CRS < 8) return false;   // (the filter loader needs K >= 8)
    a->X = (const uint16_t *)g.A;
    a->Wt = (const uint16_t *)g.B;
    a->Y = g.C;
    a->ldb = h.ws[0];
    a->syn = h.ys[0];
    a->syf = h.ys[1];
    a->x_numel = numel;
    a->M = (int32_t)NPQ; a->N = (int32_t)g.N; a->K = (int32_t)CRS;
    a->PQ = (int32_t)(h.P * h.Q); a->Q = (int32_t)h.Q; a->H = (int32_t)h.H; a->W = (int32_t)h.W;
    a->Q8 = (int32_t)Q8; a->PQ8 = (int32_t)(h.P * Q8); a->last_e = (int32_t)((h.Q - 1) % 8);
    a->HW = (int32_t)(h.H * h.W); a->CHW = (int32_t)(h.C * h.H * h.W);
    a->RS = (int32_t)(h.R * h.S); a->S = (int32_t)h.S; a->R = (int32_t)h.R; a->ph = (int32_t)h.ph; a->pw = (int32_t)h.pw;
    a->inv_rs = h.R * h.S > 1 ? (uint32_t)((1ULL << 32) / (uint64_t)(h.R * h.S)) + 1u : 0u;
    a->inv_s = h.S > 1 ? (uint32_t)((1ULL << 32) / (uint64_t)h.S) + 1u : 0u;
    a->mt = (NPQ + 255) / 256; a->nt = g.nt; a->kt = g.kt;
    a->out_dtype = g.out_dtype;
    a->ksplit = 1; a->kt_per = (int32_t)g.kt; a->slice = 0;
    a->filter_tap_major = krsc && !(h.ws[3] == 1 && h.ws[2] == h.S && h.ws[1] == h.R * h.S) ? 1 : 0;
    if (a->filter_tap_major) {                               // (no other kernel reads that layout)
        size_t unused = 0;
        if (!conv_tap_ok(g, *a, &unused)) return false;
    }
    return true;
}

// Workspace of the k splits (convolution, skinny GEMM) and of the copies and the unfolded input of a convolution: one allocation
// per device, made by the first call on that device that needs it and kept until the process ends (never freed or moved, so work
// in flight never loses it).  It is cut into lanes, one of kSplitWsMax bytes and kSmallLanes of kSmallLane bytes for what fits
// those, so that calls on a few streams overlap as calls without workspace do.  A call holds a lane through a WorkspaceLease from
// before its first launch that touches it until after its last: the lease serialises host threads (a mutex) and streams (an event
// recorded behind the last consumer, which a call on any other stream makes its stream wait for before its own first launch), so
// calls that meet on one lane queue up instead of racing.  A stream keeps to the small lane it has used before, a new one takes
// the lane that has not been taken for the longest time.  (Two streams of (2,64,56,56)*(64,64,3,3) from two threads, us a call: 30
// on one lane, 14; alternating (4,256,14,14)*(256,256,3,3) 32 and 19.)
// Calls captured into a graph never touch those lanes or their events: a replay takes no lease, so nothing would order it against
// the calls around it.  They share an allocation of their own (kSplitWsMax bytes, made by the first that needs it); within a
// capture the event between two streams becomes an edge of the graph, and replays that overlap each other are the caller's to avoid.
// The event carries no system-scope fence: it only orders kernels of one device, and what it orders is the last consumer's reads
// before the next caller's writes (a consumer's input left the writer's caches at the launch boundary between the two).  The
// fence cost every call 2 us on the device (the paper's conv task 29.5 -> 27.6 us).
static constexpr size_t kSplitWsMax = 256u << 20, kSmallLane = 32u << 20;
static constexpr int kSmallLanes = 3;

// the capture (a number above 0) that work on the stream goes into, 0: none
static unsigned long long capture_of(hipStream_t stream)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    unsigned long long id = 0;
    if (hipStreamGetCaptureInfo(stream, &st, &id) != hipSuccess) { (void)hipGetLastError(); return ~0ull; }
    return st == hipStreamCaptureStatusNone ? 0 : id;
}

class WorkspaceLease {
public:
    WorkspaceLease() = default;
    WorkspaceLease(const WorkspaceLease &) = delete;
    WorkspaceLease &operator=(const WorkspaceLease &) = delete;
    // nullptr: more than the workspace holds, no memory, or no device -- the caller then runs without it
    void *acquire(size_t bytes, hipStream_t stream)
    {
        int dev = 0;
        if (lane_ || bytes > kSplitWsMax || hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
        Device &d = table()[dev];
        const unsigned long long capture = capture_of(stream);
        if (capture == ~0ull) return nullptr;
        if (!(capture ? ready_for_captures(d) : ready(d))) return nullptr;
        Lane *w = capture ? &d.captures : bytes <= kSmallLane ? small_lane(d, stream) : &d.lane[0];
        w->mu.lock();
        // (an event recorded in another capture says nothing about this one)
        if (w->used && w->last != stream && w->capture == capture && (!w->marked || hipStreamWaitEvent(stream, w->done, 0) != hipSuccess)) {
            (void)hipGetLastError();
            w->mu.unlock();
            return nullptr;
        }
        lane_ = w;
        stream_ = stream;
        w->capture = capture;
        return w->p;
    }
    ~WorkspaceLease()
    {
        if (!lane_) return;
        lane_->last = stream_;
        lane_->used = lane_->marked = hipEventRecord(lane_->done, stream_) == hipSuccess;
        if (!lane_->marked) {
            // without the marker a later call on another stream could not wait for this one's work: wait for it here (in a capture,
            // where there is nothing to wait for yet, such a call runs without the workspace)
            (void)hipGetLastError();
            if (lane_->capture) lane_->used = true;
            else (void)hipStreamSynchronize(stream_);
        }
        lane_->mu.unlock();
    }

private:
    // (owner and stamp -- who was given the lane last, and when -- under the device's mutex, the rest under the lane's)
    struct Lane {
        void *p = nullptr;
        hipEvent_t done = nullptr;
        hipStream_t last = nullptr, owner = nullptr;
        bool used = false, marked = false;
        uint64_t stamp = 0;
        unsigned long long capture = 0;
        std::mutex mu;
    };
    struct Device { Lane lane[1 + kSmallLanes], captures; void *p = nullptr; uint64_t clock = 0; std::mutex mu; };
    static Device *table() { static Device t[64]; return t; }

    // the device's allocation, made if need be
    static bool ready(Device &d)
    {
        std::lock_guard<std::mutex> lock(d.mu);
        if (d.p) return true;
        void *p = nullptr;
        hipEvent_t ev[1 + kSmallLanes] = {};
        bool ok = hipMalloc(&p, kSplitWsMax + kSmallLanes * kSmallLane) == hipSuccess;
        for (hipEvent_t &e : ev) ok = ok && hipEventCreateWithFlags(&e, hipEventDisableTiming | hipEventDisableSystemFence) == hipSuccess;
        if (!ok) {
            (void)hipGetLastError();
            for (hipEvent_t e : ev)
                if (e) (void)hipEventDestroy(e);
            if (p) (void)hipFree(p);
            return false;
        }
        for (int i = 0; i <= kSmallLanes; ++i) {
            d.lane[i].p = (char *)p + (i ? kSplitWsMax + (size_t)(i - 1) * kSmallLane : 0);
            d.lane[i].done = ev[i];
        }
        d.p = p;
        return true;
    }
    // ... and the captured calls', which a thread in relaxed mode may make during a capture
    static bool ready_for_captures(Device &d)
    {
        std::lock_guard<std::mutex> lock(d.mu);
        if (d.captures.p) return true;
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) { (void)hipGetLastError(); return false; }
        void *p = nullptr;
        bool ok = hipMalloc(&p, kSplitWsMax) == hipSuccess;
        ok = ok && hipEventCreateWithFlags(&d.captures.done, hipEventDisableTiming | hipEventDisableSystemFence) == hipSuccess;
        if (!ok) (void)hipGetLastError();
        if (!ok && p) (void)hipFree(p);
        (void)hipThreadExchangeStreamCaptureMode(&mode);
        if (ok) d.captures.p = p;
        return ok;
    }
    // the small lane of this stream
    static Lane *small_lane(Device &d, hipStream_t stream)
    {
        std::lock_guard<std::mutex> lock(d.mu);
        Lane *w = &d.lane[1];
        for (int i = 1; i <= kSmallLanes; ++i) {
            Lane &l = d.lane[i];
            if (l.stamp && l.owner == stream) { w = &l; break; }
            if (l.stamp < w->stamp) w = &l;
        }
        w->owner = stream;
        w->stamp = ++d.clock;
        return w;
    }
    Lane *lane_ = nullptr;
    hipStream_t stream_ = nullptr;
};

// Scratch memory for callers that cannot allocate (nt_gemm_noalloc): a fixed array in the library's device image, one copy
// per GPU, held from the moment the library is loaded on that GPU until the process ends.  Host code never uses the array's
// name as an address: the device address is looked up once per device, with that device current, and kept.
static __device__ __align__(256) unsigned char scratch[NT_NOALLOC_SCRATCH_BYTES];

nt_status static_scratch(void **ptr_out, size_t *bytes_out)
{
    static void *table[64] = {};
    static std::mutex mu;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(NT_ERR_DEVICE, std::string("hipGetDevice: ") + hipGetErrorString(e));
    if (dev < 0 || dev >= 64) return fail(NT_ERR_UNSUPPORTED, "device index beyond 63");
    std::lock_guard<std::mutex> lock(mu);
    if (!table[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) { (void)hipGetLastError(); return fail(NT_ERR_DEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e)); }
        table[dev] = p;
    }
    *ptr_out = table[dev];
    *bytes_out = sizeof(scratch);
    return NT_OK;
}

// Estimated time (us) of a dense unit-stride convolution -- an implicit GEMM of M positions x N filters x kt k tiles -- on
// tiles of 256 positions x bn filters with `per` k tiles per program (ks = ceil(kt / per) programs per output tile).  A
// program costs a fixed part plus its 32-k slices (0.8 us each on the 256-filter tile, 1.15 on the narrower ones, which do
// half the work or less per slice: their loader, not the matrix pipe, sets the pace; the 256-filter tile's fixed part
// includes the copy of the filter); programs run in rounds of one per compute unit (two for the narrower tiles, which are
// co-resident); a split adds a second launch and the partial tiles' trip through memory.  Fits (us, measured):
// (256,512,7,7)*(512,512,3,3) 172 on 128-filter tiles, 111-119 on 256-filter tiles split in two; (32,512,14,14)*(512,512,3,3)
// 99 / 73; (8,256,56,56)*(256,256,3,3) 73 / 60; (16,256,28,28)*(256,256,3,3) 58.5 / 57.8; (32,256,14,14)*(1024,256,1,1) 18 / 31.
static double conv_cost(int64_t M, int64_t N, int64_t kt, int bn, int64_t per)
{
    const int64_t ks = (kt + per - 1) / per;
    const int64_t programs = ((M + 255) / 256) * ((N + bn - 1) / bn) * ks;
    const int64_t slots = bn == 256 ? 256 : 512;
    const double fixed = bn == 256 ? 14.0 : 7.0, slice = bn == 256 ? 0.8 : 1.15;
    double c = (double)((programs + slots - 1) / slots) * (fixed + 2.0 * (double)per * slice);
    if (ks > 1) c += 6.0 + (double)ks * (double)M * (double)N * 8.0 / 5.0e6;
    return c;
}

// The split of the reduction for that tile: `*kt_per` k tiles per program (none with fewer than 4), the number of parts
// returned.  Small grids (fewer than 48 tiles of 256 x 256): enough parts for about one program per compute unit
// (measured on 13 shapes from 1 to 112 programs and 8 to 72 k tiles: the split run is faster in every one, e.g.
// (8,64,14,14) * (64,64,3,3) 26 -> 21 us, (4,256,14,14) * (256,256,3,3) 78 -> 23 us).  Larger ones: the cheapest by the
// estimate above, which knows about whole rounds (5 parts of 56 tiles are 280 programs and cost two rounds, 4 parts one).
static bool conv_small(int64_t M, int64_t N) { return ((M + 255) / 256) * ((N + 255) / 256) < 48; }
static int conv_ksplit(int64_t M, int64_t N, int64_t kt, int bn, int32_t *kt_per, double *cost_out = nullptr)
{
    *kt_per = (int32_t)kt;
    if (conv_small(M, N)) {
        const int64_t programs = ((M + 255) / 256) * ((N + bn - 1) / bn);
        if (programs >= 128 || kt < 8) return 1;
        const int64_t want = std::min<int64_t>((256 + programs / 2) / programs, kt / 4);
        if (want < 2) return 1;
        const int64_t per = (kt + want - 1) / want;
        *kt_per = (int32_t)per;
        return (int)((kt + per - 1) / per);
    }
    int64_t best_per = kt;
    double best = conv_cost(M, N, kt, bn, kt);
    for (int64_t ks = 2; ks <= 64; ++ks) {
        const int64_t per = (kt + ks - 1) / ks;
        if (per < 4 || (double)ks * (double)M * (double)N * 4.0 > (double)kSplitWsMax) break;
        if ((kt + per - 1) / per != ks) continue;                              // (that many parts come out one fewer)
        const double c = conv_cost(M, N, kt, bn, per);
        if (c < best) { best = c; best_per = per; }
    }
    *kt_per = (int32_t)best_per;
    if (cost_out) *cost_out = best;
    return (int)((kt + best_per - 1) / best_per);
}

// The tile of filters for such a convolution.  Small grids: 256 filters per program when 256 would not leave half the
// compute units without a program, else 128; larger ones: by the estimate, each tile with its best split.
nt_tile_cfg pick_conv_tile(int64_t M, int64_t N, int64_t K)
{
    if (N <= 128) return nt_tile_cfg{256, 128, 64};
    if (conv_small(M, N)) return nt_tile_cfg{256, 128, 64};
    const int64_t kt = (K + 63) / 64;
    int32_t per = 0;
    double c256 = 0, c128 = 0;
    conv_ksplit(M, N, kt, 256, &per, &c256);
    conv_ksplit(M, N, kt, 128, &per, &c128);
    return c256 <= c128 ? nt_tile_cfg{256, 256, 64} : nt_tile_cfg{256, 128, 64};
}

// A map is "plain" when it is a strided matrix without bounds checks beyond rows / cols.
static bool plain(const OperandMap &m) { return m.nrd == 1 && m.ncd == 1 && m.nchk == 0; }

// The same for a GEMM with few output tiles and a long reduction (a skinny product): the split is run as a batched
// product over parts of K: equal ones, so that only a number of parts that divides the k tiles evenly is taken, or (`uneven`, the
// range-checked kernels) the last one shorter, and the cheapest number of parts is (at least 8 k tiles
// each).  The uneven ones not beyond what the entry point with its own scratch memory holds: it then sums in the same order as the
// one with the workspace, and refuses none.  Two dependent launches and the trip of the partial tiles through memory have their
// price: the split is taken when an estimate of it (the launches, a program's k tiles with its compute unit to itself, the slices
// written and read at 3 TB/s) beats the estimate of the single launch.  `small`: the 64 x 64 tile (us: 3.5 + 0.24 per 64-k tile, the split's
// launches 6), else 128 x 128 (7 + 0.37 and 12).
// Measured: 1024 x 1024 x 1024 on 128 x 128 11 us unsplit against 19 split; on 64 x 64, unsplit / split: 256 x 256 x 2048 10.6 /
// 8.0, x 8192 32.9 / 9.8, 512 x 512 x 4096 18.7 / 12.7, 16 x 1024 x 4096 20.0 / 8.0 (on 128 x 128, split: 10.3, 12.1, 13.5, 10.8).
// *cost_out: the estimate of the way taken.
static int gemm_ksplit(int64_t programs, int64_t kt, int64_t M, int64_t N, bool small, double *cost_out, bool uneven)
{
    // (operands beyond the L2s come from memory: 72 x 7136 x 3712 0.32 per k tile, 704 x 1408 x 8640 0.33, 192 x 5376 x 7488 0.46)
    const double step = small ? (beyond_l2(M, N, kt) ? 0.36 : 0.24) : 0.37, once = small ? 3.5 : 7.0, twice = small ? 6.0 : 12.0;
    const double single = once + step * (double)kt;
    *cost_out = single;
    if (programs >= (small ? 192 : 128) || kt < 32) return 1;
    // (about a program per unit; of the 64 x 64 tile's no more than that: a few units with two of them set the pace)
    const int64_t want = std::min<int64_t>(small ? 256 / programs : (256 + programs / 2) / programs, kt / 8);
    if (uneven) {
        int best = 1;
        for (int64_t d = 2; d <= want; ++d) {
            const int64_t per = (kt + d - 1) / d;
            if ((kt + per - 1) / per != d || d * M * N * 4 > (int64_t)NT_NOALLOC_SCRATCH_BYTES) continue;
            const double split = twice + step * (double)per + (double)d * (double)M * (double)N * 8.0 / 3.0e6;
            if (split < *cost_out) { *cost_out = split; best = (int)d; }
        }
        return best;
    }
    for (int64_t d = want; d >= 2; --d) {
        if (kt % d) continue;
        const double split = twice + step * (double)kt / (double)d + (double)d * (double)M * (double)N * 8.0 / 3.0e6;
        if (split >= single) return 1;
        *cost_out = split;
        return (int)d;
    }
    return 1;
}

static thread_local int t_k_split = 1;
int last_k_split() { return t_k_split; }
static thread_local nt_conv_plan t_conv_plan;
const nt_conv_plan &last_conv_plan() { return t_conv_plan; }

// Where a k split's fp32 partial tiles go: the region the caller of this launch has set aside (a route that already holds
// the workspace, or an entry point that brings its own scratch memory), else the library's workspace through `lease`.
// nullptr: none (then the launch runs unsplit); *status is set when the caller's region is too small and must be.
static float *split_region(const GemmLaunch &g, size_t bytes, WorkspaceLease &lease, nt_status *status)
{
    *status = NT_OK;
    if (g.ws_given) {
        if (bytes <= g.ws_given_bytes) return g.ws_given;
        if (g.ws_strict)
            *status = fail(NT_ERR_UNSUPPORTED, "this product's k split needs " + std::to_string(bytes) + " bytes of scratch memory, more than the " +
                                                   std::to_string(g.ws_given_bytes) + " this entry point has");
        return nullptr;
    }
    if (g.no_workspace) return nullptr;
    return (float *)lease.acquire(bytes, (hipStream_t)g.stream);
}

// operands that can stream straight into LDS: whole 32-k slices, 16-byte aligned filter rows, 32-bit byte offsets
static bool conv_direct_ok(const GemmLaunch &g, const ConvArgs &c)
{
    return c.K % 32 == 0 && c.ldb % 8 == 0 && (reinterpret_cast<uintptr_t>(c.Wt) & 15) == 0 && c.R <= 8 && c.S <= 8 &&
           c.x_numel < (1LL << 30) && ((int64_t)(c.N - 1) * c.ldb + c.K) < (1LL << 30) &&
           ((g.conv.N - 1) * c.syn + (int64_t)(c.N - 1) * c.syf + c.PQ) < (1LL << 29);   // (output offsets: 31 bits of bytes)
}

// ... and that the kernel which walks the reduction tap by tap takes (gemm_conv_tap.h): 256 filters per program, channels in
// whole blocks of 32, padding smaller than the image; it reads the filter from a tap-major copy of `*repack_bytes` bytes
static bool conv_tap_ok(const GemmLaunch &g, const ConvArgs &c, size_t *repack_bytes)
{
    *repack_bytes = c.filter_tap_major ? 0 : ((size_t)c.N * c.K * 2 + 255) / 256 * 256;
    // (a filter row fits the LDS of the kernel that copies it: K <= 32768; one bit per tap: R S <= 32)
    return conv_direct_ok(g, c) && g.tile.bn == 256 && c.N > 128 && g.conv.C % 32 == 0 && c.ph < c.H && c.pw < c.W && c.K <= 32768 && c.RS <= 32;
}

// workspace that route 1 asks for: the filter's tap-major copy, then the fp32 slices of the k split
static size_t conv_scratch_need(const GemmLaunch &g, const ConvArgs &c)
{
    size_t repack = 0;
    const bool tap = conv_tap_ok(g, c, &repack);
    int32_t kt_per = 0;
    const int ks = conv_ksplit(c.M, c.N, c.kt, g.tile.bn, &kt_per);
    return (tap ? repack : 0) + (ks > 1 ? (size_t)ks * g.conv.N * c.N * c.PQ * 4 : 0);
}

// ---- route 1: the dense unit-stride convolution on the implicit-GEMM kernels (with the k split for small grids)
static nt_status route_conv_implicit(const GemmLaunch &g, const ConvArgs &c, int *path_out)
{
    const nt_tile_cfg t = g.tile;
    if (path_out) *path_out = PATH_CONV;
    const bool edge_b = (g.N % t.bn) || (g.K % t.bk);
    hipStream_t s = (hipStream_t)g.stream;
    int32_t kt_per = 0;
    const int ksplit = g.trace.out ? 1 : conv_ksplit(c.M, c.N, c.kt, t.bn, &kt_per);
    const int64_t slice = g.conv.N * (int64_t)c.N * c.PQ;
    const bool direct = conv_direct_ok(g, c);
    size_t repack_bytes = 0;
    bool tap = conv_tap_ok(g, c, &repack_bytes);
    const size_t split_bytes = ksplit > 1 ? (size_t)ksplit * slice * 4 : 0;
    // one piece of workspace: the filter's copy, then the split's slices.  None to be had (too large, no memory, a caller
    // who holds the workspace and has set aside less): the copy is given up first (the kernel in the arrangement's k
    // order needs none), then the split.
    WorkspaceLease lease;
    char *region = nullptr;
    if ((tap && repack_bytes) || ksplit > 1) {
        nt_status st;
        region = (char *)split_region(g, (tap ? repack_bytes : 0) + split_bytes, lease, &st);
        if (!region && tap && !c.filter_tap_major) {
            tap = false;
            if (ksplit > 1) region = (char *)split_region(g, split_bytes, lease, &st);
        }
        if (st != NT_OK) return st;
    }
    uint16_t *wt_tap = tap && repack_bytes ? (uint16_t *)region : nullptr;
    float *ws = region && ksplit > 1 ? (float *)(region + (tap ? repack_bytes : 0)) : nullptr;
    if (direct && path_out) *path_out = tap ? PATH_CONV_TAP : PATH_CONV_DIRECT;
    const bool bf16 = g.in_dtype == NT_BF16;
    ConvArgs base = c;
    int tap_rows = 256;
    if (tap) {
        if (wt_tap) {
            const nt_status st = launch_conv_repack_filter(c.Wt, c.ldb, wt_tap, c.N, (int32_t)g.conv.C, c.RS, s);
            if (st != NT_OK) return st;
            base.Wt = wt_tap;
            base.ldb = c.K;
        }
        // Tile heights: the kernel is built for a first height of h = 8 or 7 blocks of 32 positions and a second of h - 1.
        // Whole rounds of programs (one per compute unit) cost their length, h blocks plus a fixed part; ra rounds of the
        // first height, then as many of the second as the remaining positions need: the cheapest (h, ra).  With a k split
        // (small grids) one height only.
        const int64_t units = 256, blocks = ((int64_t)c.M + 31) / 32;
        const int64_t per_round = units / (c.nt * ksplit) > 0 ? units / (c.nt * ksplit) : 1;      // tiles of positions per round
        const double fixed = 1.5;
        double best = 0;
        int64_t best_a = 0, best_mt = 0;
        auto consider = [&](int h, int64_t mt_a) {
            const int64_t left = blocks - mt_a * h > 0 ? blocks - mt_a * h : 0;
            const int64_t mt_b = (left + h - 2) / (h - 1);
            const int64_t ra = (mt_a * c.nt * ksplit + units - 1) / units, rb = (mt_b * c.nt * ksplit + units - 1) / units;
            const double cost = (double)ra * (h + fixed) + (double)rb * (h - 1 + fixed);
            if (best == 0 || cost < best) { best = cost; tap_rows = 32 * h; best_a = mt_a; best_mt = mt_a + mt_b; }
        };
        for (int h = 8; h >= 7; --h) {
            const int64_t all_a = (blocks + h - 1) / h;                        // tiles if every tile had the first height
            consider(h, 0);
            if (ksplit == 1)
                for (int64_t mt_a = per_round; mt_a < all_a; mt_a += per_round) consider(h, mt_a);
            consider(h, all_a);
        }
        base.mt_a = (int32_t)best_a;
        base.mt = best_mt;
    }
    if (g.trace.out) {
        if (!direct) return fail(NT_ERR_UNSUPPORTED, "this convolution does not run on the kernels that stream their operands into LDS");
        const int bn = c.N <= 64 ? 64 : (c.N <= 128 ? 128 : t.bn);
        // (positions per program: the traced program's own height)
        const int64_t rows = g.trace.operand == 0 ? (tap ? (g.trace.program < base.mt_a * c.nt ? tap_rows : tap_rows - 32) : 256) : bn;
        if ((size_t)rows * 32 > g.trace.capacity) return fail(NT_ERR_BUFFER_TOO_SMALL, "trace buffer smaller than the slice");
        if (g.trace.program < 0 || g.trace.program >= base.mt * c.nt) return fail(NT_ERR_INVALID_ARG, "program_id outside the grid");
        if (g.trace.slice < 0 || g.trace.slice >= c.K / 32) return fail(NT_ERR_INVALID_ARG, "slice outside the reduction");
        base.trace_out = g.trace.out; base.trace_program = g.trace.program; base.trace_slice = g.trace.slice; base.trace_operand = g.trace.operand;
        return tap ? launch_conv_tap_trace(base, tap_rows, s) : launch_conv_direct_trace(base, bn, s);
    }
    auto launch = [&](const ConvArgs &ca, int64_t nwg) {
        if (tap) return launch_conv_tap(ca, tap_rows, bf16, nwg, s);
        // (one column of tiles with few filters: the same grid is run by the kernel built for 64 or 128 filters per
        // program, which spends a quarter or half of the MFMAs)
        const int bn = ca.N <= 64 && direct ? 64 : (ca.N <= 128 ? 128 : t.bn);
        return direct ? launch_conv_direct(ca, bn, bf16, nwg, s) : launch_conv(ca, bn, bf16, edge_b || (ca.N % bn) != 0, nwg, s);
    };
    if (!ws) return launch(base, base.mt * c.nt);
    t_k_split = ksplit;
    ConvArgs part = base;
    part.Y = ws; part.syn = (int64_t)c.N * c.PQ; part.syf = c.PQ; part.out_dtype = NT_F32;
    part.ksplit = ksplit; part.kt_per = kt_per; part.slice = slice;
    const nt_status st = launch(part, base.mt * c.nt * ksplit);
    if (st != NT_OK) return st;
    return launch_conv_ws_sum(ws, ksplit, slice, c.Y, (int64_t)c.N * c.PQ, c.PQ, c.syn, c.syf, c.out_dtype, s);
}

static bool conv_is_bare(const GemmLaunch &g)        // a convolution and nothing else: library tile, no epilogue terms, free to use the workspace
{
    return g.conv.valid && !g.user_tile && !g.no_workspace && !g.ws_given && g.batch == 1 && !g.has_d && g.alpha == 1.f && g.act == 0;
}

// a dense row-major matrix as an operand map
static OperandMap matrix_map(int64_t rows, int64_t cols, int64_t row_pitch)
{
    OperandMap m{};
    m.rows = rows; m.cols = cols; m.base = 0; m.nrd = 1; m.ncd = 1; m.nchk = 0;
    m.rrad[0] = rows; m.crad[0] = cols; m.roff[0] = row_pitch; m.coff[0] = 1;
    return m;
}

// Y[n] (filters x positions) = W (filters x K) . U[n] (K x positions, row pitch `pitch`, image n at U + n * image) on the matrix kernels
static GemmLaunch per_image_product(const GemmLaunch &g, const void *U, int64_t K, int64_t pitch, int64_t image)
{
    const ConvHint &h = g.conv;
    const int64_t PQ = h.P * h.Q;
    GemmLaunch u{};
    u.A = g.B; u.B = U; u.C = g.C;
    u.ma = matrix_map(h.K, K, h.ws[0]);
    u.mb = matrix_map(K, PQ, pitch);
    u.mc = matrix_map(h.K, PQ, h.ys[1]);
    u.batch = h.N; u.sa_batch = 0; u.sb_batch = image; u.sc_batch = h.ys[0];
    u.M = h.K; u.N = PQ; u.K = K;
    u.tile = pick_gemm_tile(u.batch, u.M, u.N, u.K, true);
    u.mt = (u.M + u.tile.bm - 1) / u.tile.bm; u.nt = (u.N + u.tile.bn - 1) / u.tile.bn; u.kt = (u.K + u.tile.bk - 1) / u.tile.bk;
    u.in_dtype = g.in_dtype; u.out_dtype = g.out_dtype; u.stream = g.stream;
    u.alpha = 1.f; u.beta = 0.f; u.act = 0; u.has_d = false;
    u.no_workspace = true;                               // (the caller of this holds it, or needs none)
    return u;
}

static bool lower_plain(const GemmLaunch &g, FastArgs *out, int *alay_out, int *blay_out);
static nt_status route_matrix(const GemmLaunch &g, FastArgs a, int alay, int blay, int *path_out);

// what route 3 takes (if the workspace is to be had)
static bool conv_unfold_ok(const GemmLaunch &g)
{
    const ConvHint &h = g.conv;
    const int64_t K = h.C * h.R * h.S, Mp = (h.N * h.P * h.Q + 7) / 8 * 8;
    return conv_is_bare(g) && h.ys[3] == 1 && h.ys[2] == h.Q && h.ws[3] == 1 && h.ws[2] == h.S && h.ws[1] == h.R * h.S && h.ws[0] >= K &&
           h.ws[0] < (1 << 22) && h.N * h.C * h.H * h.W > 0 && (h.N - 1) * h.xs[0] + (h.H - 1) * h.xs[2] + (h.W - 1) * h.xs[3] < (1LL << 31) &&
           h.xs[0] >= 0 && h.xs[2] >= 0 && h.xs[3] >= 0 && h.P * h.Q >= 8 && K >= 8 && K <= 65535 && Mp < (1 << 22) && (size_t)K * Mp * 2 <= kSplitWsMax;
}

// Estimated time (us) of a convolution on the routes that copy its input or fetch the unfolded one: unit stride with many
// positions by conv_cost (0.9 of it: (32,512,14,14)*(512,512,3,3) 72 for 66, (32,256,56,56)*(256,256,3,3) 143 for 124,
// (7,448,56,56)*(114,448,3,3) 63 for 58); the others are fits (unit stride within a fifth, strided a tenth).
static double conv_copied_cost(const ConvHint &h)
{
    const int64_t M8 = h.N * h.P * ((h.Q + 7) / 8 * 8);
    const bool unit = h.sh == 1 && h.sw == 1 && h.dh == 1 && h.dw == 1;
    if (unit && !conv_small(M8, h.K)) {
        int32_t per = 0;
        double narrow = 0, wide = 0;
        const int64_t kt = (h.C * h.R * h.S + 63) / 64;
        conv_ksplit(M8, h.K, kt, 128, &per, &narrow);
        if (h.K <= 128) return 0.9 * narrow;
        conv_ksplit(M8, h.K, kt, 256, &per, &wide);
        return 0.9 * std::min(narrow, wide);
    }
    const double gflop = 2e-9 * (double)(h.N * h.P * h.Q) * (double)(h.K * h.C * h.R * h.S);
    const double k = 1e-3 * (double)(h.C * h.R * h.S), filter = 4e-6 * (double)(h.K * h.C * h.R * h.S);
    const double input = 4e-6 * (double)(h.N * h.C) * (double)((h.H + 2 * h.ph) * (h.W + 2 * h.pw));
    if (unit) return 9.0 + 2.4 * std::min(gflop, 8.0) + 0.8 * std::max(gflop - 8.0, 0.0) + std::min(input, 10.0) + 0.28 * k + 0.73 * filter;
    return 9.3 + 1.05 * gflop + 0.43 * input + 0.31 * k + 0.77 * filter;
}

// Tile and number of parts of a channels-last convolution (F filters x M positions, `slices` 32-k slices): the cheapest by an
// estimate of its product.  A unit runs two programs at a time; a program costs a fixed part and its slices, a split the
// kernel that adds the parts and their trip through memory.  (Fits, us: 392 programs of 128 x 128 with 36 slices 27.5, 196
// with 144 44, 144 of 64 x 64 with 72 13.8, 1568 with 36 36.)
static void conv_cl_plan(int64_t F, int64_t M, int64_t slices, int *tile_out, int *parts_out)
{
    double best = 0;
    for (int tile = 64; tile <= 128; tile += 64)
        for (int64_t ks = 1; ks <= 8; ++ks) {
            const int64_t per = (slices + ks - 1) / ks;
            if (ks > 1 && (per < 4 || (slices + per - 1) / per != ks)) continue;
            const double load = std::max(1.0, (double)(((F + tile - 1) / tile) * ((M + tile - 1) / tile) * ks) / 256.0);
            const double rounds = load <= 2.0 ? 1.0 : load / 2.0;
            double c = tile == 64 ? 4.0 * rounds + (double)per * (load <= 1.0 ? 0.12 : 0.12 * std::max(2.0, load))
                                  : 6.0 * rounds + (double)per * (load <= 1.0 ? 0.24 : 0.29 * std::max(2.0, load));
            if (ks > 1) c += 4.0 + (double)ks * (double)F * (double)M * 8.0 / 3.0e6;
            if (best == 0 || c < best) { best = c; *tile_out = tile; *parts_out = (int)ks; }
        }
}

// What that route asks the workspace for: the copy (the padded image, or, one tap per axis, only the positions that are read), the
// filter's tap-major copy, the parts' sums.
struct ConvClSizes { int64_t eh, ew, Hc, Wc; size_t copy, filter, split; };
static ConvClSizes conv_cl_sizes(const ConvHint &h, bool natural, int parts)
{
    auto up = [](size_t b) { return (b + 255) / 256 * 256; };
    ConvClSizes z;
    z.eh = h.R == 1 ? h.sh : 1; z.ew = h.S == 1 ? h.sw : 1;
    z.Hc = h.R == 1 ? h.P : h.H + 2 * h.ph; z.Wc = h.S == 1 ? h.Q : h.W + 2 * h.pw;
    z.copy = up((size_t)h.N * z.Hc * z.Wc * h.C * 2);
    z.filter = natural ? up((size_t)h.K * h.C * h.R * h.S * 2) : 0;
    z.split = parts > 1 ? (size_t)parts * h.K * h.N * h.P * h.Q * 4 : 0;
    return z;
}

// Rows of positions: whole multiples of 8 (16 bytes), even, odd.
static int row_class(int64_t n) { return n % 8 == 0 ? 0 : n % 2 == 0 ? 1 : 2; }

// How many programs' time a unit spends: between their mean number per unit and the most (`one`: of which a unit holds one at a time).
static double unit_programs(int64_t programs, bool one)
{
    const double most = (double)((programs + 255) / 256);
    return one ? most : std::max(1.0, 0.5 * (most + (double)programs / 256));
}

// Estimated time (us) of a call of one tap as a product per image: a start, a program's fixed part and its k tiles (64 x 64: more where
// rows are no multiple of 16 bytes) for the programs of a unit, MB of input -- once more for every further strip of filters -- and MB of
// output by the class of an image's positions.  Fits to 1560 calls (1 to 512 images of 3 x 3 to 56 x 56, 32 to 16384 channels, 16 to
// 2048 filters), spread 4 to 9 % by tile.
static double one_tap_product_cost(const GemmLaunch &u)
{
    struct Fit { int bm, bn; double start, program, tile, unaligned, in, again, out[3]; };
    static const Fit fits[] = {{64, 64, 3.0, 0.70, 0.20, 0.05, 0.017, 0.025, {0.0, 0.02, 0.36}}, {128, 128, 3.7, 0.98, 0.49, 0.0, 0.027, 0.010, {0.11, 0.28, 0.43}},
                               {256, 128, 3.9, 1.66, 0.71, 0.0, 0.098, 0.050, {0.12, 0.23, 0.34}}, {128, 256, 3.8, 1.70, 0.74, 0.0, 0.080, 0.017, {0.10, 0.23, 0.29}},
                               {256, 256, 0.0, 10.95, 1.03, 0.0, 0.109, 0.014, {0.0, 0.34, 0.46}}};
    const int rows = row_class(u.N);
    const double share = unit_programs(u.batch * u.mt * u.nt, u.tile.bm + u.tile.bn == 512), mb = 2e-6 * (double)u.batch * (double)u.N;
    for (const Fit &f : fits)
        if (f.bm == u.tile.bm && f.bn == u.tile.bn)
            return f.start + share * (f.program + (f.tile + (rows && u.N > 64 ? f.unaligned : 0.0)) * (double)u.K / 64) +
                   mb * ((f.in + f.again * (double)(u.mt - 1)) * (double)u.K + f.out[rows] * (double)u.M);
    return 0;
}

// The same on the kernels of route 1 without a split, by their tile (128 filters, 64, 256) and the class of an output row.  Fits to 850
// calls, spread 5 to 9 %.
static double one_tap_implicit_cost(const GemmLaunch &g)
{
    const ConvHint &h = g.conv;
    const int64_t M8 = h.N * h.P * ((h.Q + 7) / 8 * 8);
    struct Fit { double start, program, tile, in, out; };
    static const Fit fits[3][3] = {{{5.3, 2.2, 0.97, 0.067, 0.071}, {7.3, 2.95, 1.25, 0.014, 0.176}, {8.5, 1.56, 1.20, 0.070, 0.715}},
                                   {{4.0, 1.7, 0.77, 0.067, 0.080}, {4.8, 2.1, 0.90, 0.052, 0.185}, {6.6, 0.0, 0.99, 0.079, 0.758}},
                                   {{7.0, 0.0, 1.40, 0.036, 0.380}, {8.4, 5.0, 1.33, 0.045, 0.657}, {5.9, 7.6, 1.45, 0.029, 0.877}}};
    const Fit &f = fits[g.tile.bn == 256 ? 2 : h.K <= 64 ? 1 : 0][row_class(h.Q)];
    const double share = unit_programs(((M8 + 255) / 256) * ((h.K + g.tile.bn - 1) / g.tile.bn), g.tile.bn == 256), mb = 2e-6 * (double)h.N * (double)(h.P * h.Q);
    return f.start + share * (f.program + f.tile * (double)h.C / 64) + mb * (f.in * (double)h.C + f.out * (double)h.K);
}

// ... and of few positions with the reduction split over `parts` programs of `per` k tiles, the sums through the workspace.  A fit to 613 calls
// (up to 16384 channels), spread 10 to 12 %.
static double one_tap_split_cost(const ConvHint &h, int parts, int64_t per)
{
    const double sums = 8e-6 * (double)parts * (double)(h.N * h.P * h.Q) * (double)h.K;
    return h.Q % 2 ? 10.9 + 1.55 * (double)per + 0.38 * sums : 11.8 + 1.2 * (double)per + (h.Q % 8 ? 0.3 : 0.2) * sums;
}

// The same call on the kernels of route 1, if they take it and -- few positions with a split, many without -- have an estimate; else 1e30.
// *workspace: whether they go through it.
static double one_tap_route_1(const GemmLaunch &g, bool *workspace)
{
    const ConvHint &h = g.conv;
    const int64_t M8 = h.N * h.P * ((h.Q + 7) / 8 * 8);
    int32_t per = 0;
    ConvArgs c{};
    const bool small = conv_small(M8, h.K);
    const int parts = conv_ksplit(M8, h.K, (h.C + 63) / 64, g.tile.bn, &per);
    if (small != (parts > 1) || !match_conv(g, &c)) return 1e30;
    *workspace = conv_scratch_need(g, c) > 0;
    return parts > 1 ? one_tap_split_cost(h, parts, per) : one_tap_implicit_cost(g);
}

// What a call of one tap costs (us) on the routes that do without gemm_conv_patch.hip.  Unit stride: the product (a fifth more: near a tie the
// reduction is shared) or the kernels of route 1.  Strided: the unfolded input -- a launch, the image it reads, a line per channel -- and the
// product on it; 700 calls, spread 6 %.  Where that is not open either, the operand-map kernel is all there is.
static double one_tap_without_patch(const GemmLaunch &g)
{
    const ConvHint &h = g.conv;
    const bool unit = h.sh == 1 && h.sw == 1;
    if (!unit && !conv_unfold_ok(g)) return 1e30;
    const double product = unit && (h.ph != 0 || h.pw != 0) ? 1e30 : one_tap_product_cost(per_image_product(g, g.A, h.C, h.P * h.Q, h.C * h.P * h.Q));
    bool workspace = false;
    return unit ? std::min(1.2 * product, one_tap_route_1(g, &workspace)) : 4.5 + 1.08 * product + 0.45e-6 * (double)h.N * (double)h.C * (double)(h.H * h.W) + 0.82e-3 * (double)h.C;
}

// ---- route 0b: one tap, unit stride, no padding, dense images: the input is the matrix already.  No copy, no rows rounded up, no
// workspace (us a call, the kernels of route 1 / here): (2,192,28,28)*(200,192,1,1) 14.2 / 9.7,
// (7,352,7,7)*(384,352,1,1) 19.5 / 10.0, (2,480,7,7)*(103,480,1,1) 18.4 / 5.7, (22,480,13,13)*(448,480,1,1) 27.8 / 9.6,
// (26,192,28,28)*(192,192,1,1) 15.2 / 8.4, (2,512,56,56)*(383,512,1,1) 16.2 / 9.8, (23,192,56,56)*(448,192,1,1) 34.4 / 33.0.
// Each image's positions are rounded up to a tile, though, which many small images pay for, and route 1's tiles of 64 filters suit a
// handful of them: (286,96,8,8)*(438,96,1,1) 12.5 / 15.3, (256,1024,7,7)*(2048,1024,1,1) 107 / 128, (184,64,56,56)*(18,64,1,1) 30.1 /
// 33.8; and its reduction is never split: (1,8192,7,7)*(64,8192,1,1) 16.2 / 30.0, (1,8192,14,14)*(128,8192,1,1) 21.0 / 38.5.  Calls stay there
// where its estimate is 2 % ahead, but for captured ones that would need the workspace: they can do without, and their replays take no lease.
static nt_status route_conv_pointwise(const GemmLaunch &g, int *path_out, bool *taken)
{
    *taken = false;
    const ConvHint &h = g.conv;
    if (!conv_is_bare(g) || g.trace.resident || h.R != 1 || h.S != 1 || h.sh != 1 || h.sw != 1 || h.ph != 0 || h.pw != 0 || h.C % 32 != 0) return NT_OK;
    if (h.xs[3] != 1 || h.xs[2] != h.W || h.xs[0] < 0 || h.ys[3] != 1 || h.ys[2] != h.Q || h.ws[1] != 1 || h.ws[0] < h.C || h.P * h.Q < 8) return NT_OK;
    if (h.N * h.P * h.Q >= (1LL << 30) || h.K >= (1LL << 22) || h.C > 32768) return NT_OK;
    GemmLaunch u = per_image_product(g, g.A, h.C, h.xs[1], h.xs[0]);
    u.trace = g.trace;
    u.trace.operand = 1 - g.trace.operand;                   // (the product's A is the filter)
    FastArgs fa{};
    int alay, blay;
    if (!lower_plain(u, &fa, &alay, &blay)) return NT_OK;
    bool workspace = false;
    if (1.02 * one_tap_route_1(g, &workspace) < one_tap_product_cost(u) && !(workspace && capture_of((hipStream_t)g.stream) != 0)) return NT_OK;
    *taken = true;
    return launch_gemm(u, path_out);                         // (more images than one launch holds go out in several)
}

// ---- route 0: on a channels-last copy of the input (gemm_conv_cl.hip), the filter's tap-major copy beside it: convolutions
// with channels in whole blocks of 32 that are
//   strided or dilated, with more than one tap (the unfolded input, route 3, is then several times the copy: 62.0 -> 39.2 us
//   for (32,128,56,56)*(256,128,3,3) stride 2, 100 -> 50 for (16,320,27,27)*(334,320,5,5); with one tap it is no larger, and
//   route 3's wide tiles win, 30.1 against 34.1 for (32,256,56,56)*(512,256,1,1)), or
//   of unit stride with few positions (conv_small): the kernels of route 1 compute rows of 8 positions, 12 of 16 for an
//   output row of 12, and spend more on a program's start than on its few slices: (32,512,7,7)*(512,512,3,3) 48 -> 31 us,
//   (3,224,13,13)*(256,224,3,3) 21.8 -> 13.6, (8,64,14,14)*(64,64,3,3) 16.7 -> 10.3; with many, the wider tiles of route 1
//   win, 123 against 170 for (32,256,56,56)*(256,256,3,3).  The reduction is split into as many parts as there.
static nt_status route_conv_channels_last(const GemmLaunch &g, int *path_out, bool *taken)
{
    *taken = false;
    const ConvHint &h = g.conv;
    if (!conv_is_bare(g) || h.C % 32 != 0 || h.ys[3] != 1 || h.ys[2] != h.Q || h.P <= 0 || h.Q <= 0 || h.ph < 0 || h.pw < 0) return NT_OK;
    const int64_t RS = h.R * h.S, K = h.C * RS, PQ = h.P * h.Q, M = h.N * PQ, F = h.K;
    const bool unit = h.sh == 1 && h.sw == 1 && h.dh == 1 && h.dw == 1;
    if (M >= (1LL << 30) || F >= (1LL << 22) || K > 32768 || F * K >= (1LL << 30)) return NT_OK;
    const bool natural = h.ws[3] == 1 && h.ws[2] == h.S && h.ws[1] == RS && h.ws[0] >= K;
    const bool tap_major = !natural && h.ws[1] == 1 && h.ws[3] == h.C && h.ws[2] == h.S * h.C && h.ws[0] == K && (reinterpret_cast<uintptr_t>(g.B) & 15) == 0;
    if (!natural && !tap_major) return NT_OK;
    int tile = 128, parts = 1;
    int64_t per = K / 32;
    if (unit) {
        const int64_t M8 = h.N * h.P * ((h.Q + 7) / 8 * 8);          // (positions as route 1 counts them)
        if (!conv_small(M8, F)) return NT_OK;
        int32_t kt_per = 0;
        parts = conv_ksplit(M8, F, (K + 63) / 64, g.tile.bn, &kt_per);
        per = 2 * (int64_t)kt_per;
        if (RS == 1 && parts > 1) return NT_OK;              // (a copy buys nothing there)
        // Without a split route 1 needs no workspace.  Up to 128 filters it is no slower by enough to give that up ((1,32,56,56) *
        // (32,32,3,3) 12.2 / 11.5 us, (2,32,64,64) * (128,32,3,3) 15.7 / 12.8, but 6.5 / 9.8 and 9.4 / 16 on two streams; (8,32,28,28) *
        // (256,32,3,3) 19.4 / 12.5, 10.5 / 10.5); a captured call stays independent of it, as its replays take no lease.
        ConvArgs probe{};
        if (parts == 1 && ((F <= 128 && match_conv(g, &probe)) || capture_of((hipStream_t)g.stream) != 0)) return NT_OK;
        if (((F + 127) / 128) * ((M + 127) / 128) * parts < 192) tile = 64;
    } else {
        if (RS == 1) return NT_OK;
        conv_cl_plan(F, M, K / 32, &tile, &parts);
        per = (K / 32 + parts - 1) / parts;
    }
    const ConvClSizes z = conv_cl_sizes(h, natural, parts);
    const int64_t eh = z.eh, ew = z.ew, Hc = z.Hc, Wc = z.Wc;
    // (strides far beyond the filter read a fraction of a large image: the unfolded input is then the smaller copy by far.
    // (32,64,112,112) * (128,64,2,2), 51 MB, stride 8: 23.4 against 18.4; stride 4 25.7 / 25.2; (8,256,56,56) * (512,256,2,2), 13 MB,
    // stride 8: 15.7 / 22.9)
    if (!unit && h.N * Hc * Wc >= (16 << 20) / h.C && h.N * Hc * Wc >= 8 * RS * M && conv_unfold_ok(g)) return NT_OK;
    const size_t copy_bytes = z.copy, filter_bytes = z.filter, split_bytes = z.split;
    WorkspaceLease lease;
    char *region = (char *)lease.acquire(copy_bytes + filter_bytes + split_bytes, (hipStream_t)g.stream);
    if (!region) return NT_OK;
    *taken = true;
    hipStream_t s = (hipStream_t)g.stream;
    ConvClCopy c{};
    c.x = (const uint16_t *)g.A; c.P = (uint16_t *)region;
    for (int d = 0; d < 4; ++d) c.xs[d] = h.xs[d];
    c.N = (int32_t)h.N; c.C = (int32_t)h.C; c.H = (int32_t)h.H; c.W = (int32_t)h.W; c.Hc = (int32_t)Hc; c.Wc = (int32_t)Wc;
    c.ph = (int32_t)h.ph; c.pw = (int32_t)h.pw; c.eh = (int32_t)eh; c.ew = (int32_t)ew;
    c.w = natural ? (const uint16_t *)g.B : nullptr;
    c.Wt = (uint16_t *)(region + copy_bytes);
    c.ldb = h.ws[0]; c.F = (int32_t)F; c.RS = (int32_t)RS;
    nt_status st = launch_conv_cl_copy(c, s);
    if (st != NT_OK) return st;
    ConvClArgs a{};
    a.P = c.P; a.Wt = natural ? c.Wt : (const uint16_t *)g.B; a.Y = g.C;
    a.syn = h.ys[0]; a.syf = h.ys[1];
    a.F = (int32_t)F; a.M = (int32_t)M; a.C = (int32_t)h.C; a.K = (int32_t)K;
    a.PQ = (int32_t)PQ; a.Q = (int32_t)h.Q; a.Hc = (int32_t)Hc; a.Wc = (int32_t)Wc;
    a.S = (int32_t)h.S; a.sp = (int32_t)(h.sh / eh); a.sq = (int32_t)(h.sw / ew); a.dh = (int32_t)h.dh; a.dw = (int32_t)h.dw;
    a.mt = (int32_t)((F + tile - 1) / tile); a.nt = (int32_t)((M + tile - 1) / tile);
    a.ksplit = parts; a.per = (int32_t)per;
    a.ws = (float *)(region + copy_bytes + filter_bytes);
    a.out_dtype = g.out_dtype;
    if (path_out) *path_out = PATH_CONV_CL;
    if (g.trace.out) {
        if ((size_t)tile * 32 > g.trace.capacity) return fail(NT_ERR_BUFFER_TOO_SMALL, "trace buffer smaller than the slice");
        if (g.trace.program < 0 || g.trace.program >= (int64_t)a.mt * a.nt) return fail(NT_ERR_INVALID_ARG, "program_id outside the grid");
        if (g.trace.slice < 0 || g.trace.slice >= K / 32) return fail(NT_ERR_INVALID_ARG, "slice outside the reduction");
        a.trace_out = g.trace.out; a.trace_program = g.trace.program; a.trace_slice = g.trace.slice; a.trace_operand = g.trace.operand;
        return launch_conv_cl_trace(a, tile, s);
    }
    t_k_split = parts;
    return launch_conv_cl(a, tile, g.in_dtype == NT_BF16, s);
}

// ---- route 2: a unit-stride convolution that the implicit kernels do not take as it is (more than one column of padding, a
// channels-last or otherwise strided input): on a dense zero-padded copy of its input, made once in the workspace (the
// input's size, not C R S times it), it is a dense convolution without padding.  *taken = false: not this route.
// the convolution on the copy, and the copy's bytes; false: not this route's
static bool conv_on_padded_copy(const GemmLaunch &g, GemmLaunch *g2, ConvArgs *probe, size_t *bytes)
{
    const ConvHint &h = g.conv;
    if (!(conv_is_bare(g) && h.sh == 1 && h.sw == 1 && h.dh == 1 && h.dw == 1 && h.ph >= 0 && h.pw >= 0 && h.xs[0] >= 0 && h.xs[1] >= 0 && h.xs[2] >= 0 && h.xs[3] >= 0 &&
          (h.H - 1) * h.xs[2] + (h.W - 1) * h.xs[3] < (1LL << 31)))
        return false;
    const int64_t Hp = h.H + 2 * h.ph, Wp = h.W + 2 * h.pw, total = h.N * h.C * Hp * Wp;
    *g2 = g;
    g2->conv.H = Hp; g2->conv.W = Wp; g2->conv.ph = 0; g2->conv.pw = 0;
    g2->conv.xs[3] = 1; g2->conv.xs[2] = Wp; g2->conv.xs[1] = Hp * Wp; g2->conv.xs[0] = h.C * Hp * Wp;
    g2->no_workspace = true;                             // (this route holds the workspace)
    *bytes = ((size_t)((total + 7) / 8 * 8) * 2 + 255) / 256 * 256;
    return Hp * Wp >= 8 && total < (1LL << 31) && match_conv(*g2, probe);
}

static nt_status route_conv_padded_copy(const GemmLaunch &g, int *path_out, bool *taken)
{
    *taken = false;
    const ConvHint &h = g.conv;
    GemmLaunch g2;
    ConvArgs probe{};
    size_t bytes = 0;
    if (!conv_on_padded_copy(g, &g2, &probe, &bytes)) return NT_OK;
    const int64_t Hp = g2.conv.H, Wp = g2.conv.W, total = h.N * h.C * Hp * Wp;
    // the copy and, behind it, what the convolution on it will ask for (the filter's tap-major copy, the k split's slices)
    size_t split_bytes = conv_scratch_need(g2, probe);
    if (bytes + split_bytes > kSplitWsMax) split_bytes = 0;
    WorkspaceLease lease;
    uint16_t *P = (uint16_t *)lease.acquire(bytes + split_bytes, (hipStream_t)g.stream);
    if (!P) return NT_OK;
    *taken = true;
    if (split_bytes) { g2.ws_given = (float *)((char *)P + bytes); g2.ws_given_bytes = split_bytes; }
    PadArgs pa{};
    pa.x = (const uint16_t *)g.A; pa.P = P;
    for (int d = 0; d < 4; ++d) pa.xs[d] = h.xs[d];
    pa.total = total;
    pa.C = (int32_t)h.C; pa.H = (int32_t)h.H; pa.W = (int32_t)h.W; pa.Hp = (int32_t)Hp; pa.Wp = (int32_t)Wp;
    pa.ph = (int32_t)h.ph; pa.pw = (int32_t)h.pw;
    const bool nhwc = h.xs[1] == 1 && h.xs[3] == h.C && h.xs[2] == h.W * h.C && h.xs[0] == h.H * h.W * h.C &&
                      Hp <= 65535 && h.N * ((h.C + 63) / 64) <= 65535;
    if (nhwc) {
        hipLaunchKernelGGL(conv_pad_nhwc_kernel, dim3((unsigned)((Wp + 31) / 32), (unsigned)Hp, (unsigned)(h.N * ((h.C + 63) / 64))), dim3(256), 0,
                           (hipStream_t)g.stream, pa);
    } else {
        const int64_t blocks = std::min<int64_t>(((total + 7) / 8 + 255) / 256, 1 << 20);
        hipLaunchKernelGGL(conv_pad_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)g.stream, pa);
    }
    { const nt_status lst = check_launch("conv_pad_kernel"); if (lst != NT_OK) return lst; }
    g2.A = P;
    return launch_gemm(g2, path_out);
}

// ---- route 3: any other convolution on the library's own tile: the unfolded input is written out once (if it fits the
// workspace) and the product runs per image on the MFMA kernels, Y[n] (filters x positions) = W (filters x CRS) .
// U[:, n] (CRS x positions) -- far faster than gathering every element of every tile through the operand map.
static nt_status route_conv_unfold(const GemmLaunch &g, int *path_out, bool *taken)
{
    *taken = false;
    const ConvHint &h = g.conv;
    if (!conv_unfold_ok(g)) return NT_OK;
    const int64_t K = h.C * h.R * h.S, PQ = h.P * h.Q, M = h.N * PQ, Mp = (M + 7) / 8 * 8;
    WorkspaceLease lease;
    uint16_t *U = (uint16_t *)lease.acquire((size_t)K * Mp * 2, (hipStream_t)g.stream);
    if (!U) return NT_OK;
    *taken = true;
    hipStream_t s = (hipStream_t)g.stream;
    UnfoldArgs ua{};
    ua.x = (const uint16_t *)g.A; ua.U = U;
    for (int d = 0; d < 4; ++d) ua.xs[d] = h.xs[d];
    ua.M = M; ua.Mp = Mp; ua.K = K;
    ua.C = (int32_t)h.C; ua.H = (int32_t)h.H; ua.W = (int32_t)h.W; ua.R = (int32_t)h.R; ua.S = (int32_t)h.S;
    ua.P = (int32_t)h.P; ua.Q = (int32_t)h.Q; ua.sh = (int32_t)h.sh; ua.sw = (int32_t)h.sw; ua.ph = (int32_t)h.ph; ua.pw = (int32_t)h.pw;
    ua.dh = (int32_t)h.dh; ua.dw = (int32_t)h.dw;
    const int64_t blocks = std::min<int64_t>((Mp / 8 + 255) / 256, 1 << 16);
    hipLaunchKernelGGL(conv_unfold_kernel, dim3((unsigned)blocks, (unsigned)K), dim3(256), 0, s, ua);
    { const nt_status lst = check_launch("conv_unfold_kernel"); if (lst != NT_OK) return lst; }
    const GemmLaunch u = per_image_product(g, U, K, Mp, PQ);      // (this route holds the workspace)
    const nt_status st = launch_gemm(u, nullptr);
    if (path_out) *path_out = PATH_CONV_UNFOLD;
    return st;
}

// Whether the routes below run this convolution -- natural filter, dense planes, channels in whole blocks of 32, not few positions of
// unit stride (what conv_plane_kernel is asked about) -- through the workspace.
static bool conv_below_uses_workspace(const GemmLaunch &g)
{
    const ConvHint &h = g.conv;
    GemmLaunch g2;
    ConvArgs c{};
    size_t repack = 0, bytes = 0;
    const bool unit = h.sh == 1 && h.sw == 1 && h.dh == 1 && h.dw == 1;
    if (unit) {
        if (match_conv(g, &c)) {                         // route 1: the filter's copy, given up first, and the split's slices
            const bool tap = conv_tap_ok(g, c, &repack);
            const size_t both = conv_scratch_need(g, c), split = both - (tap ? repack : 0);
            return both > 0 && (both <= kSplitWsMax || (split > 0 && split <= kSplitWsMax));
        }
        if (conv_on_padded_copy(g, &g2, &c, &bytes) && bytes <= kSplitWsMax) return true;
    } else {
        int tile = 128, parts = 1;
        conv_cl_plan(h.K, h.N * h.P * h.Q, h.C * h.R * h.S / 32, &tile, &parts);
        const ConvClSizes z = conv_cl_sizes(h, true, parts);
        if (z.copy + z.filter + z.split <= kSplitWsMax) return true;
    }
    return conv_unfold_ok(g);
}

// ---- route 0a: dense planes, channels in whole blocks of 32, the input rows under a tile resident in LDS, where one of the two
// kernels that do this is estimated to be ahead of the routes below:
//   gemm_conv_patch.hip, 9 or 25 taps: one launch straight from the caller's tensors.  Of unit stride only what does not run on
//     tiles of 256 filters (few positions, or at most 128 filters), from two blocks of channels on: one block gives a program's
//     wavefronts nothing to share, and the kernels of route 1 need no copy for up to 128 filters.  Strided with one tap too (a
//     down-sampling shortcut): two launches and the workspace cost a call through the unfolded input 11 us and more, however small.
//     Unfolded / here, us a call: (3,64,14,14)*(104,64,1,1) 11.8 / 5.3, (2,512,14,14)*(128,512,1,1) 12.4 / 7.7,
//     (14,224,56,56)*(136,224,1,1) 15.5 / 15.5; but (4,384,27,27)*(1000,384,1,1) 11.1 / 13.0, (6,608,28,28)*(271,608,1,1) 12.6 / 15.3, and
//     rows that no tap reads tell, (13,288,56,56)*(327,288,1,1) 19.7 / 39.8;
//   gemm_conv_plane.hip, six taps or more: tiles of up to 256 x 256, the filter's copy in the workspace (estimate + 20 %: what it
//     is short by on rows that are far off 16 bytes).  Not the small unit-stride ones whose reduction is split, or that need no
//     workspace otherwise: those keep to the patch or the channels-last copy.
// (programs below `first` have the first height of the plan)
static nt_status trace_fits(const LoaderTrace &t, const nt_conv_plan &p, int64_t first, int64_t programs, int64_t slices)
{
    if (t.program < 0 || t.program >= programs) return fail(NT_ERR_INVALID_ARG, "program_id outside the grid");
    if (t.slice < 0 || t.slice >= slices) return fail(NT_ERR_INVALID_ARG, "slice outside the reduction");
    const int64_t rows = t.operand != 0 ? p.filters : p.positions[t.program < first ? 0 : 1];
    if ((size_t)rows * 32 > t.capacity) return fail(NT_ERR_BUFFER_TOO_SMALL, "trace buffer smaller than the slice");
    return NT_OK;
}

// all that the choice and the plans depend on
struct ResidentKey { int64_t hint[27]; int32_t tile[4]; };      // (bm, bn, bk; filter rows aligned to 16 bytes)
struct ResidentPlan {
    ConvPatchArgs patch{};
    ConvPatchPlan patch_plan{};
    ConvPlaneArgs plane{};
    ConvPlanePlan plane_plan{};
    bool patch_ahead = false, plane_ahead = false, plane_alone = false;      // plane_alone: the routes below need no workspace
    bool patch_open = false;                                                 // (one tap) the patch can be had, if not ahead
};

static nt_status route_conv_resident(const GemmLaunch &g, int *path_out, bool *taken)
{
    *taken = false;
    const ConvHint &h = g.conv;
    if (!conv_is_bare(g) || (g.trace.out && !g.trace.resident) || h.C % 32 != 0 || h.P <= 0 || h.Q <= 0 || h.ph < 0 || h.pw < 0) return NT_OK;
    const int64_t RS = h.R * h.S, K = h.C * RS, HW = h.H * h.W, lim = 1 << 20;
    const bool unit = h.sh == 1 && h.sw == 1 && h.dh == 1 && h.dw == 1, small = conv_small(h.N * h.P * ((h.Q + 7) / 8 * 8), h.K);
    if ((RS < 6 && RS != 1) || RS > 64 || h.xs[3] != 1 || h.xs[2] != h.W || h.ys[3] != 1 || h.ys[2] != h.Q || h.xs[0] < 0 || h.xs[1] < 0) return NT_OK;
    if (h.ws[3] != 1 || h.ws[2] != h.S || h.ws[1] != RS || h.ws[0] < K) return NT_OK;
    // (32-bit byte offsets; divisions through fp32 reciprocals, exact below 2^21)
    if (HW < 8 || HW >= lim || (h.H + 2 * h.ph) * (h.W + 2 * h.pw) >= lim || h.N * (h.P * h.Q + 8) >= lim || h.K >= lim || h.K * h.ws[0] >= (1LL << 30) ||
        (h.N - 1) * h.xs[0] + (h.C - 1) * h.xs[1] + HW >= (1LL << 30)) return NT_OK;
    const bool aligned = h.ws[0] % 8 == 0 && (reinterpret_cast<uintptr_t>(g.B) & 15) == 0;
    // (one tap of unit stride: the product per image, route 0b, unless a long reduction leaves units without a program)
    int32_t kt_per = 0;
    if (RS == 1 && unit && !(small && conv_ksplit(h.N * h.P * ((h.Q + 7) / 8 * 8), h.K, (K + 63) / 64, g.tile.bn, &kt_per) > 1)) return NT_OK;
    const bool patch_ok = (RS == 9 || RS == 25 || RS == 1) && aligned && !(unit && (h.C < 64 || (h.K > 128 && !small)));
    const bool plane_ok = RS >= 6 && K <= 32768 && !(unit && small);
    // (the estimates cost the host more than the rest of the call: the last 64 answers of a thread are kept, by value; 60 KB)
    static thread_local Kept<ResidentKey, ResidentPlan> plans;
    const ResidentKey key{{h.N, h.C, h.H, h.W, h.K, h.R, h.S, h.P, h.Q, h.sh, h.sw, h.ph, h.pw, h.dh, h.dw, h.xs[0], h.xs[1], h.xs[2], h.xs[3],
                           h.ws[0], h.ws[1], h.ws[2], h.ws[3], h.ys[0], h.ys[1], h.ys[2], h.ys[3]}, {g.tile.bm, g.tile.bn, g.tile.bk, aligned ? 1 : 0}};
    const ResidentPlan *kept = plans.find(key);
    if (!kept) {
        ResidentPlan k;
        double cost = RS == 1 ? one_tap_without_patch(g) : conv_copied_cost(h), c = 0;
        if (patch_ok && conv_patch_plan(h, &k.patch, &k.patch_plan, &c)) {
            k.patch_open = RS == 1 && c < 1e30;
            if (c < cost) { k.patch_ahead = true; cost = c; }
        }
        if (plane_ok && conv_plane_plan(h, &k.plane, &k.plane_plan, &c) && 1.2 * c < cost) {
            k.plane_ahead = true;
            k.plane_alone = !conv_below_uses_workspace(g);
        }
        kept = &plans.put(key, k);
    }
    const ResidentPlan &k = *kept;
    hipStream_t s = (hipStream_t)g.stream;
    const bool bf16 = g.in_dtype == NT_BF16;
    // (a captured call that needs no workspace otherwise stays independent of it, as its replays take no lease)
    if (k.plane_ahead && !(k.plane_alone && capture_of(s) != 0)) {
        WorkspaceLease lease;
        if (uint16_t *copy = (uint16_t *)lease.acquire((size_t)h.K * K * 2, s)) {
            *taken = true;
            const nt_status st = launch_conv_plane_filter((const uint16_t *)g.B, h.ws[0], copy, (int32_t)h.K, (int32_t)h.C, (int32_t)RS, s);
            if (st != NT_OK) return st;
            ConvPlaneArgs a = k.plane;
            a.x = (const uint16_t *)g.A; a.w = copy; a.ldb = (uint32_t)K;
            a.c.Y = g.C; a.c.out_dtype = g.out_dtype;
            if (path_out) *path_out = unit ? PATH_CONV_TAP : PATH_CONV_CL;
            t_conv_plan = conv_plane_describe(k.plane_plan);
            if (g.trace.out) {
                const nt_status st = trace_fits(g.trace, t_conv_plan, k.plane_plan.mt_a * a.c.nt, a.c.mt * a.c.nt, (int64_t)a.blocks * RS);
                if (st != NT_OK) return st;
                a.c.trace_out = g.trace.out; a.c.trace_program = g.trace.program; a.c.trace_slice = g.trace.slice; a.c.trace_operand = g.trace.operand;
                return launch_conv_plane_trace(a, k.plane_plan, s);
            }
            return launch_conv_plane(a, k.plane_plan, bf16, s);
        }
    }
    // (one tap, captured: what is ahead of the patch may need the workspace)
    if (k.patch_ahead || (k.patch_open && capture_of(s) != 0)) {
        ConvPatchArgs a = k.patch;
        a.x = (const uint16_t *)g.A; a.w = (const uint16_t *)g.B; a.Y = g.C;
        a.out_dtype = g.out_dtype;
        *taken = true;
        if (path_out) *path_out = RS > 1 ? PATH_CONV_CL : unit ? PATH_CONV_DIRECT : PATH_CONV_UNFOLD;
        t_k_split = k.patch_plan.waves;
        t_conv_plan = conv_patch_describe(k.patch, k.patch_plan);
        if (g.trace.out) {
            const int64_t programs = (int64_t)a.ft * a.pt;
            const nt_status st = trace_fits(g.trace, t_conv_plan, programs, programs, (int64_t)a.blocks * RS);
            if (st != NT_OK) return st;
            a.trace_out = g.trace.out; a.trace_program = (int32_t)g.trace.program; a.trace_slice = g.trace.slice; a.trace_operand = g.trace.operand;
            return launch_conv_patch_trace(a, k.patch_plan, s);
        }
        return launch_conv_patch(a, k.patch_plan, bf16, s);
    }
    return NT_OK;
}

// Plain operands, each with unit stride along one of its axes, on a tile the MFMA kernels are built for: the arguments
// of those kernels.  false: the operand-map kernel takes the launch.
static bool lower_plain(const GemmLaunch &g, FastArgs *out, int *alay_out, int *blay_out)
{
    const nt_tile_cfg t = g.tile;
    if (!(plain(g.ma) && plain(g.mb) && plain(g.mc) && (!g.has_d || plain(g.md)) && g.kt > 0)) return false;
    FastArgs a{};
    int alay, blay;
    if (g.ma.coff[0] == 1) { alay = KCONTIG; a.lda = g.ma.roff[0]; }
    else if (g.ma.roff[0] == 1) { alay = MNCONTIG; a.lda = g.ma.coff[0]; }
    else return false;
    if (g.mb.coff[0] == 1) { blay = MNCONTIG; a.ldb = g.mb.roff[0]; }
    else if (g.mb.roff[0] == 1) { blay = KCONTIG; a.ldb = g.mb.coff[0]; }
    else return false;
    if (a.lda < 0 || a.ldb < 0 || a.lda >= (1 << 22) || a.ldb >= (1 << 22)) return false;   // 32-bit lane offsets
    // the staged loader fetches a block that straddles the ragged end of the contiguous
    // axis up to 7 elements early: that axis must be at least one block (8 elements) long
    if ((alay == MNCONTIG ? g.M : g.K) < 8 || (blay == MNCONTIG ? g.N : g.K) < 8) return false;
    const int64_t esz = g.out_dtype == NT_F32 ? 4 : 2;
    a.A = (const uint16_t *)g.A + g.ma.base;
    a.B = (const uint16_t *)g.B + g.mb.base;
    a.C = (char *)g.C + g.mc.base * esz;
    a.scm = g.mc.roff[0];
    a.scn = g.mc.coff[0];
    a.sa_batch = g.sa_batch; a.sb_batch = g.sb_batch; a.sc_batch = g.sc_batch;
    a.M = g.M; a.N = g.N; a.K = g.K;
    a.mt = g.mt; a.nt = g.nt; a.kt = (g.K + 63) / 64;
    a.out_dtype = g.out_dtype;
    a.alpha = g.alpha;
    a.beta = g.has_d ? g.beta : 0.f;
    a.act = g.act;
    // bounds of the range-checked loads (the pitches are below 2^22, so every offset inside a tile's footprint fits 32 bits)
    a.a_extent = (alay == KCONTIG ? (g.M - 1) * a.lda + g.K : (g.K - 1) * a.lda + g.M) * 2;
    a.b_extent = (blay == KCONTIG ? (g.N - 1) * a.ldb + g.K : (g.K - 1) * a.ldb + g.N) * 2;
    if (g.has_d) {
        a.D = (const char *)g.D + g.md.base * esz;
        a.sdm = g.md.roff[0];
        a.sdn = g.md.coff[0];
        a.sd_batch = g.sd_batch;
    }
    // (the 64 x 64 tile is built for the direct kernel only)
    if (t.bm < 128 && !(a.scn == 1 && (!a.D || a.sdn == 1) && (alay == KCONTIG || g.K * a.lda < (1LL << 30)) && (blay == KCONTIG || g.K * a.ldb < (1LL << 30))))
        return false;
    *out = a;
    *alay_out = alay;
    *blay_out = blay;
    return true;
}

// ---- route 4: plain matrices on the MFMA kernels (with the k split for skinny products)
// (a product of few rows with the library's own tile runs on a kernel of its own, which splits the reduction inside a program)
static nt_status route_matrix(const GemmLaunch &g, FastArgs a, int alay, int blay, int *path_out)
{
    const nt_tile_cfg t = g.tile;
    const bool bf16 = g.in_dtype == NT_BF16;
    const int64_t nwg = g.batch * g.mt * g.nt;
    hipStream_t s = (hipStream_t)g.stream;
    const bool ragged_mn = (g.M % t.bm) || (g.N % t.bn), ragged_k = (g.K % 64) != 0;
    const bool skinny = g.batch == 1 && !g.user_tile && !g.trace.out && skinny_ok(a, alay, blay);
    auto run_skinny = [&]() {
        if (path_out) *path_out = PATH_DIRECT;
        t_k_split = skinny_parts(a);
        return launch_skinny(a, bf16, s);
    };
    // Operands stored to a C (and added to a D) with unit stride along n stream straight into LDS.  Full tiles of
    // 16-byte aligned operands: plain loads.  Everything else -- tiles that overhang M or N, a ragged K, rows with
    // only the element's 2-byte alignment -- takes the same loads as range-checked buffer accesses (EDGE kernels),
    // which needs every offset inside a tile's footprint to fit 32 bits.  The range check works on the 4-byte words
    // of a load, counted from the load's own start: with an odd pitch, or an extent that is no multiple of 4 bytes,
    // the word that holds the operand's last element can end 2 bytes past it and is then dropped; the kernel is told
    // (patch) and fetches that one element by itself.  The range never extends past the operand.
    auto al16 = [](const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
    const bool out_ok = a.scn == 1 && (!a.D || a.sdn == 1);
    const bool aligned = al16(a.A) && al16(a.B) && a.lda % 8 == 0 && a.ldb % 8 == 0 && a.sa_batch % 8 == 0 && a.sb_batch % 8 == 0;
    const bool plain_direct = out_ok && aligned && !ragged_k && !ragged_mn;
    auto words_aligned = [&](int64_t ld, int64_t s_batch, int64_t extent) {      // every word of every load lies at a multiple of 4 bytes from the operand's start
        return extent % 4 == 0 && ld % 2 == 0 && s_batch % 2 == 0;
    };
    const bool direct = plain_direct || (out_ok && (alay == KCONTIG || g.K * a.lda < (1LL << 30)) && (blay == KCONTIG || g.K * a.ldb < (1LL << 30)));
    // k split: `ksplit` parts of K as the entries of a batched product into fp32 slices of the workspace.  Equal parts of whole k tiles;
    // K no multiple of 64 (range-checked loads): whole k tiles but for a shorter last part.  One launch / so (us on the device, over
    // rotating operands): weights stored [K, N] 10 x 3008 x 5408 25.2 / 11.8, 31 x 3094 x 3768 19.2 / 11.2, 1 x 7779 x 7368
    // 40.6 / 30.0; [N, K] 47 x 3176 x 4264 21.5 / 12.1, 25 x 1888 x 2083 11.3 / 8.8; square ones 446 x 448 x 6712 37.1 / 15.3,
    // 448 x 234 x 2021 14.9 / 10.1.  Not those that the kernel for few rows takes, which needs no second launch.
    double split_cost = 0;
    int ksplit = 1;
    if (g.batch == 1 && (t.bm >= 128 || !g.user_tile)) {
        if (!ragged_k) ksplit = gemm_ksplit(g.mt * g.nt, a.kt, g.M, g.N, t.bm < 128, &split_cost);
        else if (direct && !skinny && !g.trace.out) ksplit = gemm_ksplit(g.mt * g.nt, a.kt, g.M, g.N, t.bm < 128, &split_cost, true);
        // (the range-checked kernels never needed scratch memory before they were split: captured calls, whose replays take no lease
        // and which nothing orders against each other, stay without it)
        if (ragged_k && ksplit > 1 && capture_of(s) != 0) ksplit = 1;
    }
    if (skinny && (ksplit == 1 || skinny_cost(a) <= split_cost)) return run_skinny();
    if (direct && !plain_direct)
        a.patch = (words_aligned(a.lda, a.sa_batch, a.a_extent) ? 0 : 1) | (words_aligned(a.ldb, a.sb_batch, a.b_extent) ? 0 : 2);
    if (path_out) *path_out = direct ? PATH_DIRECT : PATH_FAST;
    if (g.trace.out) {
        if (!direct) return fail(NT_ERR_UNSUPPORTED, "this product does not run on the kernels that stream their operands into LDS");
        const int64_t rows = g.trace.operand == 0 ? t.bm : t.bn;
        if ((size_t)rows * 32 > g.trace.capacity) return fail(NT_ERR_BUFFER_TOO_SMALL, "trace buffer smaller than the slice");
        if (g.trace.program < 0 || g.trace.program >= nwg) return fail(NT_ERR_INVALID_ARG, "program_id outside the grid");
        if (g.trace.slice < 0 || g.trace.slice >= (g.K + 31) / 32) return fail(NT_ERR_INVALID_ARG, "slice outside the reduction");
        a.trace_out = g.trace.out; a.trace_program = g.trace.program; a.trace_slice = g.trace.slice; a.trace_operand = g.trace.operand;
        return launch_direct16_trace(a, t.bm, t.bn, alay, blay, !plain_direct, s);
    }
    typedef nt_status (*Launcher)(const FastArgs &, int, int, int64_t, hipStream_t);
    // [f16, bf16]; direct: full aligned tiles (the kernel on 16 x 16 x 32 matrix instructions: fewer accumulator bits moved per
    // flop, which on this power-managed part is clock), edge: the range-checked flavour, staged: through registers
    struct Entry { int bm, bn; Launcher direct[2], edge[2], staged[2]; };
#define NT_ENTRY(BM, BN, T) {BM, BN, {launch_direct16_##T##_f16, launch_direct16_##T##_bf16}, {launch_direct16_edge_##T##_f16, launch_direct16_edge_##T##_bf16}, \
                             {launch_fast_##T##_f16, launch_fast_##T##_bf16}}
    static const Entry table[] = {{64, 64, {launch_direct16_64x64_f16, launch_direct16_64x64_bf16}, {launch_direct16_edge_64x64_f16, launch_direct16_edge_64x64_bf16}, {nullptr, nullptr}},
                                  NT_ENTRY(128, 128, 128x128), NT_ENTRY(256, 128, 256x128), NT_ENTRY(128, 256, 128x256), NT_ENTRY(256, 256, 256x256)};
#undef NT_ENTRY
    for (const Entry &e : table) {
        if (e.bm != t.bm || e.bn != t.bn) continue;
        const Launcher launch = (direct ? (plain_direct ? e.direct : e.edge) : e.staged)[bf16 ? 1 : 0];
        WorkspaceLease lease;
        float *ws = nullptr;                                 // (none: too large, or no memory; then no split)
        if (ksplit > 1) {
            nt_status st;
            ws = split_region(g, (size_t)ksplit * g.M * g.N * 4, lease, &st);
            if (st != NT_OK) return st;
        }
        if (!ws) return skinny ? run_skinny() : launch(a, alay, blay, nwg, s);
        t_k_split = ksplit;
        FastArgs part = a;
        const int64_t per = (a.kt + ksplit - 1) / ksplit, Kp = per * 64, last = g.K - (ksplit - 1) * Kp;
        part.K = Kp; part.kt = per;
        part.sa_batch = alay == KCONTIG ? Kp : Kp * a.lda;
        part.sb_batch = blay == KCONTIG ? Kp : Kp * a.ldb;
        // (Kp is a multiple of 64: a part's words are as aligned as the whole's, and a part is as streamable)
        auto a_bytes = [&](int64_t K) { return (alay == KCONTIG ? (g.M - 1) * a.lda + K : (K - 1) * a.lda + g.M) * 2; };
        auto b_bytes = [&](int64_t K) { return (blay == KCONTIG ? (g.N - 1) * a.ldb + K : (K - 1) * a.ldb + g.N) * 2; };
        part.a_extent = a_bytes(Kp);
        part.b_extent = b_bytes(Kp);
        if (last != Kp) { part.k_parts = ksplit; part.k_short = last; part.a_short = a_bytes(last); part.b_short = b_bytes(last); }
        part.C = ws; part.scm = g.N; part.scn = 1; part.sc_batch = g.M * g.N; part.out_dtype = NT_F32;
        part.D = nullptr; part.alpha = 1.f; part.beta = 0.f; part.act = 0;
        const nt_status st = launch(part, alay, blay, nwg * ksplit, s);
        if (st != NT_OK) return st;
        const int64_t blocks = std::min<int64_t>((g.M * g.N + 255) / 256, 4096);
        hipLaunchKernelGGL(splitk_sum_kernel, dim3((unsigned)blocks), dim3(256), 0, s, ws, ksplit, g.M, g.N, a.C, a.scm, a.scn, a.out_dtype,
                           (const void *)a.D, a.sdm, a.sdn, a.alpha, a.beta, a.act);
        return check_launch("splitk_sum_kernel");
    }
    return fail(NT_ERR_UNSUPPORTED, "no fast kernel for this tile");
}

nt_status launch_gemm(const GemmLaunch &g, int *path_out)
{
    if (!g.no_workspace || g.ws_strict) t_k_split = 1;
    t_conv_plan = nt_conv_plan{};
    if (g.batch * g.mt * g.nt > 0x7fffffffLL) return fail(NT_ERR_UNSUPPORTED, "grid too large");
    if (g.batch * g.mt * g.nt > kMaxWorkgroups && !g.trace.out) {
        // more programs than one launch holds: a batch goes out in several
        const int64_t most = kMaxWorkgroups / (g.mt * g.nt);
        if (g.batch == 1 || most < 1) return fail(NT_ERR_UNSUPPORTED, "grid too large");
        const int64_t esz = g.out_dtype == NT_F32 ? 4 : 2;
        for (int64_t b0 = 0; b0 < g.batch; b0 += most) {
            GemmLaunch part = g;
            part.batch = std::min(most, g.batch - b0);
            part.A = (const char *)g.A + b0 * g.sa_batch * 2;
            part.B = (const char *)g.B + b0 * g.sb_batch * 2;
            part.C = (char *)g.C + b0 * g.sc_batch * esz;
            if (g.has_d) part.D = (const char *)g.D + b0 * g.sd_batch * esz;
            const nt_status st = launch_gemm(part, path_out);
            if (st != NT_OK) return st;
        }
        return NT_OK;
    }
    FastArgs a{};
    int alay = KCONTIG, blay = MNCONTIG;
    if (!g.trace.resident && lower_plain(g, &a, &alay, &blay)) return route_matrix(g, a, alay, blay, path_out);
    // (the library's own 64 x 64 tile is built for the direct kernel only: what that does not take, an addmm input without unit
    // stride along n say, runs as before on 128 x 128)
    if (!g.user_tile && g.tile.bm == 64 && !g.conv.valid) {
        GemmLaunch w = g;
        w.tile = nt_tile_cfg{128, 128, 64};
        w.mt = (g.M + 127) / 128; w.nt = (g.N + 127) / 128; w.kt = (g.K + 63) / 64;
        if (lower_plain(w, &a, &alay, &blay)) return route_matrix(w, a, alay, blay, path_out);
    }
    if (path_out) *path_out = PATH_GENERIC;
    bool taken = false;
    nt_status st = route_conv_resident(g, path_out, &taken);
    if (taken || st != NT_OK) return st;
    if (g.trace.resident) return fail(NT_ERR_UNSUPPORTED, "this convolution does not run on the kernels that keep the input rows in LDS");
    st = route_conv_pointwise(g, path_out, &taken);
    if (taken || st != NT_OK) return st;
    st = route_conv_channels_last(g, path_out, &taken);
    if (taken || st != NT_OK) return st;
    ConvArgs c{};
    if (!g.has_d && g.alpha == 1.f && g.act == 0 && match_conv(g, &c)) return route_conv_implicit(g, c, path_out);
    if (g.trace.out) return fail(NT_ERR_UNSUPPORTED, "this launch does not run on the kernels that stream their operands into LDS");
    st = route_conv_padded_copy(g, path_out, &taken);
    if (taken || st != NT_OK) return st;
    st = route_conv_unfold(g, path_out, &taken);
    if (taken || st != NT_OK) return st;
    return launch_generic(g);
}

nt_status launch_fill_zero(void *C, const OperandMap &mc, int64_t batch, int64_t sc_batch, int out_dtype, void *stream)
{
    const int64_t total = mc.rows * mc.cols;
    if (total <= 0 || batch <= 0) return NT_OK;
    const int64_t blocks = std::min<int64_t>((total + 255) / 256, 4096);
    hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)blocks, (unsigned)std::min<int64_t>(batch, 1024)), dim3(256), 0, (hipStream_t)stream,
                       C, mc, batch, sc_batch, out_dtype);
    return check_launch("fill_zero_kernel");
}

nt_status launch_trace(const OperandMap &m, int64_t batch_off, int64_t row0, int64_t col0, int32_t rows, int32_t cols,
                       int64_t *offsets_out, uint8_t *mask_out, void *stream)
{
    const int64_t total = (int64_t)rows * cols;
    if (total <= 0) return NT_OK;
    const int64_t blocks = std::min<int64_t>((total + 255) / 256, 1024);
    hipLaunchKernelGGL(trace_tile_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream,
                       m, batch_off, row0, col0, rows, cols, offsets_out, mask_out);
    return check_launch("trace_tile_kernel");
}

}  // namespace nt
