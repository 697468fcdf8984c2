// Convolution as an implicit GEMM over a channels-last copy of the input (Section 4.3, with the reduction walked tap by tap).
//
// With the input laid out [n][h][w][c] and padded with zeros, 32 consecutive k of the unfolded input's row m = (n, p, q) --
// one filter tap, 32 channels -- are 64 consecutive bytes, whatever the stride, the dilation and the padding: the row is a
// k-contiguous operand whose lanes have a fixed offset (the position's) and whose slices have a scalar one (the tap's and the
// channels').  So the convolution runs as the product Y[f, m] = W[f, k'] U[k', m], k' = (r, s, c), on the loop of the direct
// GEMM kernel, every load 16-byte aligned, no padding test, no fix-up, and positions of several images in one tile.
// The price is one pass over the input (read once, written once, in the workspace) instead of the unfolded input's R S.
//
// Measured, (32,128,56,56) * (256,128,3,3) stride 2 fp16: copy 13.2 us (51 MB moved), product 26.1 us (14.8 GFLOP on 392
// programs, bound by two co-resident programs' loads; kernel trace, one launch at a time), 39.1 us a call back to back; through the
// unfolded input 38 + 24 us, 63.9 a call.
#include "gemm_conv_cl.h"

#include "gemm_direct16.h"

namespace nt {

// Both copies in one launch.  The first blocks: 64 positions of the padded image x 64 channels each, read along the positions
// (16 loads in flight per thread), turned in LDS, written along the channels (16 bytes per thread).  The others: one filter
// row each, through LDS.
constexpr int kClPitch = 72;       // elements per position in LDS (64 channels + 8: 16-byte chunks stay aligned)

__global__ __launch_bounds__(256) void conv_cl_copy_kernel(const ConvClCopy g, int32_t input_blocks)
{
    extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
    const int tid = threadIdx.x;
    if ((int32_t)blockIdx.x >= input_blocks) {
        const int32_t f = blockIdx.x - input_blocks, K = g.C * g.RS;
        const uint16_t *src = g.w + (int64_t)f * g.ldb;
        uint16_t *dst = g.Wt + (int64_t)f * K;
        // (K is a multiple of 32; rows of a dense, aligned filter start on 16 bytes)
        for (int32_t i = tid * 8; i < K; i += 2048) {
            u32x4 v;
            __builtin_memcpy(&v, src + i, 16);
            *reinterpret_cast<u32x4 *>(lds + i) = v;
        }
        __syncthreads();
        for (int32_t j = tid * 8; j < K; j += 2048) {           // (eight k' of one tap: C is a multiple of 8)
            const int32_t tap = j / g.C, c = j - tap * g.C;
            uint32_t e[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) e[i] = lds[(c + i) * g.RS + tap];
            *reinterpret_cast<u32x4 *>(dst + j) = u32x4{e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
        }
        return;
    }
    const int32_t HWc = g.Hc * g.Wc, pts = (HWc + 63) / 64, cts = (g.C + 63) / 64;
    const int32_t pt = blockIdx.x % pts, rest = blockIdx.x / pts, ct = rest % cts, n = rest / cts;
    const int32_t c0 = ct * 64, pos0 = pt * 64;
    const int cn = g.C - c0 < 64 ? g.C - c0 : 64;              // 64, or 32 in the last tile
    {
        const int32_t pos = pos0 + (tid & 63), cg = (tid >> 6) * 16;
        const int32_t hc = pos / g.Wc, wc = pos - hc * g.Wc;
        const int32_t h = hc * g.eh - g.ph, w = wc * g.ew - g.pw;
        const bool in = pos < HWc && (uint32_t)h < (uint32_t)g.H && (uint32_t)w < (uint32_t)g.W && cg < cn;
        const uint16_t *src = g.x + (int64_t)n * g.xs[0] + (int64_t)(c0 + (cg < cn ? cg : 0)) * g.xs[1] + (in ? (int64_t)h * g.xs[2] + (int64_t)w * g.xs[3] : 0);
        uint32_t v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = src[i * g.xs[1]];
        uint32_t *row = reinterpret_cast<uint32_t *>(lds + (tid & 63) * kClPitch + cg);
#pragma unroll
        for (int i = 0; i < 16; i += 2) row[i >> 1] = in ? v[i] | (v[i + 1] << 16) : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int i = tid + 256 * u, p = i >> 3, ch = (i & 7) * 8;
        if (pos0 + p < HWc && ch < cn) {
            const u32x4 v = *reinterpret_cast<const u32x4 *>(lds + p * kClPitch + ch);
            *reinterpret_cast<u32x4 *>(g.P + ((int64_t)n * HWc + pos0 + p) * g.C + c0 + ch) = v;
        }
    }
}

// One program: BT filters x BT positions (and, with a k split, one part of the reduction).  The loop is gemm_direct16_kernel's.
// TRACE: see gemm_direct16_kernel.
template <int BT, bool BF16, bool TRACE = false>
__global__ __launch_bounds__(kThreads, 2) void gemm_conv_cl_kernel(const ConvClArgs g)
{
    constexpr int TM = BT / 32, TN = BT / 32, kRing = ring_of(BT, BT);
    using Tile = DirectTile16<BT, KCONTIG>;
    constexpr uint32_t T_BYTES = Tile::BYTES, B_BASE = kRing * T_BYTES;
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_m = wave >> 1, wave_n = wave & 1;
    const uint32_t mt = (uint32_t)g.mt, nt_ = (uint32_t)g.nt, grid = mt * nt_;
    const uint32_t part = TRACE ? 0u : blockIdx.x / grid;
    const uint32_t pid = TRACE ? (uint32_t)(g.trace_program % mt * nt_ + g.trace_program / mt) : program_of_workgroup_t<uint32_t>(blockIdx.x - part * grid, mt, nt_);
    const uint32_t ti = pid / nt_;
    const int32_t row0 = __builtin_amdgcn_readfirstlane((int)ti) * BT, col0 = __builtin_amdgcn_readfirstlane((int)(pid - ti * nt_)) * BT;

    const int32_t all = g.K / kSliceK;
    const int32_t first = TRACE ? g.trace_slice : __builtin_amdgcn_readfirstlane((int)part) * g.per;
    const int32_t n_slices = first + g.per < all ? g.per : all - first;

    Tile ta, tb;
    ta.init(wave, lane, 0, wave_m * (BT / 2), 0);
    tb.init(wave, lane, 0, wave_n * (BT / 2), B_BASE);
#pragma unroll
    for (int j = 0; j < Tile::PER; ++j) {
        const int row = (wave * Tile::PER + j) * 16 + (lane >> 2);
        const uint32_t c = (uint32_t)(((lane & 3) ^ Tile::swizzle(row)) * 8);
        // (rows past the last filter / position repeat it: what they give is never stored)
        const uint32_t f = (uint32_t)(row0 + row < g.F ? row0 + row : g.F - 1), m = (uint32_t)(col0 + row < g.M ? col0 + row : g.M - 1);
        ta.voff[j] = (f * (uint32_t)g.K + c) * 2u;
        const uint32_t n = m / (uint32_t)g.PQ, pq = m - n * (uint32_t)g.PQ, p = pq / (uint32_t)g.Q, q = pq - p * (uint32_t)g.Q;
        tb.voff[j] = (((n * (uint32_t)g.Hc + p * (uint32_t)g.sp) * (uint32_t)g.Wc + q * (uint32_t)g.sq) * (uint32_t)g.C + c) * 2u;
    }

    // the slice that is requested next: filter pointer, input pointer, and where it stands in (tap column, channel block)
    const int32_t CS = g.C / kSliceK;
    int32_t rq = 0, cs, ss;
    const char *pa = reinterpret_cast<const char *>(g.Wt) + (int64_t)first * (kSliceK * 2), *pb;
    {
        const int32_t tap = first / CS, r = tap / g.S;
        cs = first - tap * CS;
        ss = tap - r * g.S;
        pb = reinterpret_cast<const char *>(g.P) + (((int64_t)r * g.dh * g.Wc + (int64_t)ss * g.dw) * g.C + cs * kSliceK) * 2;
    }
    const int64_t next_tap = (int64_t)(g.dw - 1) * g.C * 2, next_row = ((int64_t)g.dh * g.Wc - (int64_t)(g.S - 1) * g.dw - 1) * g.C * 2;
    auto advance = [&]() {                                     // (slices past the last: the last again, never multiplied)
        if (++rq >= n_slices) return;                          // (all scalar)
        pa += kSliceK * 2;
        pb += kSliceK * 2;
        if (++cs == CS) {
            cs = 0;
            if (++ss == g.S) { ss = 0; pb += next_row; }
            else pb += next_tap;
        }
    };

    float4v acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[a][b][v] = 0.f;

    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
    u32x4 fa[2][TM], fb[2][TN];
    constexpr int NR = TM + TN, NM = TM * TN, ND = 2 * Tile::PER;
    auto lds_read = [&](int r, int set, uint32_t ring) {
        if (r < 1) ta.read(fa[set], smem, r, ring * T_BYTES);
        else if (r < 1 + TN) tb.read(fb[set], smem, r - 1, ring * T_BYTES);
        else ta.read(fa[set], smem, r - TN, ring * T_BYTES);
    };
    auto dma = [&](int d, uint32_t ring) {
        if (d < Tile::PER) ta.issue_one(d, pa, lds0 + ring * T_BYTES, wave);
        else tb.issue_one(d - Tile::PER, pb, lds0 + B_BASE + ring * T_BYTES, wave);
    };
    if constexpr (TRACE) {
#pragma unroll
        for (int d = 0; d < ND; ++d) dma(d, 0);
        NT_WAIT_VMCNT(0);
        __syncthreads();
        for (int e = tid; e < BT * kSliceK; e += kThreads)
            g.trace_out[e] = *reinterpret_cast<const uint16_t *>(smem + (g.trace_operand == 0 ? B_BASE : 0u) + Tile::place(e / kSliceK, e % kSliceK));
        return;
    }
    auto trip = [&](auto set_c, uint32_t rring, uint32_t dring) {
        constexpr int set = decltype(set_c)::value;
        constexpr int RS = NM * 3 / 4;
#pragma unroll
        for (int idx = 0; idx < NM; ++idx) {
            const int tm = idx / TN, tn = idx % TN;
            mfma16<BF16>(acc[tm][tn], fb[set][tn], fa[set][tm]);      // transposed block: a lane holds one filter and 4 positions
            if (idx < RS)
#pragma unroll
                for (int r = idx * NR / RS; r < (idx + 1) * NR / RS; ++r) lds_read(r, set ^ 1, rring);
#pragma unroll
            for (int d = idx * ND / NM; d < (idx + 1) * ND / NM; ++d) dma(d, dring);
            __builtin_amdgcn_sched_barrier(0);
        }
        advance();
    };
#pragma unroll
    for (int s = 0; s < kRing; ++s) {
#pragma unroll
        for (int d = 0; d < ND; ++d) dma(d, s);
        advance();
    }
    NT_WAIT_VMCNT((kRing - 1) * ND);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < NR; ++r) lds_read(r, 0, 0);
    __builtin_amdgcn_sched_barrier(0);

    // (slice s at ring position s % kRing; waits, barriers and the two fragment sets as in gemm_direct16_kernel; an odd last slice
    // has a trip of its own)
    uint32_t ring = 0;
    auto top = [&](uint32_t &nxt) {
        nxt = ring + 1 == kRing ? 0 : ring + 1;
        NT_WAIT_VMCNT((kRing - 2) * ND);
        __syncthreads();
    };
    for (int32_t sl = 0; sl + 1 < n_slices; sl += 2) {
        uint32_t nxt;
        top(nxt);
        trip(std::integral_constant<int, 0>{}, nxt, ring);
        ring = nxt;
        top(nxt);
        trip(std::integral_constant<int, 1>{}, nxt, ring);
        ring = nxt;
        asm volatile("s_nop 7" ::: "memory");              // (wait states ahead of anything the compiler may do to an accumulator)
    }
    if (n_slices & 1) {
        uint32_t nxt;
        top(nxt);
        trip(std::integral_constant<int, 0>{}, nxt, ring);
        asm volatile("s_nop 15" ::: "memory");
    }
    NT_WAIT_VMCNT(0);                                      // drain the surplus loads ...
    __syncthreads();                                       // ... of every wavefront: the epilogue reuses the LDS
    asm volatile("s_nop 15" ::: "memory");                 // (see gemm_direct16_kernel)

    // ---- epilogue: the wavefront's part as fp32 through its own quarter of the LDS ([filter row][positions], 16-byte chunks XOR-ed
    // with the row), then stored along the positions
    constexpr int WT = BT / 2, RB = WT * 4, CPR = RB / 16;
    char *reg = smem + wave * (WT * RB);
    const int l16 = lane & 15, grp = lane >> 4;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn) {
            float4v blk = acc[tm][tn];
            asm volatile("" : "+a"(blk));
            const int r = tm * 16 + l16, c = tn * 4 + grp;
            lds_write16(reg + r * RB, (uint32_t)((c ^ (r & (CPR - 1))) << 4),
                        u32x4{__builtin_bit_cast(uint32_t, (float)blk[0]), __builtin_bit_cast(uint32_t, (float)blk[1]),
                              __builtin_bit_cast(uint32_t, (float)blk[2]), __builtin_bit_cast(uint32_t, (float)blk[3])});
        }
    auto four = [&](int r, int c) {                        // chunk c (4 positions) of filter row r
        return __builtin_bit_cast(float4v, lds_read16(reg, (uint32_t)(r * RB + ((c ^ (r & (CPR - 1))) << 4))));
    };
    const int32_t frow = row0 + wave_m * WT, mcol = col0 + wave_n * WT;
    if (g.ksplit > 1 || g.out_dtype == NT_F32) {
        constexpr int RPI = 64 / CPR;                      // 4 positions per lane
        for (int it = 0; it < WT / RPI; ++it) {
            const int r = it * RPI + lane / CPR, c = lane % CPR;
            const float4v v = four(r, c);
            const int32_t f = frow + r, m = mcol + c * 4;
            if (f >= g.F || m >= g.M) continue;
            if (g.ksplit > 1) {
                float *dst = g.ws + ((int64_t)part * g.F + f) * g.M + m;
                if (m + 4 <= g.M) __builtin_memcpy(dst, &v, 16);
                else
                    for (int e = 0; e < 4; ++e)
                        if (m + e < g.M) dst[e] = v[e];
                continue;
            }
            const int32_t n = (int32_t)((uint32_t)m / (uint32_t)g.PQ), pq = m - n * g.PQ;
            float *y = reinterpret_cast<float *>(g.Y) + (int64_t)f * g.syf;
            if (pq + 4 <= g.PQ) __builtin_memcpy(y + (int64_t)n * g.syn + pq, &v, 16);
            else
                for (int e = 0; e < 4; ++e)
                    if (m + e < g.M) {
                        const int32_t ne = (int32_t)((uint32_t)(m + e) / (uint32_t)g.PQ);
                        y[(int64_t)ne * g.syn + (m + e - ne * g.PQ)] = v[e];
                    }
        }
        return;
    }
    constexpr int CP8 = WT / 8, RPI = 64 / CP8;            // 8 positions per lane
    for (int it = 0; it < WT / RPI; ++it) {
        const int r = it * RPI + lane / CP8, c = lane % CP8;
        const float4v lo = four(r, 2 * c), hi = four(r, 2 * c + 1);
        const int32_t f = frow + r, m = mcol + c * 8;
        if (f >= g.F || m >= g.M) continue;
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float x0 = i < 2 ? lo[2 * i] : hi[2 * i - 4], x1 = i < 2 ? lo[2 * i + 1] : hi[2 * i - 3];
            w[i] = g.out_dtype == NT_F16 ? (uint32_t)f32_to_f16_rne(x0) | ((uint32_t)f32_to_f16_rne(x1) << 16)
                                         : (uint32_t)f32_to_bf16_rne(x0) | ((uint32_t)f32_to_bf16_rne(x1) << 16);
        }
        const int32_t n = (int32_t)((uint32_t)m / (uint32_t)g.PQ), pq = m - n * g.PQ;
        uint16_t *y = reinterpret_cast<uint16_t *>(g.Y) + (int64_t)f * g.syf;
        const u32x4 out{w[0], w[1], w[2], w[3]};
        if (pq + 8 <= g.PQ) __builtin_memcpy(y + (int64_t)n * g.syn + pq, &out, 16);
        else                                               // a chunk that straddles two images (or the last one's end)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (m + e < g.M) {
                    const int32_t ne = (int32_t)((uint32_t)(m + e) / (uint32_t)g.PQ);
                    y[(int64_t)ne * g.syn + (m + e - ne * g.PQ)] = (uint16_t)((e & 1) ? w[e >> 1] >> 16 : w[e >> 1] & 0xffffu);
                }
    }
}

// the parts of a k split, added in part order (eight loads in flight), converted once
__global__ __launch_bounds__(256) void conv_cl_sum_kernel(const ConvClArgs g)
{
    const uint32_t total = (uint32_t)g.F * (uint32_t)g.M;   // (below 2^31: it fits the workspace)
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < total; i += gridDim.x * 256) {
        float sum = 0.f;
        for (int j = 0; j < g.ksplit; j += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = j + u < g.ksplit ? g.ws[(int64_t)(j + u) * total + i] : 0.f;
#pragma unroll
            for (int u = 0; u < 8; ++u) sum += v[u];
        }
        const uint32_t f = i / (uint32_t)g.M, m = i - f * (uint32_t)g.M, n = m / (uint32_t)g.PQ;
        store_out(g.Y, (int64_t)n * g.syn + (int64_t)f * g.syf + (m - n * (uint32_t)g.PQ), sum, g.out_dtype);
    }
}

nt_status launch_conv_cl_copy(const ConvClCopy &c, hipStream_t s)
{
    const int64_t blocks = (int64_t)c.N * ((c.C + 63) / 64) * (((int64_t)c.Hc * c.Wc + 63) / 64);
    const int64_t filters = c.w ? c.F : 0;
    const size_t lds = std::max<size_t>(64 * kClPitch * 2, c.w ? (size_t)c.C * c.RS * 2 : 0);       // (at most 64 KB: C R S <= 32768)
    hipLaunchKernelGGL(conv_cl_copy_kernel, dim3((unsigned)(blocks + filters)), dim3(256), lds, s, c, (int32_t)blocks);
    return check_launch("conv_cl_copy_kernel");
}

template <int BT, bool BF16, bool TRACE = false>
static nt_status launch_conv_cl_t(const ConvClArgs &a, hipStream_t s)
{
    constexpr size_t smem = (size_t)ring_of(BT, BT) * 2 * BT * kSliceK * sizeof(uint16_t);
    auto kern = gemm_conv_cl_kernel<BT, BF16, TRACE>;
    static DeviceOnce configured;
    if (!configured.done()) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return fail(NT_ERR_DEVICE, std::string("hipFuncSetAttribute: ") + hipGetErrorString(e));
        configured.set();
    }
    hipLaunchKernelGGL(kern, dim3(TRACE ? 1u : (unsigned)(a.mt * a.nt * a.ksplit)), dim3(kThreads), smem, s, a);
    return check_launch("gemm_conv_cl_kernel");
}

nt_status launch_conv_cl_trace(const ConvClArgs &a, int tile, hipStream_t s)
{
    return tile == 64 ? launch_conv_cl_t<64, false, true>(a, s) : launch_conv_cl_t<128, false, true>(a, s);
}

nt_status launch_conv_cl(const ConvClArgs &a, int tile, bool bf16, hipStream_t s)
{
    nt_status st;
    if (tile == 64) st = bf16 ? launch_conv_cl_t<64, true>(a, s) : launch_conv_cl_t<64, false>(a, s);
    else st = bf16 ? launch_conv_cl_t<128, true>(a, s) : launch_conv_cl_t<128, false>(a, s);
    if (st != NT_OK || a.ksplit == 1) return st;
    const int64_t blocks = std::min<int64_t>(((int64_t)a.F * a.M + 255) / 256, 4096);
    hipLaunchKernelGGL(conv_cl_sum_kernel, dim3((unsigned)blocks), dim3(256), 0, s, a);
    return check_launch("conv_cl_sum_kernel");
}

}  // namespace nt
