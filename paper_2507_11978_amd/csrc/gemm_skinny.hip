// Products of few rows (M <= 32: the linear layers of a decoding step), both operands with unit stride along k (the weights
// stored [out, in]).
//
// Such a product is bound by reading B once (2 M flop per element), so what matters is that every compute unit has as many
// whole cache lines of B in flight as it can and that nothing else travels.  One workgroup owns 16 columns of C for all M
// rows; its eight wavefronts share the reduction, each streaming its own part of B and A, and add their partial sums through
// LDS at the end, in wavefront order.  The reduction is thus split eight ways inside a program: no partial tile goes through
// memory, no second launch adds them, and no wavefront waits for another before the end.
//
// A step is 64 k.  A 16-byte load instruction that fetches matrix fragments directly (16 rows, 32 k) touches 16 cache lines
// and uses half of each; here it fetches 8 rows of 64 k, whole lines, and the wavefront turns the step's 16 x 64 blocks round
// in an LDS region of its own (chunk c of row r at chunk c ^ (r % 8); LDS operations of one wavefront complete in order, so
// no barrier).  Measured at 16 x 4096 x 4096 fp16: 7.6 us a call over rotating weights (4.4 TB/s); in graph replays, gaps between
// the nodes included, 8.1 us, 10.0 with fragments fetched directly, 10.9 as two launches (a k split of 64 x 64 tiles and the
// kernel that adds the parts); 16 x 8192 x 8192 26.6 us (5.0 TB/s, a large copy's rate) against 32.5.  Two batches of U steps are in flight per wavefront; U = 4 measured no better.
#include "gemm_skinny.h"

namespace nt {

typedef float float4s __attribute__((ext_vector_type(4)));
constexpr int kSkinnyWaves = 8, kSkinnyStep = 64, kSkinnyCols = 16;

template <bool BF16>
__device__ __forceinline__ float4s mfma16s(u32x4 a, u32x4 b, float4s c)
{
    if constexpr (BF16) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bhalf8, a), __builtin_bit_cast(bhalf8, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c, 0, 0, 0);
}

// the first n of the eight elements at p (all of them if n >= 8, none if n <= 0), the rest zero
__device__ __forceinline__ u32x4 load_upto8(const uint16_t *p, int n)
{
    u32x4 v{0, 0, 0, 0};
    if (n >= 8) {
        __builtin_memcpy(&v, p, 16);
    } else {
#pragma unroll
        for (int e = 0; e < 7; ++e)
            if (e < n) v[e >> 1] |= (uint32_t)p[e] << (16 * (e & 1));
    }
    return v;
}

// MB: blocks of 16 rows of A; U: steps per batch
template <bool BF16, int MB, int U>
__global__ __launch_bounds__(64 * kSkinnyWaves) void gemm_skinny_kernel(const FastArgs g)
{
    // per wavefront and step of a batch: MB blocks of A and one of B, 16 rows x 128 bytes each; at the end the partial sums
    __shared__ __attribute__((aligned(16))) char stage[kSkinnyWaves][U][MB + 1][2048];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, grp = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t col0 = (int64_t)blockIdx.x * kSkinnyCols;
    const int M = (int)g.M, N = (int)g.N, K = (int)g.K;

    // load h of a block: row 8 h + lane / 8, chunk lane % 8 (rows past the operand repeat its last one and are never stored)
    const int cr = lane >> 3, cc = lane & 7;
    const uint16_t *p[MB + 1][2];
#pragma unroll
    for (int b = 0; b < MB; ++b)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int row = b * 16 + h * 8 + cr;
            p[b][h] = g.A + (int64_t)(row < M ? row : M - 1) * g.lda + cc * 8;
        }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int64_t n = col0 + h * 8 + cr;
        p[MB][h] = g.B + (n < N ? n : N - 1) * g.ldb + cc * 8;
    }
    const uint32_t wr = (uint32_t)(cr * 128 + ((cc ^ cr) << 4));       // (row cr + 8 has the same swizzle: + 1024)
    uint32_t rd[2];                                                     // fragment f: row l16, k 32 f + 8 grp
#pragma unroll
    for (int f = 0; f < 2; ++f) rd[f] = (uint32_t)(l16 * 128 + (((4 * f + grp) ^ (l16 & 7)) << 4));

    float4s acc[MB];
#pragma unroll
    for (int a = 0; a < MB; ++a) acc[a] = float4s{0.f, 0.f, 0.f, 0.f};

    struct Step { u32x4 v[MB + 1][2]; };
    auto fetch = [&](Step &st, int s) {
        const int k = s * kSkinnyStep;
#pragma unroll
        for (int b = MB; b >= 0; --b)
#pragma unroll
            for (int h = 0; h < 2; ++h) __builtin_memcpy(&st.v[b][h], p[b][h] + k, 16);
    };
    auto multiply = [&](const Step &st, int u) {
        char (*sm)[2048] = stage[wave][u];
#pragma unroll
        for (int b = 0; b <= MB; ++b)
#pragma unroll
            for (int h = 0; h < 2; ++h) *reinterpret_cast<u32x4 *>(sm[b] + wr + 1024 * h) = st.v[b][h];
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            const u32x4 bf = *reinterpret_cast<const u32x4 *>(sm[MB] + rd[f]);
#pragma unroll
            for (int a = 0; a < MB; ++a) acc[a] = mfma16s<BF16>(*reinterpret_cast<const u32x4 *>(sm[a] + rd[f]), bf, acc[a]);
        }
    };

    // this wavefront's whole steps s0 .. s1 - 1, in batches of U, the next batch's loads in flight during this one's arithmetic
    const int steps = K / kSkinnyStep;
    const int s0 = steps * wave / kSkinnyWaves, s1 = steps * (wave + 1) / kSkinnyWaves;
    if (s0 < s1) {
        Step st[2][U];
        auto batch = [&](Step (&t)[U], int s) {
#pragma unroll
            for (int u = 0; u < U; ++u) fetch(t[u], s + u < s1 ? s + u : s1 - 1);
        };
        auto use = [&](const Step (&t)[U], int s) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (s + u < s1) multiply(t[u], u);             // (uniform)
        };
        batch(st[0], s0);
        for (int s = s0; s < s1; s += 2 * U) {
            if (s + U < s1) batch(st[1], s + U);
            use(st[0], s);
            if (s + 2 * U < s1) batch(st[0], s + 2 * U);
            if (s + U < s1) use(st[1], s + U);
        }
    }
    // the ragged end of K, fewer than 64: the last wavefront's
    if (wave == kSkinnyWaves - 1 && steps * kSkinnyStep < K) {
        const int k = steps * kSkinnyStep;
        Step st;
#pragma unroll
        for (int b = 0; b <= MB; ++b)
#pragma unroll
            for (int h = 0; h < 2; ++h) st.v[b][h] = load_upto8(p[b][h] + k, K - k - cc * 8);
        multiply(st, 0);
    }

    // partial sums, [wavefront][row][column]: a lane holds column l16 and rows 4 grp .. + 3 of a block
    constexpr int RW = MB * 16 * kSkinnyCols;
    static_assert(sizeof(stage) >= kSkinnyWaves * RW * sizeof(float), "partial sums fit the staging region");
    float *red = reinterpret_cast<float *>(&stage[0][0][0][0]);
    __syncthreads();
#pragma unroll
    for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[wave * RW + (a * 16 + 4 * grp + v) * kSkinnyCols + l16] = acc[a][v];
    __syncthreads();
    const ActParams actp = act_params(g.act);
    for (int e = tid; e < RW; e += 64 * kSkinnyWaves) {
        const int m = e / kSkinnyCols;
        const int64_t col = col0 + e % kSkinnyCols;
        if (m >= M || col >= N) continue;
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < kSkinnyWaves; ++w) sum += red[w * RW + e];
        const float v = combine(sum, g.D ? load_as_f32(g.D, m * g.sdm + col * g.sdn, g.out_dtype) : 0.f, g.alpha, g.beta);
        store_out(g.C, m * g.scm + col * g.scn, g.act ? activate(v, actp) : v, g.out_dtype);
    }
}

// Where this kernel is ahead of the tiles (us over rotating weights, fp16, this kernel / tiles).  One block of rows, 16-byte
// aligned: up to 12288 columns always (16 x 12288 x 128 4.0 / 3.9, x 4096 20.8 / 23.6); with more, each of whose programs costs a
// workgroup's start, from K = 1024 on (16 x 65536 x 128 11.9 / 7.4, x 512 22 / 17, x 1024 30 / 30, x 4096 101 / 128; 16 x 16384 x
// 1024 8.9 / 8.6), at most 65536 of them above 8 rows (16 x 128256 x 4096 197 / 187, 1 row 164 / 183).  Unaligned rows, whose loads
// cost four times as much: up to 4096 columns (16 x 4000 x 2001 7.4 / 10.7), 8192 with K >= 1000 (16 x 8000 x 511 6.6 / 5.4, x 1001
// 6.7 / 7.3, 16 x 16384 x 2001 24.6 / 17.1), and not the shortest reductions (x 127 4.4 / 3.9).  Two blocks: aligned, up to
// 8192 columns (32 x 8192 x 4096 18.3 / 21.6, 32 x 16384 x 4096 33.9 / 31.7, 32 x 65536 x 512 26 / 18); with more rows the reads of
// A, which every program repeats, outweigh the saved launch (64 x 1024 x 8192 17.9 / 10.5).
bool skinny_ok(const FastArgs &a, int alay, int blay)
{
    // (k in 32 bits; fewer than 2^32 work-items in the launch, of more the runtime starts the remainder only)
    if (alay != KCONTIG || blay != KCONTIG || a.M > 32 || a.K < kSkinnyStep || a.K > (1 << 30) || a.N > (1 << 26)) return false;
    auto al16 = [](const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
    const bool aligned = al16(a.A) && al16(a.B) && a.lda % 8 == 0 && a.ldb % 8 == 0;
    if (a.M > 16) return aligned && a.N <= 8192;
    if (!aligned) return a.K >= 256 && (a.N <= 4096 || (a.N <= 8192 && a.K >= 1000));
    return a.N <= 12288 || (a.K >= 1024 && (a.M <= 8 || a.N <= 65536));
}

// A program's wavefronts walk an eighth of the reduction each, however few programs there are: with few columns and a long
// reduction a k split of tiles, which deals it out to the whole chip, is ahead.  Measured (us, this kernel / split; 0.28 a step of
// a wavefront with one block of rows, 0.45 to 0.6 with two): 16 x 64 x 8192 7.2 / 8.8, x 16384 11.8 / 9.6, x 65536 39 / 15;
// 16 x 1024 x 8192 7.5 / 9.8, x 16384 13.3 / 11.2; 16 x 2048 x 16384 14.1 / 15.9; 32 x 64 x 8192 9.7 / 9.0, x 4096 6.1 / 8.5;
// 32 x 2048 x 8192 over rotating weights 16.3 / 13.6.
double skinny_cost(const FastArgs &a)
{
    const double steps = (double)((a.K / kSkinnyStep + kSkinnyWaves - 1) / kSkinnyWaves);
    return 2.5 + steps * (a.M <= 16 ? 0.28 : 0.56);
}

int skinny_parts(const FastArgs &a) { return (int)std::min<int64_t>(kSkinnyWaves, a.K / kSkinnyStep); }

nt_status launch_skinny(const FastArgs &a, bool bf16, hipStream_t s)
{
    const dim3 grid((unsigned)((a.N + kSkinnyCols - 1) / kSkinnyCols)), block(64 * kSkinnyWaves);
    if (a.M <= 16) {
        if (bf16) hipLaunchKernelGGL((gemm_skinny_kernel<true, 1, 2>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((gemm_skinny_kernel<false, 1, 2>), grid, block, 0, s, a);
    } else {
        if (bf16) hipLaunchKernelGGL((gemm_skinny_kernel<true, 2, 1>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((gemm_skinny_kernel<false, 2, 1>), grid, block, 0, s, a);
    }
    return check_launch("gemm_skinny_kernel");
}

}  // namespace nt
