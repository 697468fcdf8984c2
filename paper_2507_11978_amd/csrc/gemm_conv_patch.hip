// Convolution of few output positions in one launch (Section 4.3's implicit GEMM, the reduction walked in blocks of 32 channels
// and tap by tap inside a block).
//
// A program computes 16 MF filters x 16 NP consecutive positions (n, p, q).  Its wavefronts share the reduction: each takes
// every waves-th block of channels, with LDS, loads and accumulators of its own and no barrier before the end, where the
// partial sums meet in LDS and are added in wavefront order.  Nothing is copied or laid out ahead of the launch:
//   filter   a block's 32 channels x RS taps of a filter are contiguous; they stream into LDS as they are.  A lane reads the
//            RS chunks that hold its 8 channels of every tap (8 RS elements are whole 16-byte chunks) and turns them into one
//            matrix fragment per tap with four byte permutes each: a transposition at the price of the reads it replaces.
//   input    the input rows under the tile's positions, 32 channels, are read once per block (runs of four elements along the
//            row, eight channels per lane), turned into 8-channel chunks by byte permutes, and lie in LDS as four planes of 8
//            channels, one 16-byte chunk per input position, padded with zeros.  A fragment is 16 positions' chunks; another
//            tap is the same chunks a constant further on, so the unfolded input never exists, nor a padding test.
// Planes are a multiple of 256 bytes, and a read's 16 positions are consecutive chunks wherever a row does not end: conflict free.
//
// Bound by latency: a few blocks of channels per wavefront, each the round trip of its loads and some hundred LDS reads.  The
// route it replaces made a channels-last copy of the input and a tap-major one of the filter, multiplied, and added the parts of
// a split: three dependent launches, 64 KB of partial sums per tile through memory.  Device time in graph replays, us, before /
// now: (4,512,14,14)*(512,512,3,3) 24.8 / 11.2, (8,256,14,14)*(256,256,3,3) 22.4 / 9.0, (2,64,7,7)*(300,64,3,3) 9.2 / 4.8,
// (5,224,13,13)*(200,224,5,5) 25.6 / 12.6, (9,128,28,28)*(64,128,3,3) 17.4 / 7.8, (2,320,14,14)*(70,320,3,3) stride 2 9.9 / 8.6.
#include "gemm_conv_patch.h"

#include <cmath>

#include "gemm_direct.h"

namespace nt {

typedef float float4p __attribute__((ext_vector_type(4)));

template <bool BF16>
__device__ __forceinline__ float4p mfma16p(u32x4 a, u32x4 b, float4p c)
{
    if constexpr (BF16) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bhalf8, a), __builtin_bit_cast(bhalf8, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c, 0, 0, 0);
}

// x / d, r = 1 / d rounded: exact while x < 2^21 ((x + 1/2) / d lies at least 1 / (2 d) from a whole number)
__device__ __forceinline__ int32_t quotient(int32_t x, float r) { return (int32_t)(((float)x + 0.5f) * r); }
__device__ __forceinline__ int32_t uniform(int32_t x) { return __builtin_amdgcn_readfirstlane(x); }

// UMAX: runs per lane and block; MAXW: wavefronts per workgroup.  TRACE: not a convolution; the wavefront that takes the traced slice's block of
// channels brings it in and writes out the fragments of its tap (program = tile of positions * filter tiles + tile of filters).
template <int RS, int MF, int NP, int UMAX, int MAXW, bool BF16, bool TRACE = false>
__global__ __launch_bounds__(MAXW * 64) void conv_patch_kernel(const ConvPatchArgs g)
{
    constexpr int FT = 16 * MF, PT = 16 * NP;
    constexpr uint32_t RAW = FT * RS * 64;
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, grp = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = blockDim.x >> 6;

    // program: each XCD (workgroup index mod 8) takes a contiguous share of the tiles, the one operand's tile changing slowly
    int32_t fi, pi;
    {
        const int32_t grid = g.ft * g.pt, q8 = grid >> 3, r8 = grid & 7, x = blockIdx.x & 7, l = blockIdx.x >> 3;
        const int32_t seq = (x < r8 ? x * (q8 + 1) : r8 * (q8 + 1) + (x - r8) * q8) + l;
        const int32_t outer = uniform(quotient(seq, g.inv_inner)), in = seq - outer * g.inner;
        fi = g.f_major ? outer : in;
        pi = g.f_major ? in : outer;
    }
    int32_t first = wave;                                                          // this wavefront's first block of channels
    if constexpr (TRACE) {
        fi = g.trace_program % g.ft;
        pi = g.trace_program / g.ft;
        first = g.trace_slice / RS;
        if (wave != first % waves) return;
    }
    const int32_t f0 = fi * FT, m0 = pi * PT;
    char *const mine = smem + wave * g.region;
    char *const planes = mine + RAW;
    const uint32_t raw0 = __builtin_amdgcn_readfirstlane((int)((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem + wave * g.region));

    // ---- filter: load (mf, i) brings 64 bytes of each of 16 rows; chunk c of the 64 at c ^ swz (reads: see below)
    const uint32_t swz = (uint32_t)((4 - ((lane >> 4) & 3)) & 3);                  // row lane / 4
    uint32_t woff[MF];
#pragma unroll
    for (int mf = 0; mf < MF; ++mf) {
        const int32_t f = f0 + mf * 16 + (lane >> 2);                              // (rows past the last filter repeat it and are never stored)
        woff[mf] = (uint32_t)(f < g.F ? f : g.F - 1) * g.ldb * 2u + ((((uint32_t)lane & 3u) ^ swz) << 4);
    }
    auto request_filter = [&](int32_t b) {
        const char *p = reinterpret_cast<const char *>(g.w) + (int64_t)b * (RS * 64);
#pragma unroll
        for (int mf = 0; mf < MF; ++mf)
#pragma unroll
            for (int i = 0; i < RS; ++i) dma16(p + i * 64, woff[mf], raw0 + (uint32_t)((mf * RS + i) * 1024));
    };
    request_filter(first);

    // ---- geometry of the patch
    const int32_t m1 = (m0 + PT < g.M ? m0 + PT : g.M) - 1;
    const int32_t n0 = uniform(quotient(m0, g.inv_pq)), n1 = uniform(quotient(m1, g.inv_pq)), more = n1 - n0;      // first image, images after it
    const int32_t p0 = uniform(quotient(m0 - n0 * g.PQ, g.inv_q)), p1 = uniform(quotient(m1 - n1 * g.PQ, g.inv_q));
    const int32_t rows0 = ((more ? g.P - 1 : p1) - p0) * g.sh + g.span;            // input rows of the first image
    auto row_base = [&](int32_t i) { return i == 0 ? -p0 * g.sh : rows0 + (i - 1) * g.image; };      // slot row of image i's padded row 0
    uint32_t pos[NP];                                                              // this lane's position, per fragment: byte offset of its chunk under tap 0
#pragma unroll
    for (int np = 0; np < NP; ++np) {
        const int32_t m = m0 + np * 16 + l16 < m1 ? m0 + np * 16 + l16 : m1;
        const int32_t rel = m - n0 * g.PQ, i = quotient(rel, g.inv_pq), r = rel - i * g.PQ;
        const int32_t p = quotient(r, g.inv_q), q = r - p * g.Q;
        pos[np] = (uint32_t)grp * g.plane + (uint32_t)((row_base(i) + p * g.sh) * g.row + q * g.sw) * 16u;
    }
    // runs of four elements of an image's plane: first image from row ha0 on, the others from row 0
    const int32_t ha0 = p0 * g.sh - g.ph > 0 ? p0 * g.sh - g.ph : 0;
    auto last_row = [&](int32_t p) { const int32_t h = p * g.sh + g.span - 1 - g.ph; return h < g.H - 1 ? h : g.H - 1; };
    const int32_t hb0 = more ? g.last_h : last_row(p1), hb1 = last_row(p1);
    const int32_t es0 = (ha0 * g.W) & ~3;
    const int32_t c0 = hb0 >= ha0 ? ((hb0 + 1) * g.W - es0 + 3) >> 2 : 0, c1 = hb1 >= 0 ? ((hb1 + 1) * g.W + 3) >> 2 : 0;
    const int32_t runs = more ? c0 + (more - 1) * g.units + c1 : c0;
    const uint32_t grp_off = (uint32_t)(grp * 8) * (uint32_t)g.xs1 * 2u;
    uint32_t goff[UMAX], slot[UMAX][4];
    const uint32_t trash = (uint32_t)grp * g.plane + g.plane - 16;                 // (a plane's last chunk is nobody's)
#pragma unroll
    for (int k = 0; k < UMAX; ++k) {
        goff[k] = 0;
        if (16 * k >= runs) continue;                                              // (uniform)
        const int32_t u = l16 + 16 * k, v = u - c0;
        const bool ok = u < runs, first = v < 0;
        const int32_t j = more ? quotient(v, g.inv_units) : 0;
        const int32_t i = !ok || first ? 0 : 1 + j;
        const int32_t e = !ok ? 0 : first ? es0 + 4 * u : 4 * (v - j * g.units);
        const int32_t ha = first ? ha0 : 0, hb = first ? hb0 : i == more ? hb1 : g.last_h;
        const int32_t HW = g.H * g.W, s = e < HW - 4 ? e : HW - 4;                 // (the plane's last run starts early)
        goff[k] = ((uint32_t)(n0 + i) * g.xs0 + (uint32_t)s) * 2u + grp_off;
        int32_t h = quotient(s, g.inv_w), w = s - h * g.W;
        const int32_t base = row_base(i) + g.ph;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int32_t wp = w + g.pw;
            const bool in = ok && h >= ha && h <= hb && wp < g.row;
            slot[k][t] = in ? (uint32_t)grp * g.plane + (uint32_t)((base + h) * g.row + wp) * 16u : trash;
            const bool end = ++w == g.W;
            w = end ? 0 : w;
            h += end ? 1 : 0;
        }
    }
    u32x2 X[UMAX][8];
    const int64_t xs1 = g.xs1;
    auto request_input = [&](int32_t b) {
        const char *p = reinterpret_cast<const char *>(g.x) + (int64_t)b * 64 * xs1;
#pragma unroll
        for (int k = 0; k < UMAX; ++k)
            if (16 * k < runs) {                                                   // (uniform)
#pragma unroll
                for (int j = 0; j < 8; ++j) __builtin_memcpy(&X[k][j], p + (int64_t)j * xs1 * 2 + goff[k], 8);
            }
    };
    request_input(first);
    for (uint32_t a = lane * 16; a < 4 * g.plane; a += 1024) lds_write16(planes, a, u32x4{0, 0, 0, 0});

    float4p acc[MF][NP];
#pragma unroll
    for (int mf = 0; mf < MF; ++mf)
#pragma unroll
        for (int np = 0; np < NP; ++np) acc[mf][np] = float4p{0.f, 0.f, 0.f, 0.f};

    for (int32_t b = first; b < g.blocks; b += waves) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                           // the block has arrived
        // ---- filter fragments: lane (row l16, channels 8 grp ..) of every tap.  Chunk c of a row lies in kilobyte c / 4.
        u32x4 A[MF][RS];
#pragma unroll
        for (int mf = 0; mf < MF; ++mf) {
            u32x4 r[RS];
#pragma unroll
            for (int i = 0; i < RS; ++i) {
                const uint32_t c = (uint32_t)(RS * grp + i);
                r[i] = lds_read16(mine, (uint32_t)(mf * RS * 1024) + (c >> 2) * 1024u + (uint32_t)(l16 * 64) + (((c & 3u) ^ (uint32_t)((4 - (l16 >> 2)) & 3)) << 4));
            }
#pragma unroll
            for (int t = 0; t < RS; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int lo = 2 * i * RS + t, hi = lo + RS;                   // the elements of channels 2 i and 2 i + 1
                    const uint32_t sel = ((hi & 1) ? 0x07060000u : 0x05040000u) | ((lo & 1) ? 0x0302u : 0x0100u);
                    A[mf][t][i] = __builtin_amdgcn_perm(r[hi / 8][(hi / 2) % 4], r[lo / 8][(lo / 2) % 4], sel);
                }
        }
        // ---- input: four elements x eight channels into four chunks
#pragma unroll
        for (int k = 0; k < UMAX; ++k)
            if (16 * k < runs) {
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    u32x4 v;
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = __builtin_amdgcn_perm(X[k][2 * i + 1][t >> 1], X[k][2 * i][t >> 1], (t & 1) ? 0x07060302u : 0x05040100u);
                    lds_write16(planes, slot[k][t], v);
                }
            }
        if constexpr (TRACE) {
            const int32_t tap = g.trace_slice - first * RS;
            uint16_t *out = g.trace_out + l16 * 32 + grp * 8;
            if (g.trace_operand == 0) {
#pragma unroll
                for (int np = 0; np < NP; ++np) {
                    const u32x4 v = lds_read16(planes, pos[np] + (uint32_t)g.tap[tap]);
                    __builtin_memcpy(out + np * 512, &v, 16);
                }
            } else {
#pragma unroll
                for (int mf = 0; mf < MF; ++mf)
#pragma unroll
                    for (int t = 0; t < RS; ++t)
                        if (t == tap) __builtin_memcpy(out + mf * 512, &A[mf][t], 16);
            }
            return;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");                         // (the raw filter has been read: the next block may land on it)
        if (b + waves < g.blocks) {
            request_filter(b + waves);
            request_input(b + waves);
        }
        u32x4 B[2][NP];
#pragma unroll
        for (int np = 0; np < NP; ++np) B[0][np] = lds_read16(planes, pos[np] + (uint32_t)g.tap[0]);
#pragma unroll
        for (int t = 0; t < RS; ++t) {
            if (t + 1 < RS)
#pragma unroll
                for (int np = 0; np < NP; ++np) B[(t + 1) & 1][np] = lds_read16(planes, pos[np] + (uint32_t)g.tap[t + 1]);
#pragma unroll
            for (int np = 0; np < NP; ++np)
#pragma unroll
                for (int mf = 0; mf < MF; ++mf) acc[mf][np] = mfma16p<BF16>(B[t & 1][np], A[mf][t], acc[mf][np]);
        }
    }

    // ---- the wavefronts' sums, each in its own region as [filter][positions] (a lane holds filter l16 and 4 positions of a block;
    // rows one chunk longer than their positions), added in wavefront order and stored along the positions
    constexpr uint32_t PITCH = PT * 4 + 16;
#pragma unroll
    for (int mf = 0; mf < MF; ++mf)
#pragma unroll
        for (int np = 0; np < NP; ++np) {
            const float4p v = acc[mf][np];
            lds_write16(mine, (uint32_t)(mf * 16 + l16) * PITCH + (uint32_t)(np * 64 + grp * 16),
                        u32x4{__builtin_bit_cast(uint32_t, (float)v[0]), __builtin_bit_cast(uint32_t, (float)v[1]),
                              __builtin_bit_cast(uint32_t, (float)v[2]), __builtin_bit_cast(uint32_t, (float)v[3])});
        }
    __syncthreads();
    constexpr int CH = PT / 8;                             // chunks of 8 positions per filter
    for (int it = tid; it < FT * CH; it += waves * 64) {
        const int r = it / CH, c = it - r * CH;
        const int32_t f = f0 + r, m = m0 + c * 8;
        if (f >= g.F || m >= g.M) continue;
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = 0.f;
        for (int w = 0; w < waves; ++w) {
            const char *p = smem + w * g.region;
            const float4p lo = __builtin_bit_cast(float4p, lds_read16(p, (uint32_t)r * PITCH + (uint32_t)c * 32u));
            const float4p hi = __builtin_bit_cast(float4p, lds_read16(p, (uint32_t)r * PITCH + (uint32_t)c * 32u + 16u));
#pragma unroll
            for (int e = 0; e < 4; ++e) { v[e] += lo[e]; v[4 + e] += hi[e]; }
        }
        const int32_t n = quotient(m, g.inv_pq), pq = m - n * g.PQ;
        const int64_t at = (int64_t)n * g.syn + (int64_t)f * g.syf + pq;
        const bool whole = pq + 8 <= g.PQ;                 // (else: it straddles two images, or the last one's end)
        if (g.out_dtype == NT_F32) {
            float *y = reinterpret_cast<float *>(g.Y);
            if (whole) __builtin_memcpy(y + at, v, 32);
            else
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (m + e < g.M) { const int32_t ne = quotient(m + e, g.inv_pq); y[(int64_t)ne * g.syn + (int64_t)f * g.syf + (m + e - ne * g.PQ)] = v[e]; }
            continue;
        }
        uint32_t o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            o[i] = g.out_dtype == NT_F16 ? (uint32_t)f32_to_f16_rne(v[2 * i]) | ((uint32_t)f32_to_f16_rne(v[2 * i + 1]) << 16)
                                         : (uint32_t)f32_to_bf16_rne(v[2 * i]) | ((uint32_t)f32_to_bf16_rne(v[2 * i + 1]) << 16);
        uint16_t *y = reinterpret_cast<uint16_t *>(g.Y);
        if (whole) __builtin_memcpy(y + at, o, 16);
        else
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (m + e < g.M) {
                    const int32_t ne = quotient(m + e, g.inv_pq);
                    y[(int64_t)ne * g.syn + (int64_t)f * g.syf + (m + e - ne * g.PQ)] = (uint16_t)((e & 1) ? o[e >> 1] >> 16 : o[e >> 1] & 0xffffu);
                }
    }
}

// ---- host side
// the kernels that are built: taps, blocks of 16 filters and positions per tile, runs per lane and block, wavefronts at most
#define NT_PATCH_TILES(X) \
    X(9, 1, 2, 5, 8) X(9, 1, 3, 5, 8) X(9, 1, 6, 5, 8) X(9, 2, 2, 4, 8) X(9, 2, 3, 4, 8) X(9, 2, 4, 4, 8) X(9, 2, 6, 8, 4) X(9, 4, 2, 8, 4) \
    X(25, 1, 2, 7, 4) X(25, 1, 4, 7, 4) X(25, 1, 6, 8, 4) \
    X(1, 1, 2, 5, 8) X(1, 2, 2, 5, 8) X(1, 2, 4, 8, 8) X(1, 4, 2, 5, 8) X(1, 4, 4, 8, 8)
struct PatchTile { int taps, mf, np, umax, maxw; };
#define NT_PATCH_ENTRY(RS, MF, NP, U, W) {RS, MF, NP, U, W},
static const PatchTile kPatchTiles[] = {NT_PATCH_TILES(NT_PATCH_ENTRY)};
#undef NT_PATCH_ENTRY

// sizes of a patch that the estimate needs
struct PatchSizes { int64_t rows, row, span, image, images, last_h, units, runs, plane, region, blocks, most; };

static bool patch_sizes(const ConvHint &h, const PatchTile &t, PatchSizes *z)
{
    const int64_t taps = h.R * h.S, PT = 16 * t.np, FT = 16 * t.mf, PQ = h.P * h.Q;
    z->span = (h.R - 1) * h.dh + 1;
    z->image = (h.P - 1) * h.sh + z->span;
    z->row = (h.Q - 1) * h.sw + (h.S - 1) * h.dw + 1;
    // the most output rows and images that PT positions touch, the most input rows under them (more images: span rows for sh)
    const int64_t out_rows = std::min<int64_t>((PT + h.Q - 2) / h.Q + 1, h.N * h.P);
    const int64_t images = z->images = std::min<int64_t>(std::min<int64_t>((PT + PQ - 2) / PQ + 1, h.N), out_rows);
    z->rows = std::max((out_rows - 1) * h.sh + z->span, (out_rows - images) * h.sh + images * z->span);
    z->last_h = std::min<int64_t>(h.H - 1, (h.P - 1) * h.sh + z->span - 1 - h.ph);
    z->units = z->last_h >= 0 ? ((z->last_h + 1) * h.W + 3) / 4 : 1;
    // (every image's rows start on a run of their own)
    z->runs = (std::min(z->rows, images * std::max<int64_t>(z->last_h + 1, 0)) * h.W + 3) / 4 + images;
    z->plane = (z->rows * z->row * 16 + 16 + 255) / 256 * 256;
    z->region = std::max<int64_t>(FT * taps * 64 + 4 * z->plane, (FT * (PT * 4 + 16) + 255) / 256 * 256);
    z->blocks = h.C / 32;
    z->most = std::min<int64_t>(std::min<int64_t>(t.maxw, (160 << 10) / z->region), z->blocks);
    return z->runs <= 16 * t.umax && z->most >= 1;
}

// Estimated time (us) of the launch on that tile with `waves` wavefronts per program: programs run in rounds of as many as a
// unit's LDS and registers hold; a program costs a fixed part, its blocks of channels -- each the latency of a wavefront's own
// work, or the unit's throughput for all that are resident, whichever is longer -- and the sum of its wavefronts' parts.
// A fit to launches on every tile for nine and 25 taps (64 to 512 channels and filters, images of 7 to 56, both strides).  190 drawn convolutions
// that it sends here take 1.09 times its figure in the mean, with a spread of 12 % (four sets of operands in turn, graph replays).  One tap: it picks
// the tile only, see patch_cost_one_tap.
static double patch_cost(const PatchTile &t, const PatchSizes &z, int64_t programs, int64_t waves)
{
    // (LDS is dealt out in pieces of 1280 bytes: five programs of 32 KB do not fit)
    const double slots = t.maxw == 8 ? 8 : 4, units = 256;
    const double resident = std::max(1.0, std::min((double)(128 / ((z.region * waves + 1279) / 1280)), std::floor(slots / (double)waves)));
    // (programs to a unit: between one and two, units that have two set the pace more than the mean says, in long walks.  By the
    // mean alone (4,512,14,14)*(512,512,3,3) ran on 384 programs, 13.7 us, for 192 of twice the filters, 12.2;
    // (8,416,13,13)*(88,416,3,3) on 11.3 us for 9.0.  Of less than 12 blocks programs leave their unit to the next before they get in its way:
    // there this loses, 288 channels 14.0 / 15.4, 128 6.6 / 7.9, for some that gain, 128 channels 8.0 / 7.0.  Twelve is where the drawn ones that it picks another
    // tile for stop losing: 310 of 64 to 512 channels, geometric mean 0.998, none slower)
    const double share = (double)programs / units, mine = programs > units ? std::min(resident, share < 2 && z.blocks >= 12 ? 0.5 * (share + 2) : share) : 1.0;
    double rounds = std::max(1.0, (double)programs / (units * resident));
    rounds = rounds < 4 ? std::ceil(rounds) : rounds + 0.3;
    const double runs = (double)((z.runs + 15) / 16), mm = t.taps * t.mf * t.np, reads = t.taps * (t.mf + t.np);
    const double latency = 0.139 + 0.0188 * mm + 0.112 * runs, unit = (0.0337 + 0.00615 * reads) * mine * (double)waves;
    return 2.33 + rounds * (1.30 + 0.572e-3 * (double)z.plane + (double)((z.blocks + waves - 1) / waves) * std::max(latency, unit) + 0.0324 * (double)((waves - 1) * t.mf * t.np));
}

// The same for one tap on the tile that patch_cost has picked: with two to eight matrix instructions per block the loads are all there is
// to it, and patch_cost, a fit to nine and 25 taps, is short by 10 % (stride 2) to 75 % (planes of 3 x 3).  A block costs a wavefront
// its instructions and runs, and the unit the runs of all wavefronts, more for every image whose planes are no multiple of 16 bytes apart
// (`aligned`: they are); what the launch moves comes on top, the input once more, from the caches, for every further tile of filters.
// A fit to 745 drawn launches (32 to 3400 channels, 16 to 2048 filters, planes of 3 to 56, both strides), spread 10 %.
static double patch_cost_one_tap(const ConvHint &h, const PatchTile &t, const PatchSizes &z, int64_t programs, int64_t waves, bool aligned)
{
    const double resident = std::max(1.0, std::min((double)(128 / ((z.region * waves + 1279) / 1280)), std::floor((t.maxw == 8 ? 8.0 : 4.0) / (double)waves)));
    const double share = (double)programs / 256, mine = std::max(1.0, std::min(resident, share));
    double rounds = std::max(1.0, share / resident);
    rounds = rounds < 4 ? std::ceil(rounds) : rounds + 0.3;
    const double mm = t.mf * t.np, runs = (double)((z.runs + 15) / 16);
    const double block = 0.028 * mm + 0.358 * runs + (0.0074 * runs + (aligned ? 0.0 : 0.021 * (double)z.images)) * mine * (double)waves;
    const double in = 2e-6 * (double)h.N * (double)h.C * (double)(h.H * h.W), out = 2e-6 * (double)h.N * (double)h.K * (double)(h.P * h.Q);
    return 3.4 + rounds * ((double)((z.blocks + waves - 1) / waves) * block + 0.04 * (double)(waves - 1) * mm) + (0.07 + 0.006 * (double)((h.K - 1) / (16 * t.mf))) * in + 0.57 * out;
}

bool conv_patch_plan(const ConvHint &h, ConvPatchArgs *a, ConvPatchPlan *best, double *cost_out)
{
    const int64_t M = h.N * h.P * h.Q;
    double best_cost = 0;
    int i = -1;
    PatchSizes z{};
    best->waves = 0;
    for (const PatchTile &t : kPatchTiles) {
        ++i;
        PatchSizes c;
        if (t.taps != h.R * h.S || !patch_sizes(h, t, &c)) continue;
        const int64_t programs = ((h.K + 16 * t.mf - 1) / (16 * t.mf)) * ((M + 16 * t.np - 1) / (16 * t.np));
        if (programs >= (1 << 20)) continue;               // (exact division in the kernel)
        int64_t last = 0;
        for (int64_t w = c.most; w >= 1; --w) {
            const int64_t per = (c.blocks + w - 1) / w, waves = (c.blocks + per - 1) / per;        // (no more than its rounds of blocks need)
            if (waves == last) continue;
            last = waves;
            const double cost = patch_cost(t, c, programs, waves);
            if (best->waves == 0 || cost < best_cost) { best_cost = cost; best->tile = i; best->waves = (int)waves; z = c; }
        }
    }
    if (best->waves == 0) return false;
    const PatchTile &t = kPatchTiles[best->tile];
    const int64_t PT = 16 * t.np, FT = 16 * t.mf, PQ = h.P * h.Q;
    const int64_t programs = ((h.K + FT - 1) / FT) * ((M + PT - 1) / PT);
    // (one tap beyond 10.3 of patch_cost: longer walks than the fit has seen, and slower by far than it says: (2,9120,14,14)*(35,9120,1,1) 46.7 us
    // for 17.5 on the implicit kernels, strided (17,8192,14,14)*(23,8192,1,1) 74.6 for 53.8 unfolded)
    *cost_out = t.taps > 1 ? best_cost : best_cost < 10.3 ? patch_cost_one_tap(h, t, z, programs, best->waves, h.xs[0] % 8 == 0 && h.xs[1] % 8 == 0) : 1e30;
    a->xs1 = h.xs[1]; a->syn = h.ys[0]; a->syf = h.ys[1];
    a->xs0 = (uint32_t)h.xs[0]; a->ldb = (uint32_t)h.ws[0];
    a->F = (int32_t)h.K; a->M = (int32_t)M; a->blocks = (int32_t)z.blocks;
    a->H = (int32_t)h.H; a->W = (int32_t)h.W; a->P = (int32_t)h.P; a->Q = (int32_t)h.Q; a->PQ = (int32_t)PQ;
    a->sh = (int32_t)h.sh; a->sw = (int32_t)h.sw; a->ph = (int32_t)h.ph; a->pw = (int32_t)h.pw;
    a->ft = (int32_t)((h.K + FT - 1) / FT); a->pt = (int32_t)((M + PT - 1) / PT);
    // (an XCD keeps to few tiles of the larger operand)
    a->f_major = h.K * h.R * h.S > h.N * h.H * h.W ? 1 : 0;
    a->span = (int32_t)z.span; a->image = (int32_t)z.image; a->row = (int32_t)z.row;
    a->last_h = (int32_t)z.last_h; a->units = (int32_t)z.units;
    a->plane = (uint32_t)z.plane; a->region = (uint32_t)z.region;
    a->inner = a->f_major ? a->pt : a->ft;
    a->inv_inner = 1.f / (float)a->inner; a->inv_pq = 1.f / (float)PQ; a->inv_q = 1.f / (float)h.Q; a->inv_w = 1.f / (float)h.W; a->inv_units = 1.f / (float)z.units;
    for (int64_t r = 0; r < h.R; ++r)
        for (int64_t s = 0; s < h.S; ++s) a->tap[r * h.S + s] = (int32_t)((r * h.dh * z.row + s * h.dw) * 16);
    return true;
}

nt_conv_plan conv_patch_describe(const ConvPatchArgs &a, const ConvPatchPlan &p)
{
    const PatchTile &t = kPatchTiles[p.tile];
    return nt_conv_plan{1, {16 * t.np, 16 * t.np}, 16 * t.mf, {a.pt, 0}, p.waves, t.umax};
}

template <int RS, int MF, int NP, int UMAX, int MAXW, bool BF16, bool TRACE = false>
static nt_status launch_conv_patch_t(const ConvPatchArgs &a, int waves, hipStream_t s)
{
    auto kern = conv_patch_kernel<RS, MF, NP, UMAX, MAXW, BF16, TRACE>;
    static DeviceOnce configured;
    if (!configured.done()) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 << 10);
        if (e != hipSuccess) return fail(NT_ERR_DEVICE, std::string("hipFuncSetAttribute: ") + hipGetErrorString(e));
        configured.set();
    }
    hipLaunchKernelGGL(kern, dim3(TRACE ? 1u : (unsigned)(a.ft * a.pt)), dim3((unsigned)(64 * waves)), (size_t)a.region * waves, s, a);
    return check_launch("conv_patch_kernel");
}

nt_status launch_conv_patch(const ConvPatchArgs &a, const ConvPatchPlan &p, bool bf16, hipStream_t s)
{
    typedef nt_status (*Launcher)(const ConvPatchArgs &, int, hipStream_t);
#define NT_PATCH_ENTRY(RS, MF, NP, U, W) {launch_conv_patch_t<RS, MF, NP, U, W, false>, launch_conv_patch_t<RS, MF, NP, U, W, true>},
    static const Launcher table[][2] = {NT_PATCH_TILES(NT_PATCH_ENTRY)};
#undef NT_PATCH_ENTRY
    return table[p.tile][bf16 ? 1 : 0](a, p.waves, s);
}

nt_status launch_conv_patch_trace(const ConvPatchArgs &a, const ConvPatchPlan &p, hipStream_t s)
{
    typedef nt_status (*Launcher)(const ConvPatchArgs &, int, hipStream_t);
#define NT_PATCH_ENTRY(RS, MF, NP, U, W) launch_conv_patch_t<RS, MF, NP, U, W, false, true>,
    static const Launcher table[] = {NT_PATCH_TILES(NT_PATCH_ENTRY)};
#undef NT_PATCH_ENTRY
    return table[p.tile](a, p.waves, s);
}

}  // namespace nt
