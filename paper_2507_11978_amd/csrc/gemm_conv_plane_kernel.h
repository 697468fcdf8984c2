// Convolution of many output positions: 32 TM positions x 32 TN filters per program (Section 4.3's implicit GEMM; the reduction
// in blocks of 32 channels, tap by tap inside a block).
//
// The kernels that fetch the unfolded input (gemm_conv_tap.h, gemm_conv_direct.h) bring every input element in R S times, from
// rows that are mostly misaligned, and clear the padding in LDS each time; the strided ones copied the input to channels-last
// first.  Here the input rows under a tile stay in LDS for a whole block of channels, as four planes of 8 channels with one
// 16-byte chunk per input position, zero where the padding lies: a fragment of any tap is 16 chunks at the lane's fixed
// position plus the tap's scalar offset, whatever the stride, and no tap needs a test.
//   input   the next block's rows come straight into an LDS staging area (16 bytes per lane along the row) in a block's first trip
//           and are turned into the other set of planes later in the block (four elements x eight channels per lane,
//           byte permutes), so that a block boundary costs next to nothing;
//   filter  a ring of three 32-k slices from a copy in this order ([filter][block][tap][32], launch_conv_plane_filter).
// A trip is one slice: TM TN matrix instructions per wavefront, TM + TN LDS reads, TN / 2 loads.  Every vector-memory operation of
// the loop is an explicit one, so the waits count exactly.  Bound: the widest tile by its matrix instructions (and the clock they
// leave), tiles of half its size about as much by the LDS, whose reads take as long.  Device time in graph replays, the filter's
// copy included, us before / now: (32,256,56,56)*(256,256,3,3) 124.3 / 103.6, (8,256,56,56)*(256,256,3,3) 65.8 / 36.7,
// (7,448,56,56)*(114,448,3,3) 58.1 / 38.9, (7,224,56,56)*(448,224,5,5) 131.7 / 105.2, (32,128,56,56)*(256,128,3,3) stride 2 39.0 /
// 28.6.  Positions are numbered image by image, the images' sizes rounded up
// to 8 (not the rows, which costs the other kernels one position in seven for rows of 28 and one in eight for 14).
#pragma once
#include "gemm_conv_direct.h"
#include "gemm_conv_plane.h"

namespace nt {

// x / d, r = 1 / d rounded: exact while x < 2^21 ((x + 1/2) / d lies at least 1 / (2 d) from a whole number)
__device__ __forceinline__ int32_t plane_quotient(int32_t x, float r) { return (int32_t)(((float)x + 0.5f) * r); }

// mfma16 on an accumulator among the vector registers
template <bool BF16>
__device__ __forceinline__ void mfma16v(float4v &acc, const u32x4 &a, const u32x4 &b)
{
    if constexpr (BF16) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
    else asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}

constexpr int kPlaneRing = 3;      // slices of the filter
// U: runs of four elements per lane and block.  U = 2 (at most 64 runs of eight elements under a tile): two sets of planes; U = 3 (96): one, filled in a block's last trip
constexpr int plane_sets(int u) { return u == 2 ? 2 : 1; }
// TAPS: 9 (a block is nine trips of straight code), 0: any number from 6 on
// TRACE: not a convolution; the program sets itself up at the traced slice's block of channels and writes out the fragments of its tap
template <bool BF16, int TM, int TN, int U, int TAPS, bool TRACE>
__device__ __forceinline__ void conv_plane_program(const ConvPlaneArgs &g, char *smem, int32_t m0, int32_t f0)
{
    constexpr int BM = 32 * TM, BN = 32 * TN, kRing = kPlaneRing, NX = 4 * U, SETS = plane_sets(U);
    static_assert(U == 2 || U == 3, "layout of the staging area");
    using TileB = DirectTile16<BN, KCONTIG>;
    constexpr uint32_t SLICE = TileB::BYTES, RAW0 = kRing * SLICE;      // LDS: the ring, the staging area, two sets of planes
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, grp = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_m = wave >> 1, wave_n = wave & 1;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
    auto uniform = [](int32_t x) { return __builtin_amdgcn_readfirstlane(x); };
    char *const planes = smem + RAW0 + 16 * 1024 * U;
    const uint32_t set_bytes = 4 * g.plane;

    // ---- geometry: the images and output rows of the tile (a surplus position stands for its image's last one)
    const int32_t m1 = (m0 + BM < g.c.M ? m0 + BM : g.c.M) - 1;
    const int32_t n0 = uniform(plane_quotient(m0, g.inv_pq8)), n1 = uniform(plane_quotient(m1, g.inv_pq8)), more = n1 - n0;
    const int32_t r0 = m0 - n0 * g.c.PQ8, r1 = m1 - n1 * g.c.PQ8;
    const int32_t p0 = uniform(plane_quotient(r0 < g.PQ ? r0 : g.PQ - 1, g.inv_q)), p1 = uniform(plane_quotient(r1 < g.PQ ? r1 : g.PQ - 1, g.inv_q));
    const int32_t rows0 = ((more ? g.P - 1 : p1) - p0) * g.sh + g.span;            // input rows of the first image
    auto row_base = [&](int32_t i) { return i == 0 ? -p0 * g.sh : rows0 + (i - 1) * g.image; };      // plane row of image i's padded row 0
    const int32_t ha0 = p0 * g.sh - g.ph > 0 ? p0 * g.sh - g.ph : 0;
    auto last_row = [&](int32_t p) { const int32_t h = p * g.sh + g.span - 1 - g.ph; return h < g.H - 1 ? h : g.H - 1; };
    const int32_t hb0 = more ? g.last_h : last_row(p1), hb1 = last_row(p1);
    // runs of eight elements of an image's plane: first image from row ha0 on, the others from row 0
    const int32_t es0 = (ha0 * g.W) & ~7;
    const int32_t c0 = hb0 >= ha0 ? ((hb0 + 1) * g.W - es0 + 7) >> 3 : 0, c1 = hb1 >= 0 ? ((hb1 + 1) * g.W + 7) >> 3 : 0;
    const int32_t chunks0 = more ? c0 + (more - 1) * g.units + c1 : c0;
    const int32_t HW = g.H * g.W;
    // run k: image (after the first) and first element (the plane's last run starts early)
    auto run_at = [&](int32_t k, int32_t *image, int32_t *ha, int32_t *hb) {
        const bool first = k < c0;
        const int32_t v = k - c0, j = more ? plane_quotient(v < 0 ? 0 : v, g.inv_units) : 0;
        int32_t i = first ? 0 : 1 + j;
        i = i < more ? i : more;
        *image = i;
        *ha = first ? ha0 : 0;
        *hb = first ? hb0 : i == more ? hb1 : g.last_h;
        const int32_t e = first ? es0 + 8 * k : 8 * (v - j * g.units);
        return e < HW - 8 ? e : HW - 8;
    };

    // ---- the input's loads: 64 runs of one channel each, to [channel][64 runs], and (U = 3) the next 32 of two channels, to
    // [channel][32 runs] behind all of those (lanes without a run repeat the first)
    uint32_t xoff[U - 1];
#pragma unroll
    for (int i = 0; i < U - 1; ++i) {
        const int32_t k = i == 0 ? lane : 64 + (lane & 31);
        int32_t img, ha, hb;
        const int32_t e = run_at(k < chunks0 ? k : 0, &img, &ha, &hb);
        xoff[i] = ((uint32_t)(n0 + img) * g.xs0 + (uint32_t)e + (i == 0 ? 0u : (uint32_t)(lane >> 5) * (uint32_t)g.xs1)) * 2u;
    }
    const int64_t xs2 = g.xs1 * 2;
    const int32_t RS = g.R * g.S, first_slice = TRACE ? g.c.trace_slice : 0;
    const char *const x0 = reinterpret_cast<const char *>(g.x) + (int64_t)((TRACE ? first_slice / RS * 32 : 0) + wave * 8) * xs2;      // (eight channels each)
    auto request_input = [&](const char *p, int i) {           // load i of the block whose rows of this wavefront's channels start at p
        constexpr int PER2 = U == 3 ? 3 : 2;                   // loads per two channels
        const int c = i / PER2 * 2 + (i % PER2 == PER2 - 1 ? 1 : 0);
        if (U == 3 && i % 3 == 1) dma16(p + c * xs2, xoff[U - 2], lds0 + RAW0 + 32768u + (uint32_t)(wave * 4 + c / 2) * 1024u);
        else dma16(p + c * xs2, xoff[0], lds0 + RAW0 + (uint32_t)(wave * 8 + c) * 1024u);
    };
#pragma unroll
    for (int i = 0; i < NX; ++i) request_input(x0, i);

    // ---- the filter: the direct kernel's k-major operand, range checked (filters past the last read as zeros)
    TileB tb;
    tb.init(wave, lane, g.ldb, wave_n * (BN / 2), 0);
    const u32x4 rsrc = make_rsrc(g.w + (int64_t)f0 * g.ldb, (int64_t)(g.c.N - f0) * g.ldb * 2);
    const int32_t n_slices = g.blocks * RS;
    constexpr int ND = TileB::PER;
    // (slices past the last, requested by the last trips: whatever lies there, or zeros, never multiplied)
#pragma unroll
    for (int s = 0; s < kRing; ++s)
#pragma unroll
        for (int d = 0; d < ND; ++d) tb.issue_one_buf(d, rsrc, (uint32_t)(first_slice + s) * (kSliceK * 2), lds0 + s * SLICE, wave);

    // ---- this lane's runs of four elements (half a run of eight) on their way into the planes: where they lie in the staging
    // area, and each element's chunk.  Lane l writes its elements in the order t ^ ((l / 4) % 4): 16 lanes then write 16 different
    // chunks of a row's 256 bytes, not four (which took a fill 900 cycles)
    const int turn = (lane >> 2) & 3;
    const uint32_t even = turn & 1 ? 0x07060302u : 0x05040100u, odd = even ^ 0x02020202u;
    uint32_t from[U], slot[U][4];
    const uint32_t trash = (uint32_t)wave * g.plane + g.plane - 16;                // (a plane's last chunk is nobody's)
#pragma unroll
    for (int k = 0; k < U; ++k) {
        const int32_t u = lane + 64 * k;
        const bool ok = u < 2 * chunks0;
        int32_t img, ha, hb;
        const int32_t e = run_at(ok ? u >> 1 : 0, &img, &ha, &hb) + (ok ? (u & 1) * 4 : 0);
        from[k] = RAW0 + (k < 2 ? (uint32_t)wave * 8192u + (uint32_t)(ok ? u : 0) * 8u : 32768u + (uint32_t)wave * 4096u + (uint32_t)(ok ? u - 128 : 0) * 8u) + (uint32_t)(turn >> 1) * 4u;
        const int32_t base = row_base(img) + g.ph;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int32_t el = e + (t ^ turn), h = plane_quotient(el, g.inv_w), wp = el - h * g.W + g.pw;
            const bool in = ok && h >= ha && h <= hb && wp < g.row;
            slot[k][t] = in ? (uint32_t)wave * g.plane + (uint32_t)((base + h) * g.row + wp) * 16u : trash;
        }
    }
    uint32_t pos[TM];                                          // this lane's position, per fragment: its chunk under tap 0
#pragma unroll
    for (int t = 0; t < TM; ++t) {
        int32_t m = m0 + wave_m * (BM / 2) + t * 16 + l16;
        m = m < m1 ? m : m1;
        const int32_t rel = m - n0 * g.c.PQ8, i = plane_quotient(rel, g.inv_pq8);
        int32_t r = rel - i * g.c.PQ8;
        r = r < g.PQ ? r : g.PQ - 1;
        const int32_t p = plane_quotient(r, g.inv_q), q = r - p * g.Q;
        pos[t] = (uint32_t)grp * g.plane + (uint32_t)((row_base(i) + p * g.sh) * g.row + q * g.sw) * 16u;
    }
    // (each wavefront clears and later fills the plane of its number: LDS operations of one wavefront complete in order)
    for (uint32_t a = lane * 16; a < g.plane; a += 1024) {
        lds_write16(planes, wave * g.plane + a, u32x4{0, 0, 0, 0});
        if (SETS == 2) lds_write16(planes, set_bytes + wave * g.plane + a, u32x4{0, 0, 0, 0});
    }
    uint32_t X[U][2][8];                                       // [run][pair of elements, as this lane orders them][channel]
    auto take = [&](int k, int j) {
#pragma unroll
        for (int d = 0; d < 2; ++d) X[k][d][j] = *reinterpret_cast<const uint32_t *>(smem + (from[k] ^ (d * 4u)) + (uint32_t)j * (k < 2 ? 1024u : 512u));
    };
    auto put = [&](int k, int t, uint32_t set) {
        u32x4 v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = __builtin_amdgcn_perm(X[k][t >> 1][2 * i + 1], X[k][t >> 1][2 * i], t & 1 ? odd : even);
        lds_write16(planes, set + slot[k][t], v);
    };
    auto move_rows = [&](uint32_t set) {
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int j = 0; j < 8; ++j) take(k, j);
#pragma unroll
        for (int k = 0; k < U; ++k)
#pragma unroll
            for (int t = 0; t < 4; ++t) put(k, t, set);
    };

    float4v acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[a][b][v] = 0.f;

    // The matrix instructions are inline assembly: the compiler does not know when their results arrive, nor that an accumulator must not be
    // written right ahead of one, and so must find no cause to move an accumulator between them.
    //   settle: wait states, and every accumulator pinned to where the instructions left it until these are over.  (Without the pins the
    //   256 x 256 tile's epilogue had one block moved three instructions behind its last matrix instruction after an odd number
    //   of blocks of channels: 256 wrong outputs per wavefront.)
    //   Of the 64 accumulator blocks of that tile, which fill the accumulator half of the file to the last register, eight live in the other
    //   half, which has room (full, one block was parked at the top of the loop and put back right ahead of its first use).
    constexpr int TMA = TM * TN == 64 ? TM - 1 : TM;           // rows of blocks in the accumulator half
    auto multiply = [&](int tm, int tn, const u32x4 &a, const u32x4 &b) {
        if (tm < TMA) mfma16<BF16>(acc[tm][tn], a, b);
        else mfma16v<BF16>(acc[tm][tn], a, b);
    };
    auto settle = [&] {
        asm volatile("s_nop 15" ::: "memory");
#pragma unroll
        for (int a = 0; a < TM; ++a)
#pragma unroll
            for (int b = 0; b < TN; ++b) {
                if (a < TMA) asm volatile("" : "+a"(acc[a][b]));
                else asm volatile("" : "+v"(acc[a][b]));
            }
    };

    // lane t: byte offset of tap t in a plane (at most 64 taps)
    const int32_t tr = plane_quotient(lane, 1.f / (float)g.S);
    const int32_t tap_table = tr * (int32_t)g.tap_row + (lane - tr * g.S) * (int32_t)g.tap_col;
    uint32_t rd_off = 0;                                       // of the slice whose fragments are read next, its set of planes included
    u32x4 fa[2][TM], fb[2][TN];
    constexpr int NR = TM + TN, NM = TM * TN;
    auto lds_read = [&](int r, int set, uint32_t at) {         // at: the slice's ring position in bytes
        if (r < 1) fa[set][0] = lds_read16(planes, pos[0] + rd_off);
        else if (r < 1 + TN) tb.read(fb[set], smem, r - 1, at);
        else fa[set][r - TN] = lds_read16(planes, pos[r - TN] + rd_off);
    };

    using std::integral_constant;

    // prologue: the first block's rows into the first set of planes, slice 0's fragments into set 0
    NT_WAIT_VMCNT(kRing * ND);
    __syncthreads();
    move_rows(0);
    NT_WAIT_VMCNT((kRing - 1) * ND);
    __syncthreads();
    if constexpr (TRACE) {
        NT_WAIT_VMCNT(0);
        rd_off = (uint32_t)__builtin_amdgcn_readlane(tap_table, first_slice % RS);
#pragma unroll
        for (int r = 0; r < NR; ++r) lds_read(r, 0, 0);
        uint16_t *out = g.c.trace_out + l16 * 32 + grp * 8;
        if (g.c.trace_operand == 0 && wave_n == 0) {
#pragma unroll
            for (int t = 0; t < TM; ++t) __builtin_memcpy(out + (wave_m * (BM / 2) + t * 16) * 32, &fa[0][t], 16);
        } else if (g.c.trace_operand == 1 && wave_m == 0) {
#pragma unroll
            for (int t = 0; t < TN; ++t) __builtin_memcpy(out + (wave_n * (BN / 2) + t * 16) * 32, &fb[0][t], 16);
        }
        return;
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) lds_read(r, 0, 0);
    __builtin_amdgcn_sched_barrier(0);

    // Slice s sits at ring position s % 3.  One trip: the matrix instructions of slice s, whose fragments are in registers; behind
    // them the LDS reads of slice s + 1 into the other set of registers and the loads of slice s + 3 to where slice s was.  At the
    // top of a trip this wavefront's loads of slice s + 1 must have landed; those of slice s + 2 may be outstanding, and the next
    // block's rows where they were requested (behind their trip's other loads) one or two trips ago.  The barrier says that slice
    // s + 1 (in a block's fourth trip also the rows) is complete and that every wavefront holds its fragments of slice s.
    constexpr int LR = NM * 5 / 8;                             // trip's share in which the reads go out
    if constexpr (TAPS == 9) {
        // A block's trips are straight code: with one wavefront per SIMD every taken branch and every chain of scalar instructions
        // between two trips is time in which the matrix pipe idles (a loop over single trips took 950 cycles for 512 of matrix
        // instructions).  The next block's rows: loads in trip 0, out of the staging area in trip 3 and into the planes in trip 4
        // (one set of planes: trips 7 and 8, and slice 0's fragments once more behind a barrier), in the last block for nothing.
        constexpr int TAKE = SETS == 2 ? 3 : 7;
        int32_t tap[9];
#pragma unroll
        for (int t = 0; t < 9; ++t) tap[t] = __builtin_amdgcn_readlane(tap_table, t);
        uint32_t set = 0;
        auto block = [&](auto parity_c, int32_t b) {
            constexpr int PAR = decltype(parity_c)::value;
            const uint32_t other = SETS == 2 ? set ^ set_bytes : 0u;
            const char *const xp = x0 + (int64_t)(b + 1 < g.blocks ? b + 1 : b) * 32 * xs2;
            const uint32_t w_off = (uint32_t)b * (9u * kSliceK * 2u);
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                const int set_r = (PAR + t) & 1;
                if (t == 1 || t == 2) NT_WAIT_VMCNT(ND + NX);
                else NT_WAIT_VMCNT(ND);
                __syncthreads();
                rd_off = t == 8 ? other + (uint32_t)tap[0] : set + (uint32_t)tap[t == 8 ? 0 : t + 1];
#pragma unroll
                for (int idx = 0; idx < NM; ++idx) {
                    const int tm = idx / TN, tn = idx % TN;
                    multiply(tm, tn, fa[set_r][tm], fb[set_r][tn]);               // a lane holds one filter and 4 positions (see conv_store_rows16)
                    if (idx < LR)
#pragma unroll
                        for (int r = idx * NR / LR; r < (idx + 1) * NR / LR; ++r) lds_read(r, set_r ^ 1, (uint32_t)((t + 1) % 3) * SLICE);
                    if (idx < NM / 2)
#pragma unroll
                        for (int d = idx * ND / (NM / 2); d < (idx + 1) * ND / (NM / 2); ++d)
                            dma16_buf(rsrc, tb.voff[d], w_off + (uint32_t)(t + 3) * (kSliceK * 2), lds0 + (uint32_t)(t % 3) * SLICE + (uint32_t)((wave * ND + d) * 1024));
                    else if (t == 0)
#pragma unroll
                        for (int i = (idx - NM / 2) * NX / (NM / 2); i < (idx - NM / 2 + 1) * NX / (NM / 2); ++i) request_input(xp, i);
                    if (t == TAKE)
#pragma unroll
                        for (int i = idx * 8 * U / NM; i < (idx + 1) * 8 * U / NM; ++i) take(i / 8, i % 8);
                    if (t == TAKE + 1)
#pragma unroll
                        for (int i = idx * 4 * U / NM; i < (idx + 1) * 4 * U / NM; ++i) put(i / 4, i % 4, other);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (SETS == 1 && t == 8) {                     // (what this trip has read of the planes was being overwritten)
                    __syncthreads();
#pragma unroll
                    for (int i = 0; i < TM; ++i) fa[set_r ^ 1][i] = lds_read16(planes, pos[i] + rd_off);
                }
            }
            set = other;
        };
        int32_t b = 0;
        for (; b + 1 < g.blocks; b += 2) {
            block(integral_constant<int, 0>{}, b);
            block(integral_constant<int, 1>{}, b + 1);
            settle();
        }
        if (b < g.blocks) block(integral_constant<int, 0>{}, b);
    } else {
        int32_t tap = 0, left = g.blocks - 1;                  // left: blocks after this one
        uint32_t here = 0, set = 0, rq_off = 3 * kSliceK * 2;
        const char *xp = x0;
        auto step = [&](auto set_c) {
            constexpr int SET = decltype(set_c)::value;
            const uint32_t next = here + SLICE == 3 * SLICE ? 0u : here + SLICE;
            const int32_t at = left > 0 ? tap : -1;
            if (__builtin_expect((uint32_t)(at - 1) < 2u, 0)) NT_WAIT_VMCNT(ND + NX);
            else NT_WAIT_VMCNT(ND);
            __syncthreads();
            const bool wrap = tap + 1 == RS, fill = at == (SETS == 2 ? 3 : RS - 1);
            const uint32_t other = SETS == 2 ? set ^ set_bytes : 0u;
            const int32_t tap_next = wrap ? 0 : tap + 1;
            rd_off = (wrap ? other : set) + (uint32_t)__builtin_amdgcn_readlane(tap_table, tap_next);
#pragma unroll
            for (int idx = 0; idx < NM; ++idx) {
                const int tm = idx / TN, tn = idx % TN;
                multiply(tm, tn, fa[SET][tm], fb[SET][tn]);
                if (idx < LR)
#pragma unroll
                    for (int r = idx * NR / LR; r < (idx + 1) * NR / LR; ++r) lds_read(r, SET ^ 1, next);
#pragma unroll
                for (int d = idx * ND / NM; d < (idx + 1) * ND / NM; ++d) tb.issue_one_buf(d, rsrc, rq_off, lds0 + here, wave);
                __builtin_amdgcn_sched_barrier(0);
            }
            rq_off += kSliceK * 2;
            if (__builtin_expect(at == 0, 0)) {
                xp += 32 * xs2;
#pragma unroll
                for (int i = 0; i < NX; ++i) request_input(xp, i);
            }
            if (__builtin_expect(fill, 0)) {
                move_rows(other);
                if (SETS == 1) {                               // (what this trip has read of the planes was being overwritten)
                    __syncthreads();
#pragma unroll
                    for (int i = 0; i < TM; ++i) fa[SET ^ 1][i] = lds_read16(planes, pos[i] + rd_off);
                }
            }
            tap = tap_next;
            set = wrap ? other : set;
            left = wrap ? left - 1 : left;
            here = next;
        };
        for (int32_t s = 0; s + 1 < n_slices; s += 2) {
            step(integral_constant<int, 0>{});
            step(integral_constant<int, 1>{});
            settle();
        }
        if (n_slices & 1) step(integral_constant<int, 0>{});
    }
    settle();
    NT_WAIT_VMCNT(0);
    __syncthreads();
    asm volatile("s_nop 15" ::: "memory");

    const int64_t row_w = (int64_t)m0 + wave_m * (BM / 2), col_w = (int64_t)f0 + wave_n * (BN / 2);
    if (g.c.out_dtype == NT_F32) conv_store_rows16<BM, BN, NT_F32>(g.c, smem, wave, acc, 0, row_w, col_w, lane);
    else if (g.c.out_dtype == NT_F16) conv_store_rows16<BM, BN, NT_F16>(g.c, smem, wave, acc, 0, row_w, col_w, lane);
    else conv_store_rows16<BM, BN, NT_BF16>(g.c, smem, wave, acc, 0, row_w, col_w, lane);
}

// The grid: c.mt_a tiles of 32 TMA positions, then c.mt - c.mt_a of 32 TMB, each kind times c.nt filter tiles: whole rounds of
// programs (one per compute unit) cost their length, and two heights leave the last round little to wait for.
template <bool BF16, int TMA, int TMB, int TN, int U, int TAPS, bool TRACE = false>
__global__ __launch_bounds__(kThreads, 1) void conv_plane_kernel(const ConvPlaneArgs g)
{
    extern __shared__ __attribute__((aligned(1024))) char smem[];
    const uint32_t nt32 = (uint32_t)g.c.nt, mta = (uint32_t)g.c.mt_a, mtb = (uint32_t)g.c.mt - mta, n_a = mta * nt32;
    const uint32_t w = TRACE ? (uint32_t)g.c.trace_program : blockIdx.x;
    const bool first = w < n_a;                                // (uniform)
    // (the trace numbers programs tile of positions by tile of positions over both kinds)
    const uint32_t pid = TRACE ? (first ? w : w - n_a) : first ? program_of_workgroup_t<uint32_t>(w, mta, nt32) : program_of_workgroup_t<uint32_t>(w - n_a, mtb, nt32);
    const uint32_t ti = pid / nt32;
    const int32_t f0 = __builtin_amdgcn_readfirstlane((int)(pid - ti * nt32)) * 32 * TN, i = __builtin_amdgcn_readfirstlane((int)ti);
    if (first) conv_plane_program<BF16, TMA, TN, U, TAPS, TRACE>(g, smem, i * 32 * TMA, f0);
    else conv_plane_program<BF16, TMB, TN, U, TAPS, TRACE>(g, smem, (int32_t)mta * 32 * TMA + i * 32 * TMB, f0);
}

template <bool BF16, int TMA, int TMB, int TN, int U, int TAPS, bool TRACE = false>
nt_status launch_conv_plane_inst(const ConvPlaneArgs &a, hipStream_t s)
{
    auto kern = conv_plane_kernel<BF16, TMA, TMB, TN, U, TAPS, TRACE>;
    static DeviceOnce configured;
    if (!configured.done()) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 << 10);
        if (e != hipSuccess) return fail(NT_ERR_DEVICE, std::string("hipFuncSetAttribute: ") + hipGetErrorString(e));
        configured.set();
    }
    // (the output tile goes through the same LDS: 64 KB per 128 filters)
    const size_t lds = std::max<size_t>((size_t)kPlaneRing * 32 * TN * 64 + (size_t)U * 16 * 1024 + (size_t)plane_sets(U) * 4 * a.plane, (size_t)2 * 32 * TN * 256);
    hipLaunchKernelGGL(kern, dim3(TRACE ? 1u : (unsigned)(a.c.mt * a.c.nt)), dim3(kThreads), lds, s, a);
    return check_launch("conv_plane_kernel");
}

template <int TMA, int TMB, int TN, int U, int TAPS>
nt_status launch_conv_plane_t(const ConvPlaneArgs &a, bool bf16, hipStream_t s)
{
    return bf16 ? launch_conv_plane_inst<true, TMA, TMB, TN, U, TAPS>(a, s) : launch_conv_plane_inst<false, TMA, TMB, TN, U, TAPS>(a, s);
}

}  // namespace nt
