// Scaled dot-product attention, forward (Section 5.1: the paper's sdpa kernels implement the
// FlashAttention-2 algorithm): O = softmax(scale * Q K^T) V per (batch, head), head size 64.
//
// Arrangement: Q and O are tiled into blocks of 128 query rows (32 or 64 in launches that leave units empty, 256 where that costs no more
// rounds of them), one program per (batch, head, block); K and V are tiled into blocks of 64 keys, all of which every program visits in turn.
// Application (per program): a row reference M (close to the running row maximum), row sum l,
// accumulator O; per key block
//   S = Q K_j^T;  P = 2^(c S - M)  (c = scale * log2 e);  l += rowsum P;  O += P V_j;   finally O / l.
// M only has to stay within a band of the running maximum for this to be exact up to rounding:
// every term carries the same factor 2^-M, which cancels in O / l.  M is raised (and O, l scaled
// by 2^(M - M')) when a block holds a score more than 15 above it, which the row sum of that block
// reveals (2^15 is half the largest fp16 number), and it is set to the block's maximum at the first
// block that holds a score above -inf.  FlashAttention-2 raises M to the exact maximum at every block; keeping a lagging one
// removes the maximum search from all but a few blocks.
//
// Mapping onto the matrix cores: everything is computed transposed.  A wavefront owns 32 query
// rows.  S^T = K_j Q^T puts the query on the lane axis of the 32 x 32 MFMA result (lane % 32) and
// the keys on the register axis, so the row maximum and sum run over a lane's own registers plus
// one exchange with the other half-wavefront.  The fp32 P^T values a lane holds (keys in groups of
// four, interleaved between the half-wavefronts) are, packed to 16 bits, already a valid B
// operand of the second product O^T = V_j^T P^T if the matching A operand lists the keys in the
// same order: V_j sits in LDS as [key][d] and the transposing LDS read (ds_read_b64_tr_b16)
// delivers, for a lane's d, four consecutive keys at any position.  O^T again has the query on
// the lane axis, so rescaling by 2^(M - M') is a per-lane scalar.  Q fragments stay in registers.
// K_j and V_j travel straight into LDS (range-checked loads; through registers where strides do not allow it), K two blocks
// ahead and V one: rings of three and two blocks, 40 KB, and 126 registers (256 queries: 124) let sixteen wavefronts share a compute unit, which
// overlaps the exponentials of one with the MFMAs of another.  (Through registers, one block ahead, two blocks of each, three
// workgroups: 69.8 us against 63.8 at 4 x 48 heads x 1024 fp16, 90.5 / 81.2 at 4 x 16 x 2048; the next half block's scores
// computed between this one's exponentials measured no gain.)  What bounds it: per 64 keys and wavefront 16 MFMAs (512 cycles) and 80
// vector instructions (32 fma, 32 exponentials, 16 packs: 400 cycles), which run behind another wavefront's MFMAs (670 cycles for both, in a loop of just these, four
// wavefronts per SIMD) as long as there are four, and the clock, 1.65 to 1.75 GHz on real data: without the loads into LDS the same cycles
// take 53 us for 63, without LDS reads 46 (4 x 48 heads x 1024).  Blocks of 64 queries per wavefront with the MFMAs of one half behind the
// exponentials of the other measured the same 62 us at half the LDS reads.
#include "gemm_direct.h"
#include <type_traits>

namespace nt {

struct SdpaArgs {
    const uint16_t *Q, *K, *V;
    uint16_t *O;
    int64_t q_sb, q_sh, q_ss;        // strides (elements) of batch, head, sequence; the head dimension has stride 1
    int64_t k_sb, k_sh, k_ss;
    int64_t v_sb, v_sh, v_ss;
    int64_t o_sb, o_sh, o_ss;
    int32_t H, Sq, Sk;
    int32_t BH, nqb;                 // batch * heads, query blocks per head (the grid is their product)
    float scale_log2e;               // scale * log2(e): exponentials are taken in base 2
};

constexpr int kHeadDim = 64, kQBlock = 128, kKeyBlock = 64;
constexpr uint32_t kSdpaLds = 5 * kKeyBlock * kHeadDim * 2;        // LDS of one group of wavefronts: 40 KB

typedef short short4v_a __attribute__((ext_vector_type(4)));

typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2v __attribute__((ext_vector_type(2)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));

// two fp32 values -> one register of two 16-bit values, round to nearest even (v_cvt_pk_{f16,bf16}_f32)
template <bool BF16>
__device__ __forceinline__ uint32_t pack2(float a, float b)
{
    if constexpr (BF16) return __builtin_bit_cast(uint32_t, __builtin_convertvector(float2v{a, b}, bf16x2v));
    else return __builtin_bit_cast(uint32_t, half2v{(_Float16)a, (_Float16)b});
}

// acc + the two 16-bit values of w (v_dot2c_f32_{f16,bf16} against a pair of ones)
template <bool BF16>
__device__ __forceinline__ float add_pair(uint32_t w, float acc)
{
    if constexpr (BF16) return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2v, w), __builtin_bit_cast(bf16x2v, 0x3f803f80u), acc, false);
    else return __builtin_amdgcn_fdot2(__builtin_bit_cast(half2v, w), __builtin_bit_cast(half2v, 0x3c003c00u), acc, false);
}

template <bool BF16>
__device__ __forceinline__ float4v mfma16s(u32x4 a, u32x4 b, float4v c)
{
    if constexpr (BF16) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bhalf8, a), __builtin_bit_cast(bhalf8, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a), __builtin_bit_cast(half8, b), c, 0, 0, 0);
}

// SPLIT: the key blocks are dealt out to SPLIT groups of four wavefronts (group i: blocks i, i + SPLIT, ...), each with rings, a
// row reference, sums and an accumulator of its own; group 0 merges them at the end.
// AHEAD: rows that the range-checked loads do not take, one group: K and V through registers, one block ahead (loaded and
// written to LDS at the top of a block instead, bf16, rows of pitch 63: 4 x 48 heads x 1024 78 us against 68, 8 x 64 heads,
// 128 x 2048, 66 against 56; 2.1 M packed keys x 8 heads 32.0 ms in four groups, 29.1 so).
// NW: wavefronts per group, 32 queries each (4; 1 or 2 where 128 queries a workgroup leave units empty; 8 where 256 fill them).
// LONG (groups with some blocks to walk): how the wait for Q and the row sums are arranged, see below.
template <bool BF16, bool DMA, int SPLIT, int NW, bool LONG>
__global__ __launch_bounds__(64 * NW * SPLIT, NW >= 4 && (DMA || SPLIT > 1) ? 4 : 2) void sdpa_kernel(const SdpaArgs g)
{
    constexpr bool AHEAD = !DMA && SPLIT == 1;
    static_assert(NW == 4 || !AHEAD, "one group ahead of its arithmetic: four wavefronts");
    constexpr int QB = 32 * NW, PER = 8 / NW;                          // queries; 1 KB loads per wavefront and block
    constexpr uint32_t BLK = kKeyBlock * kHeadDim * 2;                 // bytes of one K or V block in LDS (8 KB)
    extern __shared__ __attribute__((aligned(1024))) char all_smem[];  // per group, rings of three K and two V blocks: [K0][K1][K2][V0][V1]
    const int lane = threadIdx.x & 63, group = __builtin_amdgcn_readfirstlane((int)threadIdx.x / (64 * NW)), tid = threadIdx.x % (64 * NW), wave = tid >> 6;
    char *smem = all_smem + group * (kSdpaLds);
    const int l32 = lane & 31, hi = lane >> 5;
    // Workgroup -> (batch * head, query block).  Consecutive workgroup indices go to different XCDs (index mod 8),
    // each with an L2 of its own; the query blocks of one head all read that head's K and V, so every group of
    // eight heads is dealt out one head per XCD instead of one head across all eight.
    const int w = blockIdx.x, nqb = g.nqb;
    int bh = w / nqb, qblk = w % nqb;
    if (w < (g.BH & ~7) * nqb) {
        const int j = w >> 3;
        bh = (j / nqb) * 8 + (w & 7);
        qblk = j % nqb;
    }
    const int b = bh / g.H, h = bh % g.H;
    const uint16_t *Qp = g.Q + b * g.q_sb + h * g.q_sh;
    const uint16_t *Kp = g.K + b * g.k_sb + h * g.k_sh;
    const uint16_t *Vp = g.V + b * g.v_sb + h * g.v_sh;
    uint16_t *Op = g.O + b * g.o_sb + h * g.o_sh;

    // ---- Q fragments (B operand of S^T = K Q^T: column = query l32, 8 consecutive d per k step)
    const int qrow = qblk * QB + wave * 32 + l32;
    const int qrow_c = qrow < g.Sq ? qrow : g.Sq - 1;
    u32x4 qf[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) __builtin_memcpy(&qf[ks], Qp + (int64_t)qrow_c * g.q_ss + 16 * ks + 8 * hi, 16);

    // ---- a K or V block into an LDS slot: 64 rows of 128 bytes, PER 1 KB loads per wavefront.  Lane l's 16 bytes land at
    // l * 16, so the swizzle is applied to the chunk it fetches.  Rows past Sk read as zero (the range check).
    const int nblk = (g.Sk + kKeyBlock - 1) / kKeyBlock;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem;
    const int swave = __builtin_amdgcn_readfirstlane(wave);
    int ld_row[PER], k_ch[PER], v_ch[PER];                                   // this lane's row and 16-byte chunk of K and of V
    uint32_t k_off[PER], v_off[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        ld_row[u] = (wave * PER + u) * 8 + (lane >> 3);
        k_ch[u] = (lane & 7) ^ ((ld_row[u] ^ (ld_row[u] >> 3)) & 7);
        v_ch[u] = (lane & 7) ^ (((ld_row[u] >> 1) & 1) << 2);
        k_off[u] = ((uint32_t)ld_row[u] * (uint32_t)g.k_ss + (uint32_t)(k_ch[u] * 8)) * 2u;
        v_off[u] = ((uint32_t)ld_row[u] * (uint32_t)g.v_ss + (uint32_t)(v_ch[u] * 8)) * 2u;
    }
    const u32x4 k_rsrc = make_rsrc(Kp, ((int64_t)(g.Sk - 1) * g.k_ss + kHeadDim) * 2), v_rsrc = make_rsrc(Vp, ((int64_t)(g.Sk - 1) * g.v_ss + kHeadDim) * 2);
    auto request = [&](int kb, uint32_t slot, const uint16_t *p, int64_t ss, const int (&ch)[PER], u32x4 rsrc, const uint32_t (&off)[PER]) {
        if constexpr (DMA) {
            // (blocks past the last: an offset beyond the range, no traffic; the count of outstanding loads stays the same)
            const uint32_t at = kb < nblk ? (uint32_t)kb * (uint32_t)(kKeyBlock * 2) * (uint32_t)ss : 0x80000000u;
#pragma unroll
            for (int u = 0; u < PER; ++u) dma16_buf(rsrc, off[u], at, lds0 + slot + (uint32_t)((swave * PER + u) * 1024));
        } else if (kb < nblk) {
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const int key = kb * kKeyBlock + ld_row[u];
                u32x4 v{0, 0, 0, 0};
                if (key < g.Sk) __builtin_memcpy(&v, p + (int64_t)key * ss + ch[u] * 8, 16);
                lds_write16(smem, slot + (uint32_t)((wave * PER + u) * 1024 + lane * 16), v);
            }
        }
    };
    auto request_k = [&](int kb, uint32_t slot) { request(kb, slot, Kp, g.k_ss, k_ch, k_rsrc, k_off); };
    auto request_v = [&](int kb, uint32_t slot) { request(kb, 3 * BLK + slot, Vp, g.v_ss, v_ch, v_rsrc, v_off); };

    // Row sums.  v_dot2c holds up the matrix pipe (a loop of 16 matrix instructions of 32 cycles, 2 dot2 behind each: 830 cycles, without
    // 515; the exponentials, fma and packs of a block run behind matrix instructions of other wavefronts, the dots only between
    // them), so LONG takes the sums on the matrix pipe: four 16 x 16 x 32 instructions a block against an operand of ones and zeros.
    // With few blocks to walk their chain is the longer one.  Lane l of a 16 x 16 x 32 matrix instruction supplies row l % 16 and
    // k 8 (l / 16) .. + 7 of it; of the weights (B operand) lanes c and c + 32 hold query c, lanes c + 16 and c + 48 query c + 16.
    // Rows 4 i .. 4 i + 3 with i even take the former, the others the latter: lane l then receives the sum of query l % 32.
    const uint32_t one_pair = ((lane >> 4) & 1) == ((lane >> 2) & 1) ? (BF16 ? 0x3f803f80u : 0x3c003c00u) : 0u;
    const u32x4 ones{one_pair, one_pair, one_pair, one_pair};

    // ---- per-lane LDS read addresses
    // K fragment (A operand, row = key l32 of a 32-key half, chunk 2 ks + hi, swizzled like the write)
    // Key row 32 + l32 has the swizzle of row l32 with bit 2 flipped, so its chunk for k step ks sits where row
    // l32's chunk for k step ks ^ 2 does: four addresses serve both halves, everything else is an immediate offset.
    uint32_t k_rd[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) k_rd[ks] = (uint32_t)(l32 * 128 + (((hi + 2 * ks) ^ ((l32 ^ (l32 >> 3)) & 7)) << 4));
    // V^T fragment through the transposing read: 16-lane group gq covers d = 16 (gq & 1) .. + 15 and
    // keys 4 (gq >> 1) .. + 3 of an 8-key part; lane i of the group points at key i / 4, columns 4 (i % 4) .. + 3
    const int gq = lane >> 4, li = lane & 15;
    const int v_key = 4 * (gq >> 1) + (li >> 2);                       // + jb * 32 + 16 * s2 + 8 * part
    const int v_c8 = 4 * (gq & 1) + (li & 3);                          // 8-byte chunk within the 32-d block; + 8 * db
    // the swizzle flips bit 3 of the 8-byte chunk index on keys with bit 1 set (key offsets added later are multiples of 8)
    uint32_t v_rd[2];
#pragma unroll
    for (int db = 0; db < 2; ++db)
        v_rd[db] = (uint32_t)(v_key * 128) + ((((uint32_t)(v_c8 + 8 * db)) ^ (uint32_t)(((v_key >> 1) & 1) << 3)) << 3);

    float16v ot[2];
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int v = 0; v < 16; ++v) ot[db][v] = 0.f;
    // Row reference M (base-2 units of the scaled scores; -inf: no score above -inf yet) and row sum.  While a row has no reference,
    // its blocks are weighed against 0, which gives the weight 0 that scores of -inf have (against -inf it would be -inf + inf).
    float m_ref = -INFINITY, l_run = 0.f;
    bool pending = true;                                               // wavefront-uniform: some row has no reference

    if constexpr (!AHEAD) {
        request_k(group, 0);
        request_v(group, 0);
        // LONG: Q is waited for here, with the first blocks.  Its loads are ordinary ones; left to the compiler, the last two are waited for
        // at their first use inside the loop, by a wait for everything outstanding, the blocks just requested among it: 192 heads,
        // 1024 x 1024 66.6 us for 64.3.  With few blocks to walk, the start is what counts, and this costs 0.1 us.
        if constexpr (LONG) {
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) asm volatile("" : "+v"(qf[ks]));
        }
        request_k(group + SPLIT, BLK);
    }
    // one key block: K in the slot at LDS offset `slot`, V in the slot at `vslot` behind the K ring
    auto block = [&](const uint32_t slot, const uint32_t vslot, const int kb) __attribute__((always_inline)) {
        // ---- S^T = K Q^T: st[jb][v] <-> key jb * 32 + 8 (v / 4) + 4 hi + v % 4, query l32
        float16v st[2];
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
#pragma unroll
            for (int v = 0; v < 16; ++v) st[jb][v] = 0.f;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const u32x4 kf = lds_read16(smem, k_rd[jb ? (ks ^ 2) : ks] + slot + (uint32_t)(jb * 4096));
                st[jb] = mfma32<BF16>(kf, qf[ks], st[jb]);
            }
        }
        // ---- keys past Sk (last block only) get weight 0: their scaled score becomes -inf
        const int key_base = kb * kKeyBlock;
        if (key_base + kKeyBlock > g.Sk) {                                // wavefront-uniform
            const float out = g.scale_log2e >= 0.f ? -INFINITY : INFINITY;
#pragma unroll
            for (int jb = 0; jb < 2; ++jb)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (key_base + jb * 32 + 8 * (v / 4) + 4 * hi + (v % 4) >= g.Sk) st[jb][v] = out;
        }
        // ---- P^T = 2^(c S^T - M), packed to 16 bits, and its row sum (LONG: over all 64 keys; else this lane's, the halves are added at the end)
        float rs;
        u32x4 pk[2][2];
        auto exponentials = [&](const float m) {
#pragma unroll
            for (int jb = 0; jb < 2; ++jb)
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(st[jb][8 * s2 + 2 * j], g.scale_log2e, -m));
                        const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(st[jb][8 * s2 + 2 * j + 1], g.scale_log2e, -m));
                        pk[jb][s2][j] = pack2<BF16>(p0, p1);
                    }
        };
        auto own_sum = [&] {                                             // of this lane's keys
            float t = 0.f;
#pragma unroll
            for (int jb = 0; jb < 2; ++jb)
#pragma unroll
                for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
                    for (int j = 0; j < 4; ++j) t = add_pair<BF16>(pk[jb][s2][j], t);
            return t;
        };
        bool accept = false;
        if (!pending) {
            exponentials(m_ref);
            if constexpr (LONG) {
                float4v sum{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int jb = 0; jb < 2; ++jb)
#pragma unroll
                    for (int s2 = 0; s2 < 2; ++s2) sum = mfma16s<BF16>(ones, pk[jb][s2], sum);
                rs = sum[0];
            } else {
                rs = own_sum();
            }
            accept = __all(rs < 32768.f);                                // no weight beyond 2^15: the reference is close enough
        }
        if (!accept) {                                                   // wavefront-uniform: a row without reference, or a score far above M
            float mx = st[0][0] * g.scale_log2e;
#pragma unroll
            for (int jb = 0; jb < 2; ++jb)
#pragma unroll
                for (int v = 0; v < 16; ++v) mx = fmaxf(mx, st[jb][v] * g.scale_log2e);
            mx = fmaxf(mx, __shfl_xor(mx, 32, 64));                      // block maximum of the scaled scores
            const float m_new = fmaxf(m_ref, mx);                        // M only rises
            const float m_use = m_new == -INFINITY ? 0.f : m_new;
            const float alpha = __builtin_amdgcn_exp2f(m_ref - m_use);
            exponentials(m_use);
            rs = own_sum();                                              // (not by matrix instructions: a row's NaN stays its own)
            if constexpr (LONG) rs += __shfl_xor(rs, 32, 64);
            l_run *= alpha;
#pragma unroll
            for (int db = 0; db < 2; ++db)
#pragma unroll
                for (int v = 0; v < 16; ++v) ot[db][v] *= alpha;
            m_ref = m_new;
            pending = __any(m_new == -INFINITY);
        }
        l_run += rs;
        // ---- O^T += V^T P^T: k step (jb, s2) lists its 16 keys as jb*32 + 16 s2 + 8 part + 4 hi + 0..3
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
                for (int db = 0; db < 2; ++db) {
                    u32x2 part[2];
#pragma unroll
                    for (int pt = 0; pt < 2; ++pt) {
                        const uint32_t addr = v_rd[db] + vslot + (3 * BLK + (uint32_t)((jb * 32 + 16 * s2 + 8 * pt) * 128));
                        typedef short4v_a __attribute__((address_space(3))) * lds_s4;
                        const short4v_a t = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(smem + addr));
                        part[pt] = __builtin_bit_cast(u32x2, t);
                    }
                    const u32x2 p0 = part[0], p1 = part[1];
                    ot[db] = mfma32<BF16>(u32x4{p0[0], p0[1], p1[0], p1[1]}, pk[jb][s2], ot[db]);
                }
    };
    if constexpr (AHEAD) {
        // the next block's loads are in flight during this one's arithmetic and go to the other of two slots each behind it
        u32x4 k_st[2], v_st[2];
        auto fetch = [&](int kb) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int key = kb * kKeyBlock + ld_row[u];
                k_st[u] = v_st[u] = u32x4{0, 0, 0, 0};
                if (key < g.Sk) {
                    __builtin_memcpy(&k_st[u], Kp + (int64_t)key * g.k_ss + k_ch[u] * 8, 16);
                    __builtin_memcpy(&v_st[u], Vp + (int64_t)key * g.v_ss + v_ch[u] * 8, 16);
                }
            }
        };
        auto stash = [&](uint32_t at) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                lds_write16(smem, at + (uint32_t)((wave * 2 + u) * 1024 + lane * 16), k_st[u]);
                lds_write16(smem, 3 * BLK + at + (uint32_t)((wave * 2 + u) * 1024 + lane * 16), v_st[u]);
            }
        };
        auto step = [&](auto cur, int kb) {                               // (a compile-time slot: every LDS address is base + immediate)
            constexpr uint32_t at = decltype(cur)::value;
            if (kb + 1 < nblk) fetch(kb + 1);
            block(at, at, kb);
            if (kb + 1 < nblk) stash(at ^ BLK);
            __syncthreads();
        };
        fetch(0);
        stash(0);
        __syncthreads();
        for (int kb = 0; kb < nblk; kb += 2) {
            step(std::integral_constant<uint32_t, 0>{}, kb);
            if (kb + 1 < nblk) step(std::integral_constant<uint32_t, BLK>{}, kb + 1);
        }
    } else {
        // At the top of block kb this wavefront's part of K and V has landed (the loads of K's next block may be in flight); the
        // barrier says that all parts have, and that everybody is done with block kb - 1: its V slot takes V's next block, its K
        // slot K's next but one.
        uint32_t slot = 0, ahead = 2 * BLK, vslot = 0;
        for (int kb = group; kb - group < nblk; kb += SPLIT) {               // (the same number of passes, and barriers, in every group)
            if constexpr (DMA) NT_WAIT_VMCNT(PER);
            __syncthreads();
            request_v(kb + SPLIT, vslot ^ BLK);
            request_k(kb + 2 * SPLIT, ahead);
            if (SPLIT == 1 || kb < nblk) block(slot, vslot, kb);
            ahead = slot;
            vslot ^= BLK;
            slot = slot == 2 * BLK ? 0 : slot + BLK;
        }
    }
    if constexpr (DMA) NT_WAIT_VMCNT(0);                                  // (no load of this workgroup may land in its LDS after it has ended)

    if constexpr (SPLIT > 1) {
        // the other groups' (reference, sum, accumulator) through LDS, 34 floats per lane, lane by lane the same (query, d)
        __syncthreads();                                                  // (everybody's loads have landed, everybody's reads are done)
        float *ex = reinterpret_cast<float *>(all_smem);
        if (group > 0) {
            float *e = ex + (group - 1) * (34 * 64 * NW) + tid;
            e[0] = m_ref;                                                 // (-inf, a group whose keys have no weight: 0 below)
            e[64 * NW] = l_run;
#pragma unroll
            for (int i = 0; i < 32; ++i) e[(2 + i) * 64 * NW] = ot[i >> 4][i & 15];
        }
        __syncthreads();
        if (group > 0) return;
        float top = m_ref;
#pragma unroll
        for (int i = 0; i < SPLIT - 1; ++i) top = fmaxf(top, ex[i * (34 * 64 * NW) + tid]);
        const float own = __builtin_amdgcn_exp2f(m_ref - top);
        l_run *= own;
#pragma unroll
        for (int v = 0; v < 32; ++v) ot[v >> 4][v & 15] *= own;
#pragma unroll
        for (int i = 0; i < SPLIT - 1; ++i) {
            const float *e = ex + i * (34 * 64 * NW) + tid;
            const float c = __builtin_amdgcn_exp2f(e[0] - top);
            l_run = __builtin_fmaf(e[64 * NW], c, l_run);
#pragma unroll
            for (int v = 0; v < 32; ++v) ot[v >> 4][v & 15] = __builtin_fmaf(e[(2 + v) * 64 * NW], c, ot[v >> 4][v & 15]);
        }
    }

    // ---- O = O^T / l, stored along d: after the half-wavefronts trade register groups a lane owns
    // d = 32 db + 16 hi .. + 15 of its query row
    const float l_tot = LONG ? l_run : l_run + __shfl_xor(l_run, 32, 64);
    const float inv = 1.0f / l_tot;
#pragma unroll
    for (int db = 0; db < 2; ++db) {
#pragma unroll
        for (int v = 0; v < 16; ++v) ot[db][v] *= inv;
        uint32_t o[16];
        gather_row16(ot[db], o);                                       // (all lanes take part)
        if (qrow < g.Sq) {
            uint16_t *dst = Op + (int64_t)qrow * g.o_ss + 32 * db + 16 * hi;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const u32x4 w{pack2<BF16>(__builtin_bit_cast(float, o[8 * i]), __builtin_bit_cast(float, o[8 * i + 1])),
                              pack2<BF16>(__builtin_bit_cast(float, o[8 * i + 2]), __builtin_bit_cast(float, o[8 * i + 3])),
                              pack2<BF16>(__builtin_bit_cast(float, o[8 * i + 4]), __builtin_bit_cast(float, o[8 * i + 5])),
                              pack2<BF16>(__builtin_bit_cast(float, o[8 * i + 6]), __builtin_bit_cast(float, o[8 * i + 7]))};
                __builtin_memcpy(dst + 8 * i, &w, 16);
            }
        }
    }
}

// ---- few query rows (a decoding step: one query per head against a cache of keys)
// Bound by reading K and V once; of the 128 query rows of sdpa_kernel's block all but a few would be padding, and its one
// workgroup per head walks the keys in turn.  Here one workgroup of 16 wavefronts (4 or 8: short sequences, or heads
// enough to fill the chip) per (head, query) deals the keys out to its
// wavefronts, 32 at a time: eight lanes hold one key's 64 elements (a load instruction covers 8 keys, 1 KB), four keys per lane
// group in flight and the next four behind them.  Scores, weights and sums stay in fp32 (a lane group keeps a maximum and a
// sum of its own: no exchange in the loop but the score's, three adds across eight lanes); the groups' results are brought to a
// common maximum at the end, first within a wavefront, then through LDS.
// Measured, bf16, 4 x 48 heads x 2047 keys (100 MB): 33.9 us with sdpa_kernel, 19.1 here (5.3 TB/s, a large copy's rate); 8 heads x 2048 keys 30.2 and 10.7.
constexpr int kDecodeKeys = 4;                                // keys per lane group and batch

template <bool BF16>
__device__ __forceinline__ void unpack8_f32(u32x4 v, float (&f)[8])
{
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint32_t w = v[q];
        if constexpr (BF16) {
            f[2 * q] = __builtin_bit_cast(float, w << 16);
            f[2 * q + 1] = __builtin_bit_cast(float, w & 0xffff0000u);
        } else {
            f[2 * q] = (float)__builtin_bit_cast(_Float16, (uint16_t)(w & 0xffffu));
            f[2 * q + 1] = (float)__builtin_bit_cast(_Float16, (uint16_t)(w >> 16));
        }
    }
}

// sum over the eight lanes of a group (lanes 8 i .. 8 i + 7), in all of them
__device__ __forceinline__ float sum_of_eight(float v)
{
    auto from = [](float x, auto ctrl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    v += from(v, std::integral_constant<int, 0xB1>{});        // lane ^ 1
    v += from(v, std::integral_constant<int, 0x4E>{});        // lane ^ 2
    v += from(v, std::integral_constant<int, 0x141>{});       // mirrored within eight: the other four's sum
    return v;
}

template <bool BF16, int kDecodeWaves>
__global__ __launch_bounds__(64 * kDecodeWaves) void sdpa_decode_kernel(const SdpaArgs g)
{
    constexpr int BATCH = 8 * kDecodeKeys;                     // keys per wavefront and batch
    __shared__ float red_o[kDecodeWaves][kHeadDim], red_m[kDecodeWaves], red_l[kDecodeWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int sub = lane & 7, slot = lane >> 3;
    // (all queries of a head on one XCD, see sdpa_kernel; nqb: the queries)
    const int w = blockIdx.x, nq = g.nqb;
    int bh = w / nq, qi = w % nq;
    if (w < (g.BH & ~7) * nq) {
        const int j = w >> 3;
        bh = (j / nq) * 8 + (w & 7);
        qi = j % nq;
    }
    const int b = bh / g.H, h = bh % g.H;
    const uint16_t *Kp = g.K + b * g.k_sb + h * g.k_sh + 8 * sub;
    const uint16_t *Vp = g.V + b * g.v_sb + h * g.v_sh + 8 * sub;
    float q[8];
    {
        u32x4 raw;
        __builtin_memcpy(&raw, g.Q + b * g.q_sb + h * g.q_sh + (int64_t)qi * g.q_ss + 8 * sub, 16);
        unpack8_f32<BF16>(raw, q);
    }
    float m = -INFINITY, l = 0.f, o[8];                        // this lane group's maximum (base-2 units), sum and output
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = 0.f;

    struct Keys { u32x4 k[kDecodeKeys], v[kDecodeKeys]; };
    auto fetch = [&](Keys &t, int batch) {
#pragma unroll
        for (int u = 0; u < kDecodeKeys; ++u) {
            const int key = batch * BATCH + u * 8 + slot;
            const int64_t kc = key < g.Sk ? key : g.Sk - 1;
            __builtin_memcpy(&t.k[u], Kp + kc * g.k_ss, 16);
            __builtin_memcpy(&t.v[u], Vp + kc * g.v_ss, 16);
        }
    };
    auto use = [&](const Keys &t, int batch) {
        float s[kDecodeKeys], top = m;
#pragma unroll
        for (int u = 0; u < kDecodeKeys; ++u) {
            float k[8], dot = 0.f;
            unpack8_f32<BF16>(t.k[u], k);
#pragma unroll
            for (int e = 0; e < 8; ++e) dot = __builtin_fmaf(q[e], k[e], dot);
            dot = sum_of_eight(dot) * g.scale_log2e;
            s[u] = batch * BATCH + u * 8 + slot < g.Sk ? dot : -INFINITY;
            top = fmaxf(top, s[u]);
        }
        const float ref = top == -INFINITY ? 0.f : top;        // (nothing to weigh yet: weights 0, not 0 / 0)
        const float alpha = __builtin_amdgcn_exp2f(m - ref);
        m = top;
        l *= alpha;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] *= alpha;
#pragma unroll
        for (int u = 0; u < kDecodeKeys; ++u) {
            const float p = __builtin_amdgcn_exp2f(s[u] - ref);
            float v[8];
            unpack8_f32<BF16>(t.v[u], v);
            l += p;
            // (a key that does not exist repeats the last one with weight 0: an infinity there must not become 0 * inf)
            const bool live = batch * BATCH + u * 8 + slot < g.Sk;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = __builtin_fmaf(p, live ? v[e] : 0.f, o[e]);
        }
    };
    const int batches = (g.Sk + BATCH - 1) / BATCH;
    Keys t[2];
    if (wave < batches) fetch(t[0], wave);
    for (int n = wave; n < batches; n += 2 * kDecodeWaves) {
        if (n + kDecodeWaves < batches) fetch(t[1], n + kDecodeWaves);
        use(t[0], n);
        if (n + 2 * kDecodeWaves < batches) fetch(t[0], n + 2 * kDecodeWaves);
        if (n + kDecodeWaves < batches) use(t[1], n + kDecodeWaves);
    }
    // the wavefront's eight groups to a common maximum, summed
    float top = m;
#pragma unroll
    for (int x = 8; x < 64; x <<= 1) top = fmaxf(top, __shfl_xor(top, x, 64));
    const float ref = top == -INFINITY ? 0.f : top;
    const float c = __builtin_amdgcn_exp2f(m - ref);
    l *= c;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] *= c;
#pragma unroll
    for (int x = 8; x < 64; x <<= 1) {
        l += __shfl_xor(l, x, 64);
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] += __shfl_xor(o[e], x, 64);
    }
    if (lane < 8) {
#pragma unroll
        for (int e = 0; e < 8; ++e) red_o[wave][8 * lane + e] = o[e];
        if (lane == 0) { red_m[wave] = top; red_l[wave] = l; }
    }
    __syncthreads();
    // ... and the wavefronts': thread d has element d of the output row
    if (tid < kHeadDim) {
        float mx = red_m[0];
#pragma unroll
        for (int i = 1; i < kDecodeWaves; ++i) mx = fmaxf(mx, red_m[i]);
        const float r = mx == -INFINITY ? 0.f : mx;
        float lsum = 0.f, osum = 0.f;
#pragma unroll
        for (int i = 0; i < kDecodeWaves; ++i) {
            const float f = __builtin_amdgcn_exp2f(red_m[i] - r);
            lsum = __builtin_fmaf(red_l[i], f, lsum);
            osum = __builtin_fmaf(red_o[i][tid], f, osum);
        }
        const float v = osum / lsum;
        g.O[b * g.o_sb + h * g.o_sh + (int64_t)qi * g.o_ss + tid] = BF16 ? f32_to_bf16_rne(v) : f32_to_f16_rne(v);
    }
}

static thread_local nt_sdpa_plan t_plan;
const nt_sdpa_plan &last_sdpa_plan() { return t_plan; }

template <bool BF16, bool DMA, int SPLIT, int NW, bool LONG>
static nt_status launch_sdpa_inst(const SdpaArgs &k, int64_t programs, hipStream_t s)
{
    auto kern = sdpa_kernel<BF16, DMA, SPLIT, NW, LONG>;
    static DeviceOnce configured;
    if (!configured.done()) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)(SPLIT * kSdpaLds));
        if (e != hipSuccess) return fail(NT_ERR_DEVICE, std::string("hipFuncSetAttribute: ") + hipGetErrorString(e));
        configured.set();
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)programs), dim3(64 * NW * SPLIT), SPLIT * kSdpaLds, s, k);
    t_plan = nt_sdpa_plan{32 * NW, SPLIT, NW * SPLIT, LONG ? 1 : 0, DMA ? 1 : 0};
    return check_launch("sdpa_kernel");
}

template <bool BF16, bool DMA, int SPLIT, int NW>
static nt_status launch_sdpa_length(const SdpaArgs &k, int64_t programs, hipStream_t s)
{
    // Blocks per group from which on LONG is ahead (us, without / with): one wavefront a group 5 (17 blocks in four groups 11.0 / 10.2,
    // 16 8.5 / 8.7, 7 6.3 / 6.5), else 3 (12 blocks in four groups 9.4 / 8.9, 10 in two 8.8 / 8.2, 3 in one 9.0 / 8.5, 2 in one 6.4 / 6.8;
    // 2 with more programs than are resident from the start 12.8 / 12.3).
    // (rows through registers go by the same rule, and give the same bits)
    // By the rules of launch_sdpa some kernels only ever walk more blocks than that, or fewer: four groups of more than one wavefront have twelve to share
    // at least, two of four seven; two groups of one wavefront have six at most, one group of one or two wavefronts a single one.
    if constexpr ((SPLIT == 4 && NW > 1) || (SPLIT == 2 && NW == 4)) {
        return launch_sdpa_inst<BF16, DMA, SPLIT, NW, true>(k, programs, s);
    } else if constexpr ((SPLIT == 2 && NW == 1) || (SPLIT == 1 && NW < 4)) {
        return launch_sdpa_inst<BF16, DMA, SPLIT, NW, false>(k, programs, s);
    } else {
        const int64_t blocks = (((int64_t)k.Sk + kKeyBlock - 1) / kKeyBlock + SPLIT - 1) / SPLIT;
        if (blocks >= (NW == 1 ? 5 : programs > 1024 ? 2 : 3)) return launch_sdpa_inst<BF16, DMA, SPLIT, NW, true>(k, programs, s);
        return launch_sdpa_inst<BF16, DMA, SPLIT, NW, false>(k, programs, s);
    }
}

template <bool BF16, bool DMA, int NW>
static nt_status launch_sdpa_groups(const SdpaArgs &k, int64_t programs, int split, hipStream_t s)
{
    if (split == 4) return launch_sdpa_length<BF16, DMA, 4, NW>(k, programs, s);
    if constexpr (DMA || NW < 4)
        if (split == 2) return launch_sdpa_length<BF16, DMA, 2, NW>(k, programs, s);
    if constexpr (DMA || NW == 4) return launch_sdpa_length<BF16, DMA, 1, NW>(k, programs, s);
    return fail(NT_ERR_UNSUPPORTED, "no attention kernel for this split");
}

template <bool BF16, bool DMA>
static nt_status launch_sdpa_split(const SdpaArgs &k, int64_t programs, int split, int nw, hipStream_t s)
{
    if constexpr (DMA)
        if (nw == 8) return launch_sdpa_inst<BF16, true, 1, 8, true>(k, programs, s);
    if (nw == 1) return launch_sdpa_groups<BF16, DMA, 1>(k, programs, split, s);
    if (nw == 2) return launch_sdpa_groups<BF16, DMA, 2>(k, programs, split, s);
    return launch_sdpa_groups<BF16, DMA, 4>(k, programs, split, s);
}

// One workgroup per query pays while they do not queue up for the units with the same keys (bf16, us, sdpa_kernel / this one):
// 192 heads x 1 query x 2047 keys 33.9 / 19.1, x 2 34.5 / 29.2, x 4 35.4 / 39.3; 8 heads x 16 x 2047 30.6 / 11.0, x 32 30.6 / 12.0.
static bool few_queries(int64_t heads, int64_t queries)
{
    return heads <= 0x3fffffff && (queries == 1 || (queries == 2 && heads <= 256) || (queries <= 32 && heads * queries <= 256));
}

nt_status launch_sdpa(const SdpaArgs &a, int64_t batch, bool bf16, void *stream)
{
    if (batch <= 0 || a.H <= 0 || a.Sq <= 0) return NT_OK;
    const int64_t per_entry = a.H * (((int64_t)a.Sq + kQBlock - 1) / kQBlock);
    if (batch * per_entry > kMaxWorkgroups && batch > 1 && per_entry <= kMaxWorkgroups) {
        // more programs than one launch holds (few queries: as many, one workgroup per head): in several
        const int64_t most = kMaxWorkgroups / per_entry;
        for (int64_t b0 = 0; b0 < batch; b0 += most) {
            SdpaArgs part = a;
            part.Q += b0 * a.q_sb; part.K += b0 * a.k_sb; part.V += b0 * a.v_sb; part.O += b0 * a.o_sb;
            const nt_status st = launch_sdpa(part, std::min(most, batch - b0), bf16, stream);
            if (st != NT_OK) return st;
        }
        return NT_OK;
    }
    if (few_queries(batch * a.H, a.Sq)) {
        SdpaArgs k = a;
        k.BH = (int32_t)(batch * a.H);
        k.nqb = a.Sq;
        const int64_t programs = batch * a.H * a.Sq;
        // A workgroup of 16 wavefronts has a unit to itself (122 registers): beyond 256 programs they queue up for the units, and with few
        // keys most of its wavefronts have none.  4 / 8 / 16 wavefronts (us, f16, in graph replays): 560 heads x 130 keys 7.1 / 8.3 / 11.3,
        // x 488 15.6 / 14.6 / 18.0, 310 x 310 8.2 / 8.3 / 9.8, x 2047 35.6 / 36.5 / 38.0; 252 x 310 6.6 / 6.8 / 6.7, x 1338 15.7 / 15.9 / 15.9;
        // 54 x 225 4.1 / 4.1 / 4.5, x 600 6.2 / 5.6 / 5.9, x 902 8.4 / 7.8 / 7.1, x 4096 24.3 / 20.1 / 19.1.
        const int waves = programs > 256 ? (programs > 512 && a.Sk > 384 ? 8 : 4) : a.Sk <= (programs > 160 ? 640 : 256) ? 4 : a.Sk <= 640 ? 8 : 16;
        const dim3 grid((unsigned)programs), block(64 * waves);
        auto launch = [&](auto kern) { hipLaunchKernelGGL(kern, grid, block, 0, (hipStream_t)stream, k); };
        if (waves == 4) bf16 ? launch(sdpa_decode_kernel<true, 4>) : launch(sdpa_decode_kernel<false, 4>);
        else if (waves == 8) bf16 ? launch(sdpa_decode_kernel<true, 8>) : launch(sdpa_decode_kernel<false, 8>);
        else bf16 ? launch(sdpa_decode_kernel<true, 16>) : launch(sdpa_decode_kernel<false, 16>);
        t_plan = nt_sdpa_plan{1, 1, waves, 0, 0};
        return check_launch("sdpa_decode_kernel");
    }
    const int64_t bh = batch * a.H;
    if (batch * per_entry > kMaxWorkgroups) return fail(NT_ERR_UNSUPPORTED, "heads * query blocks exceeds 2^24 - 1");
    SdpaArgs k = a;
    k.BH = (int32_t)bh;
    // (rows that do not overlap, and offsets that fit the range-checked loads: else through registers)
    const int nblk = (int)(((int64_t)a.Sk + kKeyBlock - 1) / kKeyBlock);
    auto streams = [&](int64_t ss) { return ss >= kHeadDim && ((int64_t)a.Sk + 10 * kKeyBlock) * ss * 2 < (1LL << 31); };
    const bool dma = streams(a.k_ss) && streams(a.v_ss);
    const bool far = a.k_ss >= kHeadDim && a.v_ss >= kHeadDim && !dma;     // (keys spread over 2 GB and more: every load a long way off)
    // A unit holds four groups of four wavefronts: launches with fewer programs than that split the keys, where there are enough
    // blocks to pay for the larger workgroup and the merge.  Measured (us, one group / split): 160 programs x 24 blocks 26.7 /
    // 19.3, 90 x 32 34.1 / 23.1, 8 x 32 27.0 / 21.0, 144 x 13 15.8 / 14.0, 288 x 32 46.5 (as it was) / 36.3, 228 x 11 15.0 / 13.5,
    // 208 x 7 11.2 / 10.6; 256 x 8 11.4 / 12.2 in four groups, 330 x 7 14.1 / 15.3.
    // Launches that leave units without a program take narrower blocks of queries, as long as one round of the units holds them:
    // the keys are read more often, but sixteen wavefronts on one unit and none on the next cost more.  128 queries / best (us, in
    // graph replays): 64 queries, four groups, 2 x 10 heads, 611 x 1102 16.8 / 13.2, two groups, 13 heads, 824 x 248 6.9 / 5.9;
    // 32 queries, four groups, 2 x 8 heads, 384 x 1216 15.7 / 10.0, 10 x 2 heads, 152 x 512 9.2 / 6.5, two groups, 37 heads, 175 x
    // 384 8.1 / 6.5.  Beyond a round they lose: 26 heads, 896 x 984 on 364 blocks of 64 21.8 for 16.1.  Four groups of 32 from seven
    // blocks of keys on (6: 6.3 in two / 6.6, 8: 8.1 / 7.2), of 64 from twelve (9: 8.5 / 8.8, 15: 11.1 / 10.4).
    auto blocks_of = [&](int64_t queries) { return bh * (((int64_t)a.Sq + queries - 1) / queries); };
    const int64_t programs = blocks_of(kQBlock);
    int split = 1, nw = 4;
    if (far && nblk >= 12) {                                             // (a few blocks: dealt out like anybody's, the same bits)
    } else if (blocks_of(32) <= 256) {
        split = nblk >= 7 ? 4 : nblk >= 2 ? 2 : 1;
        nw = dma || split > 1 ? 1 : 4;
    } else if (blocks_of(64) <= 256) {
        split = nblk >= 12 ? 4 : nblk >= 2 ? 2 : 1;
        nw = dma || split > 1 ? 2 : 4;
    } else if (dma) {
        split = programs <= 256 ? (nblk >= 12 ? 4 : nblk >= 7 ? 2 : 1) : programs <= 512 && nblk >= 12 ? 2 : 1;
    } else {
        // Through registers, where a group's loads are not ahead of its arithmetic, four groups pay while units stay empty (32
        // programs x 64 blocks 57 / 44, 160 x 24 24.2 / 22.0, 256 x 32 32 / 35), two do not (512 x 32 51 / 56).
        split = nblk >= 12 && programs <= 160 ? 4 : 1;
    }
    // Blocks of 256 queries where that costs no more rounds of the units: the keys travel from L2 to LDS half as often.  Measured (us, 128 /
    // 256 queries): 192 heads, 1024 x 1024 64.2 / 61.7, 93 heads, 1280 x 581 28.5 / 26.7, 80 heads, 408 x 397 12.5 / 12.0; with a round
    // more they lose: 100 heads, 1815 x 227 22.0 / 25.0, 72 heads, 2040 x 736 39.2 / 42.2.
    if (dma && split == 1 && nw == 4 && nblk >= 3 && 2 * ((blocks_of(2 * kQBlock) + 255) / 256) <= (programs + 255) / 256) nw = 8;
    k.nqb = (int32_t)(((int64_t)a.Sq + 32 * nw - 1) / (32 * nw));
    hipStream_t s = (hipStream_t)stream;
    const int64_t grid = bh * k.nqb;
    if (bf16) return dma ? launch_sdpa_split<true, true>(k, grid, split, nw, s) : launch_sdpa_split<true, false>(k, grid, split, nw, s);
    return dma ? launch_sdpa_split<false, true>(k, grid, split, nw, s) : launch_sdpa_split<false, false>(k, grid, split, nw, s);
}

nt_status launch_sdpa_desc(const void *q, const nt_tensor_desc *dq, const void *k, const nt_tensor_desc *dk,
                           const void *v, const nt_tensor_desc *dv, void *o, const nt_tensor_desc *dout,
                           float scale, int dtype, void *stream)
{
    t_plan = nt_sdpa_plan{};
    const nt_tensor_desc *d[4] = {dq, dk, dv, dout};
    for (const nt_tensor_desc *t : d) {
        if (!t) return fail(NT_ERR_INVALID_ARG, "null tensor descriptor");
        if (t->ndim != 4) return fail(NT_ERR_SHAPE_MISMATCH, "sdpa tensors must be 4-D [batch, heads, seq, head_dim]");
        for (int i = 0; i < 4; ++i)
            if (t->size[i] < 0) return fail(NT_ERR_INVALID_ARG, "negative size");
        if (t->size[0] != dq->size[0] || t->size[1] != dq->size[1]) return fail(NT_ERR_SHAPE_MISMATCH, "batch / head counts differ");
        if (t->size[3] != kHeadDim) return fail(NT_ERR_UNSUPPORTED, "sdpa is built for head_dim 64");
        if (t->size[3] > 1 && t->stride[3] != 1) return fail(NT_ERR_UNSUPPORTED, "sdpa needs unit stride along the head dimension");
    }
    if (dk->size[2] != dv->size[2]) return fail(NT_ERR_SHAPE_MISMATCH, "K and V sequence lengths differ");
    if (dout->size[2] != dq->size[2]) return fail(NT_ERR_SHAPE_MISMATCH, "Q and O sequence lengths differ");
    if (dq->size[0] == 0 || dq->size[1] == 0 || dq->size[2] == 0) return NT_OK;
    if (dk->size[2] == 0) return fail(NT_ERR_INVALID_ARG, "sdpa over an empty key sequence is undefined");
    if (!q || !k || !v || !o) return fail(NT_ERR_INVALID_ARG, "null device pointer");
    if (dq->size[2] > 0x7fffffffLL - kQBlock || dk->size[2] > 0x7fffffffLL - kKeyBlock || dq->size[1] > 65535) return fail(NT_ERR_UNSUPPORTED, "sequence too long");
    if (!(scale == scale)) return fail(NT_ERR_INVALID_ARG, "scale is NaN");
    SdpaArgs a{};
    a.Q = (const uint16_t *)q; a.K = (const uint16_t *)k; a.V = (const uint16_t *)v; a.O = (uint16_t *)o;
    a.q_sb = dq->stride[0]; a.q_sh = dq->stride[1]; a.q_ss = dq->stride[2];
    a.k_sb = dk->stride[0]; a.k_sh = dk->stride[1]; a.k_ss = dk->stride[2];
    a.v_sb = dv->stride[0]; a.v_sh = dv->stride[1]; a.v_ss = dv->stride[2];
    a.o_sb = dout->stride[0]; a.o_sh = dout->stride[1]; a.o_ss = dout->stride[2];
    a.H = (int32_t)dq->size[1]; a.Sq = (int32_t)dq->size[2]; a.Sk = (int32_t)dk->size[2];
    const float sc = scale == 0.f ? 0.125f : scale;                  // default 1 / sqrt(64)
    a.scale_log2e = sc * 1.4426950408889634f;
    return launch_sdpa(a, dq->size[0], dtype == NT_BF16, stream);
}

}  // namespace nt
