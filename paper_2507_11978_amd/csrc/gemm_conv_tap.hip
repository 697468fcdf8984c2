// Instantiations of the convolution kernel that walks the reduction tap by tap, and the filter's copy in that order.
#include "gemm_conv_tap.h"

namespace nt {

// filter [F][C][R * S] (row pitch ldb) -> [F][R * S][C] (row pitch K = C R S): one workgroup per filter, the row read and
// written 16 bytes per thread (C is a multiple of 32: eight k' belong to one tap), permuted on its way through LDS
// (256 filters of 2304: 4.4 us, 4.8 with two bytes per thread: the launch and two trips to memory)
__global__ __launch_bounds__(256) void conv_repack_filter_kernel(const uint16_t *w, int64_t ldb, uint16_t *out, int32_t C, int32_t RS)
{
    extern __shared__ __attribute__((aligned(16))) uint16_t row[];
    const int32_t K = C * RS;
    const uint16_t *src = w + (int64_t)blockIdx.x * ldb;
    uint16_t *dst = out + (int64_t)blockIdx.x * K;
    for (int32_t i = threadIdx.x * 8; i < K; i += 2048) {
        u32x4 v;
        __builtin_memcpy(&v, src + i, 16);
        *reinterpret_cast<u32x4 *>(row + i) = v;
    }
    __syncthreads();
    for (int32_t j = threadIdx.x * 8; j < K; j += 2048) {
        const int32_t tap = j / C, c = j - tap * C;
        uint32_t e[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) e[i] = row[(c + i) * RS + tap];
        const u32x4 v{e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
        *reinterpret_cast<u32x4 *>(dst + j) = v;
    }
}

nt_status launch_conv_tap(const ConvArgs &a, int rows, bool bf16, int64_t nwg, hipStream_t s)
{
    if (rows == 256) return bf16 ? launch_conv_tap_inst<true, 8, 7>(a, nwg, s) : launch_conv_tap_inst<false, 8, 7>(a, nwg, s);
    if (rows == 224) return bf16 ? launch_conv_tap_inst<true, 7, 6>(a, nwg, s) : launch_conv_tap_inst<false, 7, 6>(a, nwg, s);
    return fail(NT_ERR_UNSUPPORTED, "no convolution kernel for this tile height");
}

nt_status launch_conv_tap_trace(const ConvArgs &a, int rows, hipStream_t s)
{
    if (rows == 256) return launch_conv_tap_inst<false, 8, 7, true>(a, 1, s);
    if (rows == 224) return launch_conv_tap_inst<false, 7, 6, true>(a, 1, s);
    return fail(NT_ERR_UNSUPPORTED, "no convolution kernel for this tile height");
}

nt_status launch_conv_repack_filter(const uint16_t *w, int64_t ldb, uint16_t *out, int32_t F, int32_t C, int32_t RS, hipStream_t s)
{
    // (the reduction is below 2^16 elements: a row fits LDS)
    hipLaunchKernelGGL(conv_repack_filter_kernel, dim3((unsigned)F), dim3(256), (size_t)C * RS * sizeof(uint16_t), s, w, ldb, out, C, RS);
    return check_launch("conv_repack_filter_kernel");
}

}  // namespace nt
