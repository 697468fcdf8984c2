// Instantiations of the direct-to-LDS kernel on 16 x 16 x 32 matrix instructions, 64 x 64 tile, bf16 inputs, both flavours.
#include "gemm_direct16.h"

namespace nt {
nt_status launch_direct16_64x64_bf16(const FastArgs &a, int alay, int blay, int64_t nwg, hipStream_t s)
{
    return launch_direct16_t<64, 64, true>(a, alay, blay, nwg, s);
}
nt_status launch_direct16_edge_64x64_bf16(const FastArgs &a, int alay, int blay, int64_t nwg, hipStream_t s)
{
    return launch_direct16_t<64, 64, true, true>(a, alay, blay, nwg, s);
}
}  // namespace nt
