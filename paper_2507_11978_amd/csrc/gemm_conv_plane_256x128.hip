// Instantiation: 256 and 224 positions x 128 filters per program, both input formats.
#include "gemm_conv_plane_kernel.h"

namespace nt {
template nt_status launch_conv_plane_t<8, 7, 4, 2, 9>(const ConvPlaneArgs &a, bool bf16, hipStream_t s);
template nt_status launch_conv_plane_t<8, 7, 4, 2, 0>(const ConvPlaneArgs &a, bool bf16, hipStream_t s);
template nt_status launch_conv_plane_t<8, 7, 4, 3, 0>(const ConvPlaneArgs &a, bool bf16, hipStream_t s);
}
