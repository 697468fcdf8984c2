// Instantiation: 128 and 96 positions x 256 filters per program, both input formats.
#include "gemm_conv_plane_kernel.h"

namespace nt {
template nt_status launch_conv_plane_t<4, 3, 8, 2, 9>(const ConvPlaneArgs &a, bool bf16, hipStream_t s);
template nt_status launch_conv_plane_t<4, 3, 8, 3, 9>(const ConvPlaneArgs &a, bool bf16, hipStream_t s);
template nt_status launch_conv_plane_t<4, 3, 8, 2, 0>(const ConvPlaneArgs &a, bool bf16, hipStream_t s);
template nt_status launch_conv_plane_t<4, 3, 8, 3, 0>(const ConvPlaneArgs &a, bool bf16, hipStream_t s);
}
