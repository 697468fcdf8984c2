// Instantiation: 256 and 224 positions x 256 filters per program, both input formats.
#include "gemm_conv_plane_kernel.h"

namespace nt {
template nt_status launch_conv_plane_t<8, 7, 8, 2, 9>(const ConvPlaneArgs &a, bool bf16, hipStream_t s);
template nt_status launch_conv_plane_t<8, 7, 8, 3, 0>(const ConvPlaneArgs &a, bool bf16, hipStream_t s);
}
