// Instantiation: 224 and 192 positions x 256 filters per program, both input formats.
#include "gemm_conv_plane_kernel.h"

namespace nt {
template nt_status launch_conv_plane_t<7, 6, 8, 2, 9>(const ConvPlaneArgs &a, bool bf16, hipStream_t s);
}
