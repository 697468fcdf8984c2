// Instantiation: 192 and 160 positions x 128 filters per program, both input formats.
#include "gemm_conv_plane_kernel.h"

namespace nt {
template nt_status launch_conv_plane_t<6, 5, 4, 2, 9>(const ConvPlaneArgs &a, bool bf16, hipStream_t s);
}
