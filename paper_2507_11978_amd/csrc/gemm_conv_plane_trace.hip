// Loader trace of the convolution kernel whose input rows stay in LDS: every tile's set-up, one block of channels, one slice of the filter.
#include "gemm_conv_plane_kernel.h"

namespace nt {

nt_status launch_conv_plane_trace(const ConvPlaneArgs &a, const ConvPlanePlan &p, hipStream_t s)
{
    typedef nt_status (*Launcher)(const ConvPlaneArgs &, hipStream_t);
#define NT_PLANE_ENTRY(TMA, TMB, TN, U, TAPS) launch_conv_plane_inst<false, TMA, TMB, TN, U, TAPS, true>,
    static const Launcher table[] = {NT_PLANE_TILES(NT_PLANE_ENTRY)};
#undef NT_PLANE_ENTRY
    return table[p.tile](a, s);
}

}  // namespace nt
