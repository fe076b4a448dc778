// ROCKET transform for MI355X (gfx950): forward kernels of long series for masks with softPPV.
#include "rocket_forward_impl.hpp"

int rk_launch_forward_soft(const rocket_kernels *h, const float *xpad, int32_t B, uint32_t mask, float nl, float ns, float *partials, int spread,
                           void *stream)
{
    return rk_forward_launch_mask<kThreads, ROCKET_F_SOFTPPV>(h, xpad, B, mask, nl, ns, partials, spread, stream);
}
