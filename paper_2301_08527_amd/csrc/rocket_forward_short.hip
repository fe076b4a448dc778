// ROCKET transform for MI355X (gfx950): forward kernel for short series, one
// 64-lane wavefront per (series, kernel).  With a few thousand outputs or fewer a
// 256-lane workgroup would leave most lanes without a strip; a single wavefront
// fills its lanes with shorter strips and needs no cross-wavefront reduction.
#include "rocket_forward_impl.hpp"

int rk_launch_forward_short(const rocket_kernels *h, const float *xpad, int32_t B, uint32_t mask, float nl, float ns,
                            float *partials, void *stream)
{
    const int spread = 0;   // measured: the per-XCD series mapping makes the short-series launch 2 % slower
    if (mask & ROCKET_F_SOFTPPV) return rk_launch_forward_short_soft(h, xpad, B, mask, nl, ns, partials, spread, stream);
    return rk_forward_launch_mask<64, 0>(h, xpad, B, mask, nl, ns, partials, spread, stream);
}
