// ROCKET transform for MI355X (gfx950): forward kernels of short series for masks with softPPV.
#include "rocket_forward_impl.hpp"

int rk_launch_forward_short_soft(const rocket_kernels *h, const float *xpad, int32_t B, uint32_t mask, float nl, float ns, float *partials, int spread,
                                 void *stream)
{
    constexpr uint32_t soft = ROCKET_F_SOFTPPV;
    switch (mask) {
    case soft: return rk_forward_launch<64, soft>(h, xpad, B, nl, ns, partials, spread, stream);
    case soft | ROCKET_F_MAX: return rk_forward_launch<64, soft | ROCKET_F_MAX>(h, xpad, B, nl, ns, partials, spread, stream);
    case soft | ROCKET_F_PPV: return rk_forward_launch<64, soft | ROCKET_F_PPV>(h, xpad, B, nl, ns, partials, spread, stream);
    default: return rk_forward_launch<64, soft | ROCKET_F_MAX | ROCKET_F_PPV>(h, xpad, B, nl, ns, partials, spread, stream);
    }
}
