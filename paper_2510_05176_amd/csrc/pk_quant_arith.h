// The stored parameters of a quantization group (Sec. 2.1 Eq. 1 with this library's
// rounding rules: z = group minimum rounded to fp16 towards -inf, s = (max - z) / (2^b - 1) rounded to fp16 towards
// +inf; the code of a residual is clamp(rint((r - z) * (1/s)), 0, 2^b - 1) in binary32, ties to even, and s == 0 gives
// 1/s = 0 and code 0).  Files that use it switch FMA contraction off.
#pragma once

#include "pk_divide.h"
#include "pk_internal.h"

namespace pk {

struct GroupParams {
    unsigned short s16, z16;
    float s, z, inv;
};

__device__ __forceinline__ GroupParams group_params(float mn, float mx, int bits)
{
    GroupParams g;
    g.z16 = f2h_down(mn);
    g.z = hbits2f(g.z16);
    const float s32 = div_by_levels(mx - g.z, bits);
    g.s16 = f2h_up(s32);
    g.s = hbits2f(g.s16);
    g.inv = g.s == 0.f ? 0.f : recip_of_scale(g.s);
    return g;
}

}  // namespace pk
