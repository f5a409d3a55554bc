// O(n) bond activation with Wolff's embedding (Sec. 2 of the paper), shared
// by the tiled pyrochlore sweep and the generic graph sweep:
//   sigma = fmaf(s_z, r_z, fmaf(s_y, r_y, s_x * r_x))      (XY: no z term)
//   x     = (x0 * sigma_a) * sigma_b,   x0 = (float)(2 J / T)
//   bond active iff (double)x > -log1p(-u), u = (r32 + 0.5) 2^-32.
// The FP64 log1p is evaluated only when x lies within 1e-4 (1 + t) of
// t = -ln(1 - u) computed in FP32 with the native base-2 logarithm: that
// margin exceeds the FP32 error by orders of magnitude, so outside it the
// FP32 comparison gives the same answer as the exact one.  1 - u is
// (not r32 + 0.5) 2^-32: one conversion and one fused multiply-add give it
// within a relative 2^-23, where five FP64 instructions per bond had.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

namespace pyro {

template <int NV>
__device__ __forceinline__ float project(const float v[NV], const float r[NV])
{
    float sig = __fmul_rn(v[0], r[0]);
    sig = __fmaf_rn(v[1], r[1], sig);
    if (NV == 3) sig = __fmaf_rn(v[NV - 1], r[NV - 1], sig);
    return sig;
}

// The exact comparison, out of line: it is rarely reached, and 48 inlined
// copies per cell would swell the tile kernel's code.
static __device__ __noinline__ bool on_bond_exact(float x, uint32_t r32)
{
    return (double)x > -log1p(-(((double)r32 + 0.5) * 0x1p-32));
}

// FP32 decision of one bond (see the file comment): active, or *close when
// only the exact comparison can tell.
__device__ __forceinline__ bool on_bond_filter(float x, uint32_t r32, bool *close)
{
    const float v = __fmaf_rn((float)~r32, 0x1p-32f, 0x1p-33f);  // 1 - u, at least 2^-33: a normal number
    const float t = -0.6931472f * __log2f(v);  // native base-2 logarithm
    const float m = __fmaf_rn(1e-4f, t, 1e-4f);
    *close = x > 0.0f && !(x > t + m) && !(x < t - m);
    return x > t + m;
}

// Activation of one bond.
__device__ __forceinline__ bool on_bond_active(float x, uint32_t r32)
{
    if (!(x > 0.0f)) return false;
    bool close;
    const bool active = on_bond_filter(x, r32, &close);
    return close ? on_bond_exact(x, r32) : active;
}

}  // namespace pyro
