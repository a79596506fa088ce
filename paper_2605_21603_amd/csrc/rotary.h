// The rotation of a pair of head-dim elements, shared by every kernel that applies it.
#pragma once
#include "common.h"

namespace dyn {

// A row has the same bits whichever kernel its launch took, so what the compiler could contract either way
// is written out: the rotation of a pair here, the sums of squares of the norms where they are taken.
__device__ __forceinline__ float rotated_lo(float a, float b, float c, float s) { return __builtin_fmaf(a, c, -(b * s)); }
__device__ __forceinline__ float rotated_hi(float a, float b, float c, float s) { return __builtin_fmaf(b, c, a * s); }

// Sine and cosine of pos * inv_freq, reduced to [-pi, pi] in fp64.
__device__ __forceinline__ void rotary_angle(int pos, double inv_freq, float &s, float &c) {
    const double ang = (double)pos * inv_freq;
    const double turns = rint(ang * 0.15915494309189535);              // 1 / (2 pi)
    sincosf((float)fma(-turns, 6.283185307179586, ang), &s, &c);
}

}  // namespace dyn
