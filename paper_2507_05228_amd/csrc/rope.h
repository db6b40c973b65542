// Rotary angles, shared by the row kernels and the few-row shard GEMM.
#pragma once
#include <hip/hip_runtime.h>

// cos and sin of position * theta^(-2i/d), i < d/2.  The angle is carried in revolutions: rev = theta^(-2i/d) /
// (2 pi) in double precision, split into two floats, and position * rev is formed with a compensated product, so
// the fractional part (all that sine and cosine need) stays accurate to ~1e-7 revolutions however large the
// position (below 2^24); sine and cosine are then single hardware instructions.
struct RopeRev { float hi, lo; };
__device__ __forceinline__ RopeRev rope_rev_log2(double log2_theta, int i, int head_dim) {
    const double rev = exp2(-2.0 * i / head_dim * log2_theta) / 6.283185307179586476925;
    RopeRev r;
    r.hi = (float)rev;
    r.lo = (float)(rev - (double)r.hi);
    return r;
}
__device__ __forceinline__ RopeRev rope_rev(float theta, int i, int head_dim) { return rope_rev_log2(log2((double)theta), i, head_dim); }
__device__ __forceinline__ void rope_cos_sin(float pos, float c_hi, float c_lo, float &cs, float &sn) {
#pragma clang fp contract(off)   // r_hi fused into the subtraction of its floor would count r_err twice
    const float r_hi = pos * c_hi;
    const float r_err = fmaf(pos, c_hi, -r_hi) + pos * c_lo;      // pos * (hi + lo) = r_hi + r_err
    const float rev = (r_hi - floorf(r_hi)) + r_err;
    sn = __builtin_amdgcn_sinf(rev);
    cs = __builtin_amdgcn_cosf(rev);
}
