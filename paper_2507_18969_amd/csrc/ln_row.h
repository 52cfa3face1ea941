// LayerNorm (Eq. 9) of a row of 256, by one wave with 4 columns a lane, and its
// adjoint.  The row kernels (kernels.hip) and the FP32 row-block kernel
// (fused_fp32.hip) must give the same bits, so both come here and every rounding is
// written out: nothing is left to what a compiler contracts.  (0.f + s: sums start at
// zero, which is what the sign of an empty one comes from.)
#pragma once
#include "common.h"

namespace edpc {

typedef float f32q __attribute__((ext_vector_type(4)));
constexpr int kLnRow = 256;

__device__ __forceinline__ f32q ln_row_fwd(f32q x, f32q gm, f32q bt, float* mean, float* rstd) {
#pragma clang fp contract(off)
  const float mu = wave_sum(0.f + ((x[0] + x[1]) + (x[2] + x[3]))) / (float)kLnRow;
  const f32q d = x - mu;
  const float q = fmaf(d[0], d[0], d[1] * d[1]) + fmaf(d[2], d[2], d[3] * d[3]);
  const float var = wave_sum(0.f + q) / (float)kLnRow;
  const float rs = 1.0f / sqrtf(var + 1e-5f);
  f32q z;
#pragma unroll
  for (int e = 0; e < 4; ++e) z[e] = fmaf(d[e] * rs, gm[e], bt[e]);
  *mean = mu;
  *rstd = rs;
  return z;
}

// d: adjoint of the output, dn: of the residual stream past the block.
__device__ __forceinline__ f32q ln_row_bwd(f32q x, float mu, float rs, f32q gm, f32q d, f32q dn) {
#pragma clang fp contract(off)
  const f32q xh = (x - mu) * rs, dx = d * gm;
  const float s1 = fmaf(d[1], gm[1], dx[0]) + fmaf(d[2], gm[2], dx[3]);
  const float s2 = fmaf(xh[0], dx[0], xh[1] * dx[1]) + fmaf(xh[2], dx[2], xh[3] * dx[3]);
  const float m1 = wave_sum(0.f + s1) / (float)kLnRow, m2 = wave_sum(0.f + s2) / (float)kLnRow;
  f32q o;
  o[0] = fmaf(rs, fmaf(-xh[0], m2, dx[0] - m1), dn[0]);
#pragma unroll
  for (int e = 1; e < 4; ++e) o[e] = fmaf(rs, fmaf(-xh[e], m2, fmaf(d[e], gm[e], -m1)), dn[e]);
  return o;
}

}  // namespace edpc
