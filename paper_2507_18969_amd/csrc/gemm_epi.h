// Epilogues of the 4-wave product tiles, one output element at a time.
#pragma once
#include "gemm.h"

namespace edpc {

// Global operands of one output element (m, n) of a product, read ahead of
// the sum where the tile is small enough to hold them.  NB: branches of a
// gated forward product; a gated adjoint takes its branch count (1..3) from
// g.bias_branch_stride.
template <int EPI, int NB>
struct EpiOperands {
  static constexpr int N = EPI == EPI_STORE ? 2 : EPI == EPI_GATE_FWD ? NB : 3;
  float v[N];
  __device__ __forceinline__ void load(const GemmArgs& g, int m, int n) {
    if constexpr (EPI == EPI_STORE) {
      v[0] = g.bias ? g.bias[n] : 0.f;
      v[1] = g.resid ? g.resid[(long long)m * g.ld_resid + n] : 0.f;
    } else if constexpr (EPI == EPI_GATE_FWD) {
#pragma unroll
      for (int b = 0; b < NB; ++b) v[b] = g.bias[b * g.bias_branch_stride + n];
    } else {
      const float* a = g.aux + (long long)m * g.ld_aux + n;
#pragma unroll
      for (int b = 0; b < 3; ++b) v[b] = b < g.bias_branch_stride ? a[b * g.aux_branch] : 1.0f;
    }
  }
};

// Output element (m, n) from its sums acc[0 .. NB-1] and operands.
template <int EPI, int NB>
__device__ __forceinline__ void epi_element(const GemmArgs& g, int m, int n, const float (&acc)[NB],
                                            const EpiOperands<EPI, NB>& p) {
  if constexpr (EPI == EPI_STORE) {
    float v = acc[0];
    if (g.bias) v += p.v[0];
    if (g.resid) v += p.v[1];
    if (g.out32) g.out32[(long long)m * g.ld_out32 + n] = v;
    if (g.out16) g.out16[(long long)m * g.ld_out16 + n] = f2bf(v);
  } else if constexpr (EPI == EPI_GATE_FWD) {
    float prod = 1.0f;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const float a = acc[b] + p.v[b];
      g.aux[(long long)m * g.ld_aux + b * g.aux_branch + n] = a;
      prod = (b == 0) ? a : prod * a;
    }
    const float v = gelu_f(prod);
    if (g.out32) g.out32[(long long)m * g.ld_out32 + n] = v;
    if (g.out16) g.out16[(long long)m * g.ld_out16 + n] = f2bf(v);
  } else {  // EPI_GATE_BWD
    const int nbr = g.bias_branch_stride;
    float prod = 1.0f;
#pragma unroll
    for (int b = 0; b < 3; ++b)
      if (b < nbr) prod = (b == 0) ? p.v[b] : prod * p.v[b];
    const float dp = acc[0] * gelu_grad_f(prod);
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      if (b >= nbr) break;
      float o = dp;
#pragma unroll
      for (int c = 0; c < 3; ++c)
        if (c != b && c < nbr) o *= p.v[c];
      if (g.out32) g.out32[(long long)m * g.ld_out32 + b * g.aux_branch + n] = o;
      if (g.out16) g.out16[(long long)m * g.ld_out16 + b * g.aux_branch + n] = f2bf(o);
    }
  }
}

}  // namespace edpc
