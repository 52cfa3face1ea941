// FP32 row-block kernel: LTE up product .. head .. coder .. adjoint back to dY.
#pragma once
#include "kernels.h"

namespace edpc {

// Arrays of refinement block 0; block j's lie j strides (in floats) further on.
template <class T>
struct BlockArray {
  T* p;
  long long stride;
  __device__ __forceinline__ T* of(int j) const { return p + j * stride; }
};

struct FusedFp32Args {
  const StepState* st;
  int n_blocks, L, H;
  BlockArray<const float> gamma, beta, w0, b0, wo, bo;
  // input, LayerNorm output and statistics, branches, gated product
  BlockArray<float> h, z, mean, rstd, abr, g;
  BlockArray<float> da, dz, dh;  // adjoints of the branches, the LayerNorm's output, the input
  const float *y, *w2, *b2, *wh, *bh;
  float *hn, *dhn, *dy;  // the head's input, its adjoint, the adjoint of y
  HeadArgs head;
  int buf;               // set by the launcher
};

// Rows of a step that take it.  One workgroup has 16 rows and a CU's share of the
// matrix cores, but none of the launches between the products (2 blocks of 128,
// whole update: 8 rows 109 us as launches, 92 so; 64 rows 115 and 97; 1024 rows
// 146 and 125; 4000 rows 283 and 223).  From 4096 rows the LayerNorm's adjoint also
// forms column sums, in another order.
constexpr int kFusedFp32Rows = 4095;
// F = 256, L and H multiples of 64 up to 256 and 128, 1..3 branches.
bool fused_fp32_supported(int F, int L, int H, int branches);
hipError_t launch_fused_fp32(FusedFp32Args a, int branches, const StreamIO& io, int max_rows, hipStream_t s);

}  // namespace edpc
