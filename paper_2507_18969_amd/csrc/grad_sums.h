// Gradients that are sums over rows other than the products': embedding and
// column sums.  Device code of a workgroup of 256, by itself (kernels.hip) or in
// the launch of the FP32 weight gradients (gemm_fp32.hip).
#pragma once
#include "kernels.h"

namespace edpc {

// ---------------------------------------------------------------------------
// Embedding gradient: dEmb[v] = sum over (row, position) with ctx = v of the
// matching E-slice of dX.  A block takes a chunk of rows, a few rows at a time;
// the chunk partials are then added in chunk order.
//
// dEmb_chunk[v][e] = sum over the chunk's (row, position) pairs of
// [ctx = v] * dX[row][position*E + e]: a matrix product on the BF16 MFMA
// whose A operand, the one-hot of the context bytes, is formed in registers
// (exact in BF16).  An FP32 value x is the exact sum of three BF16 values
// (x rounded to 8 significant bits, then the rounding errors of what is
// left), so dX enters as three BF16 operands accumulated in FP32: an FP32
// sum of the same terms, 3 MFMA instructions per 32 pairs where the FP32
// MFMA (K = 4) takes 8.
// Wave w owns byte values 64w .. 64w+63; pairs are visited in row-major
// order, 32 per step.  The work is in preparing operands, so each value is split
// once, on its way to LDS, and read there transposed (16384 rows of 2048: 100 us;
// 157 us split by every wave that uses it).
// ---------------------------------------------------------------------------
// pairs of a sub-batch, in whole steps
inline __host__ __device__ int emb_pairs(int sub_rows, int C) { return (sub_rows * C + 31) & ~31; }
inline size_t emb_lds_bytes(int sub_rows, int C, int E) {
  return (size_t)emb_pairs(sub_rows, C) * (6 * E + 1);
}

template <int E>
__device__ __forceinline__ void emb_grad_block(int rows, const uint8_t* __restrict__ ctx,
                                               const float* __restrict__ dx, int C, int chunk_rows,
                                               int sub_rows, float* __restrict__ partial, int block,
                                               char* smem) {
  constexpr int NE = E / 16;
  const int F = C * E;
  const int plane = emb_pairs(sub_rows, C) * E * 2;          // bytes
  uint8_t* lds_ctx = (uint8_t*)smem + 3 * plane;             // [pairs]
  const int r0 = block * chunk_rows;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  f32x4 acc[4][NE];
#pragma unroll
  for (int vb = 0; vb < 4; ++vb)
#pragma unroll
    for (int nb = 0; nb < NE; ++nb) acc[vb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int r_end = min(rows, r0 + chunk_rows);
  // The next sub-batch of rows is loaded into registers while the current
  // one feeds the MFMAs from LDS: up to 8192 floats of dX (8 float4 a
  // thread) and 512 context bytes (sub_rows * C <= 8192 / E).  Wider rows
  // (F > 8192, one row a sub-batch) are copied straight to LDS instead.
  constexpr int kStage = 8;
  const bool staged = sub_rows * F <= 4 * kStage * 256;
  float4 nx[kStage];
  uint32_t nc[2] = {0u, 0u};
  auto fetch = [&](int rs) {
    const int nr = min(sub_rows, r_end - rs);
    const float4* src = (const float4*)(dx + (size_t)rs * F);
#pragma unroll
    for (int q = 0; q < kStage; ++q) {
      const int k = (int)threadIdx.x + 256 * q;
      nx[q] = k < nr * F / 4 ? src[k] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int k = (int)threadIdx.x + 256 * q;
      nc[q] = k < nr * C ? (uint32_t)ctx[(size_t)rs * C + k] : 0u;
    }
  };
  auto put = [&](int k, float4 x) {  // 4 values of one pair, split into the three planes
    const float v[4] = {x.x, x.y, x.z, x.w};
    bf16_t b[3][4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      b[0][u] = f2bf(v[u]);
      const float r1 = v[u] - bf2f(b[0][u]);
      b[1][u] = f2bf(r1);
      b[2][u] = f2bf(r1 - bf2f(b[1][u]));
    }
#pragma unroll
    for (int t = 0; t < 3; ++t)
      *(uint2*)(smem + t * plane + 8 * k) =
          make_uint2((uint32_t)b[t][0] | ((uint32_t)b[t][1] << 16), (uint32_t)b[t][2] | ((uint32_t)b[t][3] << 16));
  };
  if (staged && r0 < r_end) fetch(r0);
  for (int rs = r0; rs < r_end; rs += sub_rows) {
    const int nr = min(sub_rows, r_end - rs);
    const int np = nr * C, np32 = (np + 31) & ~31;  // pairs past the end: zeros
    __syncthreads();  // the previous sub-batch's LDS reads are done
    if (staged) {
#pragma unroll
      for (int q = 0; q < kStage; ++q) {
        const int k = (int)threadIdx.x + 256 * q;
        if (k < np32 * E / 4) put(k, nx[q]);
      }
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int k = (int)threadIdx.x + 256 * q;
        if (k < np32) lds_ctx[k] = (uint8_t)nc[q];
      }
    } else {
      const float4* src = (const float4*)(dx + (size_t)rs * F);
      for (int k = threadIdx.x; k < np32 * E / 4; k += 256)
        put(k, k < nr * F / 4 ? src[k] : make_float4(0.f, 0.f, 0.f, 0.f));
      for (int k = threadIdx.x; k < np32; k += 256) lds_ctx[k] = k < np ? ctx[(size_t)rs * C + k] : 0;
    }
    __syncthreads();
    if (staged && rs + sub_rows < r_end) fetch(rs + sub_rows);
    // lane group g = lane / 16 takes pairs p0 .. p0 + 7 of each 32-pair step;
    // pairs past the chunk's end take no byte value
    for (int k0 = 0; k0 < np; k0 += 32) {
      const int p0 = k0 + 8 * (lane >> 4);
      const uint2 by = *(const uint2*)(lds_ctx + p0);
      uint32_t bytes[8];
#pragma unroll
      for (int v = 0; v < 8; ++v)
        bytes[v] = p0 + v < np ? ((v < 4 ? by.x : by.y) >> (8 * (v & 3))) & 0xFFu : 0xFFFFu;
      bf16x8 b[3][NE];
      const char* at = smem + (size_t)(p0 + ((lane & 15) >> 2)) * E * 2 + 8 * (lane & 3);
#pragma unroll
      for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int nb = 0; nb < NE; ++nb)
          b[t][nb] = lds_frag_tr(at + t * plane + 32 * nb, at + t * plane + 32 * nb + 8 * E);
#pragma unroll
      for (int vb = 0; vb < 4; ++vb) {
        const uint32_t me = (uint32_t)(64 * w + 16 * vb + (lane & 15));
        uint32_t q[4];
#pragma unroll
        for (int h = 0; h < 4; ++h)
          q[h] = (bytes[2 * h] == me ? 0x3F80u : 0u) | ((bytes[2 * h + 1] == me ? 0x3F80u : 0u) << 16);
        const bf16x8 a = __builtin_bit_cast(bf16x8, make_uint4(q[0], q[1], q[2], q[3]));
#pragma unroll
        for (int nb = 0; nb < NE; ++nb)
#pragma unroll
          for (int t = 0; t < 3; ++t)
            acc[vb][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b[t][nb], acc[vb][nb], 0, 0, 0);
      }
    }
  }
  float* out = partial + (size_t)block * 256 * E;
#pragma unroll
  for (int vb = 0; vb < 4; ++vb)
#pragma unroll
    for (int nb = 0; nb < NE; ++nb)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int v = 64 * w + 16 * vb + 4 * (lane >> 4) + r;
        out[(size_t)v * E + 16 * nb + (lane & 15)] = acc[vb][nb][r];
      }
}

// ---------------------------------------------------------------------------
// Column sums over the active rows (bias and LayerNorm affine gradients).
// Two passes with a fixed order: rows are cut into chunks of kColChunk; a
// block sums 64 columns of one chunk (4 interleaved row slices added in slice
// order) into partial[chunk][col]; the second pass adds the chunks in order.
// lds: 1 KiB.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void colsum_block(const StepState* __restrict__ st,
                                             const ColsumJob* __restrict__ jobs, int n_jobs, int total_cols,
                                             float* __restrict__ partial, int block, int chunk, float* lds) {
  const int rows = st->rows;
  const int r0 = chunk * kColChunk;
  if (r0 >= rows) return;
  const ColsumJob jb =
      jobs[find_entry(jobs, n_jobs, block, [](const ColsumJob& j) { return j.col_block_begin; })];
  const int lc = (block - jb.col_block_begin) * 64 + (threadIdx.x & 63);
  const int slice = threadIdx.x >> 6;
  const int r1 = min(rows, r0 + kColChunk);
  float acc = 0.f;
  const auto src = gl(jb.src);
  if (lc < jb.cols) {
    if (jb.h) {
      const auto h = gl(jb.h), mean = gl(jb.mean), rstd = gl(jb.rstd);
#pragma unroll 4
      for (int r = r0 + slice; r < r1; r += 4) {
        const float xh = (h[(size_t)r * jb.ld + lc] - mean[r]) * rstd[r];
        acc = fmaf(src[(size_t)r * jb.ld + lc], xh, acc);
      }
    } else {
#pragma unroll 4
      for (int r = r0 + slice; r < r1; r += 4) acc += src[(size_t)r * jb.ld + lc];
    }
  }
  lds[64 * slice + (threadIdx.x & 63)] = acc;
  __syncthreads();
  if (slice == 0 && lc < jb.cols) {
    const int t = threadIdx.x;
    partial[(size_t)chunk * total_cols + jb.col_offset + lc] = (lds[t] + lds[64 + t]) + (lds[128 + t] + lds[192 + t]);
  }
}

}  // namespace edpc
