// Kraskov's mutual-information estimator on the GPU (Sec. 3.1.1, Eq. 7):
// the analysis the paper uses to compare refinement blocks with one, two
// and three branches (the IFR metric, Eq. 8).
//
//   1. D_z[i][j] = max_c |z_ic - z_jc| and D_y likewise: tiled like a matrix
//      product, but with max(|a - b|) in place of the multiply-add, so it
//      runs on the vector ALUs (three instructions per pair and two
//      dimensions).
//   2. per sample i, one wave: eps_i = the v-th smallest of
//      max(D_z[i][j], D_y[i][j]) over j != i (ties with multiplicity), then
//      c_z(i) = #{j != i: D_z[i][j] < eps_i}, c_y(i) likewise.
//   3. on the host: psi(v) + psi(c) - mean(psi(c_z + 1) + psi(c_y + 1)),
//      psi at integers from harmonic numbers.
// Distances are FP32 (correctly rounded differences, exact maxima), so the
// neighbour counts are those of any FP32 evaluation of the definition.
#include <cmath>
#include <optional>
#include <vector>

#include "model.h"

namespace edpc {

constexpr int kKsgTile = 32;   // 32 x 32 sample pairs per workgroup
constexpr int kKsgDim = 64;    // dimensions per LDS stage, 16 for each of the 4 waves
constexpr int kKsgMaxV = 16;   // largest neighbour order v
constexpr int kKsgLd = kKsgDim + 4;  // LDS row stride: 17 16-byte bank groups

// 32 x 32 tile of both distance matrices (blockIdx.y chooses), tile pairs of
// the upper triangle only: |a - b| = |b - a|, and a maximum has no order, so
// the mirrored tile is the same values.  What bounds it is the vector ALU: per
// pair and two dimensions two subtractions and one three-way maximum of
// absolute values, 20 us for two matrices of 1024 samples in 512 dimensions.
// Hence
// * small tiles, because 1024 samples give 528 pairs of them a matrix (136 of
//   64 x 64, which leaves most CUs idle in a second round);
// * the four waves of a tile share out the dimensions, not the pairs: each
//   lane keeps 4 x 4 pairs for its 16-byte LDS reads, and the partial maxima
//   are combined once at the end;
// * rows stay row-major in LDS (vector stores, and a read of four dimensions
//   of 8 consecutive rows hits 8 different bank groups), the next stage's loads
//   in flight under this one's arithmetic.
// Both matrices: 200 us as 64 x 64 tiles of all pairs, one launch a matrix;
// now 35 us.
template <bool VEC>
__global__ void __launch_bounds__(256) maxnorm_kernel(const float* __restrict__ z, int dz,
                                                      float* __restrict__ Dz,
                                                      const float* __restrict__ y, int dy,
                                                      float* __restrict__ Dy, int c) {
  __shared__ __align__(16) float sx[2][2 * kKsgTile][kKsgLd];  // rows of the i tile, then of the j tile
  const float* x = blockIdx.y ? y : z;
  const int d = blockIdx.y ? dy : dz;
  float* D = blockIdx.y ? Dy : Dz;
  // tile pair (bi <= bj) of the blockIdx.x-th column-wise entry of the triangle
  int bj = (int)((sqrtf(8.0f * (float)blockIdx.x + 1.0f) - 1.0f) * 0.5f);
  while ((long long)bj * (bj + 1) / 2 > (long long)blockIdx.x) --bj;
  while ((long long)(bj + 1) * (bj + 2) / 2 <= (long long)blockIdx.x) ++bj;
  const int bi = (int)(blockIdx.x - (long long)bj * (bj + 1) / 2);
  const int i0 = bi * kKsgTile, j0 = bj * kKsgTile;
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int ti = lane >> 3, tj = lane & 7;  // rows ti + 8 u and tj + 8 v of the two tiles

  // thread t stages dimensions 4 (t % 16) .. + 3 of rows t / 16 + 16 p; rows past
  // the end are read from the last one (their distances are not written) and
  // dimensions past the end are zero on both sides, which leaves a maximum
  // of absolute values
  const int kq = 4 * (t & 15);
  const float* src[4];
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const int r = (t >> 4) + 16 * p;
    src[p] = x + (size_t)min(r < kKsgTile ? i0 + r : j0 + r - kKsgTile, c - 1) * d;
  }
  float4 reg[4];
  auto load = [&](int d0) {
    const int dd = d0 + kq;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      if constexpr (VEC) {  // d a multiple of 4, 16-byte aligned rows
        reg[p] = __builtin_bit_cast(float4, ld_global16_or_zero(src[p] + dd, dd < d));
      } else {
        reg[p] = make_float4(dd < d ? src[p][dd] : 0.f, dd + 1 < d ? src[p][dd + 1] : 0.f,
                             dd + 2 < d ? src[p][dd + 2] : 0.f, dd + 3 < d ? src[p][dd + 3] : 0.f);
      }
    }
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int p = 0; p < 4; ++p) *(float4*)&sx[buf][(t >> 4) + 16 * p][kq] = reg[p];
  };
  float acc[4][4];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[u][v] = 0.0f;
  load(0);
  store(0);
  load(kKsgDim);
  lds_barrier();
  int buf = 0;
  for (int d0 = 0; d0 < d; d0 += kKsgDim, buf ^= 1) {
    store(buf ^ 1);
    load(d0 + 2 * kKsgDim);
    if (d0 + 16 * w < d) {
#pragma unroll
      for (int k = 0; k < 16; k += 4) {
        float4 a[4], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          a[u] = *(const float4*)&sx[buf][ti + 8 * u][16 * w + k];
          b[u] = *(const float4*)&sx[buf][kKsgTile + tj + 8 * u][16 * w + k];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            acc[u][v] = fmaxf(fmaxf(acc[u][v], fabsf(a[u].x - b[v].x)), fabsf(a[u].y - b[v].y));
            acc[u][v] = fmaxf(fmaxf(acc[u][v], fabsf(a[u].z - b[v].z)), fabsf(a[u].w - b[v].w));
          }
      }
    }
    lds_barrier();
  }
  float (*part)[kKsgTile][kKsgTile + 1] = (float (*)[kKsgTile][kKsgTile + 1])&sx[0][0][0];
  static_assert(4 * kKsgTile * (kKsgTile + 1) <= 2 * 2 * kKsgTile * kKsgLd, "partial maxima in LDS");
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int v = 0; v < 4; ++v) part[w][ti + 8 * u][tj + 8 * v] = acc[u][v];
  __syncthreads();
  const int lj = t & 31;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int li = (t >> 5) + 8 * q;
    auto at = [&](int i, int j) {
      return fmaxf(fmaxf(part[0][i][j], part[1][i][j]), fmaxf(part[2][i][j], part[3][i][j]));
    };
    if (i0 + li < c && j0 + lj < c) D[(size_t)(i0 + li) * c + j0 + lj] = at(li, lj);
    if (bi != bj && j0 + li < c && i0 + lj < c) D[(size_t)(j0 + li) * c + i0 + lj] = at(lj, li);
  }
}

// One wave per sample: no barriers, and a row pair is read twice in 256-byte
// pieces (1024 samples: 10.9 to 5.9 us against one workgroup a sample).
// MAXV: length of the lists, at least v.
template <int MAXV>
__global__ void __launch_bounds__(256) ksg_select_kernel(const float* __restrict__ Dz,
                                                         const float* __restrict__ Dy, int c, int v,
                                                         float* __restrict__ eps_out,
                                                         int32_t* __restrict__ counts) {
  const int lane = threadIdx.x & 63;
  const int i = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (i >= c) return;
  const float* rz = Dz + (size_t)i * c;
  const float* ry = Dy + (size_t)i * c;
  // the v smallest joint distances this lane sees, ascending
  float best[MAXV];
#pragma unroll
  for (int q = 0; q < MAXV; ++q) best[q] = INFINITY;
  // entries j0 + lane + 64 k of the sample's two rows, the reads of kBatch of
  // them issued together; the sample itself and entries past the end are
  // infinitely far
  constexpr int kBatch = 8;
  float dz[kBatch], dy[kBatch];
  auto fetch = [&](int j0) {
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const int j = j0 + lane + 64 * k, jj = min(j, c - 1);
      dz[k] = rz[jj];
      dy[k] = ry[jj];
      if (j != jj || j == i) dz[k] = dy[k] = INFINITY;
    }
  };
  for (int j0 = 0; j0 < c; j0 += 64 * kBatch) {
    fetch(j0);
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      float x = fmaxf(dz[k], dy[k]);
#pragma unroll
      for (int q = 0; q < MAXV; ++q) {  // insertion keeps duplicates
        const float lo = fminf(best[q], x);
        x = fmaxf(best[q], x);
        best[q] = lo;
      }
    }
  }
  // v rounds: the smallest head over the wave leaves its list, of the lowest
  // lane where several hold it
  float eps = 0.0f;
  for (int r = 0; r < v; ++r) {
    const float m = wave_reduce(best[0], [](float a, float b) { return fminf(a, b); });
    eps = m;
    const uint64_t holds = __ballot(best[0] == m);
    if (lane == __builtin_ctzll(holds | (1ull << 63))) {
#pragma unroll
      for (int q = 0; q + 1 < MAXV; ++q) best[q] = best[q + 1];
      best[MAXV - 1] = INFINITY;
    }
  }
  int nz = 0, ny = 0;
  for (int j0 = 0; j0 < c; j0 += 64 * kBatch) {
    fetch(j0);
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      nz += dz[k] < eps ? 1 : 0;
      ny += dy[k] < eps ? 1 : 0;
    }
  }
  nz = wave_sum_i(nz);
  ny = wave_sum_i(ny);
  if (lane == 0) {
    if (eps_out) eps_out[i] = eps;
    counts[2 * i] = nz;
    counts[2 * i + 1] = ny;
  }
}

double mutual_info(const float* d_z, size_t dz, const float* d_y, size_t dy, size_t c, uint32_t v,
                   int32_t* d_counts, float* d_eps, hipStream_t s) {
  if (c < 2 || c > 32768) fail(EDPC_E_INVALID_ARG, "number of samples must be in 2..32768");
  if (v < 1 || v >= c || v > (uint32_t)kKsgMaxV) fail(EDPC_E_INVALID_ARG, "v must be in 1..min(16, c - 1)");
  if (dz < 1 || dy < 1 || dz > (1u << 20) || dy > (1u << 20)) fail(EDPC_E_INVALID_ARG, "bad dimension");
  std::vector<int32_t> h(2 * c);
  // One block where it is kept for the next call, else one for each matrix and the
  // counts: a block of up to 64 MiB comes out of a larger allocation of the
  // runtime's (13 us), one above it costs an allocation and a free (270 us, and
  // milliseconds where memory has been in use; 3500 samples: 543 us in one block).
  const size_t dist = (c * c * sizeof(float) + 255) & ~(size_t)255, counts = 2 * c * sizeof(int32_t);
  const bool together = 2 * dist + counts <= kScratchKept;
  Scratch sz(together ? 2 * dist + counts : dist, s);
  std::optional<Scratch> sy, sc;
  if (!together) {
    sy.emplace(dist, s);
    if (!d_counts) sc.emplace(counts, s);
  }
  float* Dz = (float*)sz.get();
  float* Dy = together ? (float*)((char*)Dz + dist) : (float*)sy->get();
  int32_t* cnt = d_counts ? d_counts : (int32_t*)(together ? (char*)Dz + 2 * dist : sc->get());
  const unsigned tiles = (unsigned)((c + kKsgTile - 1) / kKsgTile);
  const dim3 grid(tiles * (tiles + 1) / 2, 2);
  const bool vec = dz % 4 == 0 && dy % 4 == 0 && ((uintptr_t)d_z | (uintptr_t)d_y) % 16 == 0;
  hipLaunchKernelGGL(vec ? maxnorm_kernel<true> : maxnorm_kernel<false>, grid, dim3(256), 0, s, d_z,
                     (int)dz, Dz, d_y, (int)dy, Dy, (int)c);
  const dim3 sgrid((unsigned)((c + 3) / 4));
  hipLaunchKernelGGL(v <= 4 ? ksg_select_kernel<4> : ksg_select_kernel<kKsgMaxV>, sgrid, dim3(256),
                     0, s, Dz, Dy, (int)c, (int)v, d_eps, cnt);
  hip_check(hipGetLastError(), "ksg launch");
  hip_check(hipMemcpyAsync(h.data(), cnt, h.size() * sizeof(int32_t), hipMemcpyDeviceToHost, s),
            "copy");
  hip_check(hipStreamSynchronize(s), "ksg");
  // psi(n) = -gamma + H(n - 1) at integers
  std::vector<double> H(c + 2, 0.0);
  for (size_t m = 1; m < H.size(); ++m) H[m] = H[m - 1] + 1.0 / (double)m;
  const double gamma = 0.57721566490153286061;
  auto psi = [&](size_t n) { return -gamma + H[n - 1]; };
  double sum = 0.0;
  for (size_t i = 0; i < c; ++i) sum += psi((size_t)h[2 * i] + 1) + psi((size_t)h[2 * i + 1] + 1);
  const double mi = psi(v) + psi(c) - sum / (double)c;
  return mi;
}

}  // namespace edpc
