// The FP32 step from the LTE's up product through the head and the coder back to
// dY, one workgroup per 16 rows (gfx950 MFMA).
//
// As launches of their own these 20 products, normalisations and the head take 3 to
// 7 us each at a few rows, most of it launch and first loads: 80 us of a 112 us step
// of 8 streams (2 blocks of 128).  Here the rows stay in LDS, each product's weights
// are requested under the epilogue of the one before, and the whole takes 58 us:
// about 25 us of products, the rest their epilogues, normalisations and the head.
// Every sum has the order and rounding of the separate kernels: results are the same
// bits.
#include "fused_fp32.h"

#include <algorithm>

#include "head_row.h"
#include "lds_limit.h"
#include "ln_row.h"

namespace edpc {

namespace {

constexpr int kWaves = 8, kThreads = 64 * kWaves;
constexpr int kRows = 16;
constexpr int kF = 256;          // features: one float4 a lane and row
constexpr int kLdRow = kF + 4;   // row-major LDS rows

// Accesses to rows [0, rows) of an array, `bytes` in all, at byte offset `at` (+
// soff within the row): past the end they go nowhere and read zeros.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_of(const float* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, (short)0, bytes, kBufferWord3);
}
__device__ __forceinline__ void put(float* base, uint32_t bytes, uint32_t at, uint32_t soff, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rows_of(base, bytes), at, soff, 0);
}
__device__ __forceinline__ void put4(float* base, uint32_t bytes, uint32_t at, f32q v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rows_of(base, bytes), at, 0, 0);
}
__device__ __forceinline__ void put2(float* base, uint32_t bytes, uint32_t at, uint32_t soff, float v0, float v1) {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  __builtin_amdgcn_raw_buffer_store_b64(u32x2{__float_as_uint(v0), __float_as_uint(v1)}, rows_of(base, bytes), at,
                                        soff, 0);
}
__device__ __forceinline__ float2 get2(const float* base, uint32_t bytes, uint32_t at, uint32_t soff) {
  return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rows_of(base, bytes), at, soff, 0));
}

// The thread's number, opaque to the compiler: what is formed from it stays in its
// stage (kept for the whole kernel, the addresses of every stage do not fit the
// registers).
__device__ __forceinline__ int here() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// A row block [16][K] as MFMA operand: the lane (g = lane / 16, m = lane mod 16)
// reads the 4 steps' k = 16 i + 4 s + g at once.
__device__ __forceinline__ int frag_at(int m, int k) {
  return (k >> 4) * 256 + (k & 3) * 64 + 4 * m + ((k >> 2) & 3);
}

// Weights are read as whole 128-byte lines: an L2 request takes as long whatever its
// size, and a CU has at most about 64 in flight (products on 64-byte pieces, without
// the detours below, got 11 to 16 bytes a clock, on lines 27; over the whole kernel,
// epilogues included, 22 to 36 requests are in flight: 18 thousand of 186 clocks at
// 1024 rows, of 295 at 16).
//
// One wave's 16 columns of [16, K] x W^T, W[n][k], NB times (the matrices of a gated
// product, or columns further on), with D groups of 32 k in flight.  A load takes 8 rows of 32 k; the
// wave turns them through its piece of LDS into the instruction's order.
template <int NB>
struct RowProduct {
  static constexpr int D = 2;
  static constexpr int HALF = 256 + 32;      // floats: 16 k of the tile (+ 32: the halves' banks)
  static constexpr int STAGE = 2 * HALF;
  uint4 r[D][NB][2];
  __amdgpu_buffer_rsrc_t rs;
  uint32_t voff, branch, half;  // bytes
  int G;

  // columns 16 t ..; t >= tiles: nothing is read
  __device__ __forceinline__ void start(const float* W, int K, int t, int tiles, int branch_elems) {
    const int lane = here() & 63;
    rs = raw_buffer(W);
    G = K >> 5;
    branch = 4u * (uint32_t)branch_elems;
    half = 32u * (uint32_t)K;
    voff = t >= tiles ? kBufferNone : 4u * (uint32_t)((16 * t + (lane >> 3)) * K + 4 * (lane & 7));
#pragma unroll
    for (int q = 0; q < D; ++q) load(q, q, voff);
  }
  __device__ __forceinline__ void load(int q, int i, uint32_t v) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        r[q][b][h] = __builtin_bit_cast(
            uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, v, b * branch + h * half + 128u * i, 0));
  }
  // Group i + 1 goes through LDS and the loads of group i + 1 + D are issued under
  // the products of group i (left to itself the compiler moves loads down to their
  // use, one round trip after the other).
  __device__ __forceinline__ void run(const float* a, float* stage, f32x4 (&acc)[NB]) {
    const int lane = here() & 63;
    const float* al = a + 4 * lane;
    float* put = stage + ((lane & 7) >> 2) * HALF + 4 * (lane >> 3) + (lane & 3);
    const float* got = stage + 4 * lane;
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32q av[2][2], w[2][2][NB];
    auto ready = [&](int q, int i, int set, uint32_t v_more) {
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint32_t v[4] = {r[q][b][h].x, r[q][b][h].y, r[q][b][h].z, r[q][b][h].w};
#pragma unroll
          for (int e = 0; e < 4; ++e) put[b * STAGE + 64 * e + 32 * h] = __uint_as_float(v[e]);
        }
      load(q, i + D, v_more);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");  // (a wave's LDS accesses are in order)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        av[set][h] = *(const f32q*)(al + 512 * i + 256 * h);
#pragma unroll
        for (int b = 0; b < NB; ++b) w[set][h][b] = *(const f32q*)(got + b * STAGE + h * HALF);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
      __builtin_amdgcn_sched_barrier(0);
    };
    auto mma = [&](int set) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int b = 0; b < NB; ++b)
            acc[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[set][h][s], w[set][h][b][s], acc[b], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    };
    static_assert(D == 2, "operand sets; G is even");
    ready(0, 0, 0, G > D ? voff : kBufferNone);
    int i = 0;
    for (; i + D < G; i += D) {
      ready(1, i + 1, 1, voff);
      mma(0);
      ready(0, i + 2, 0, i + 2 + D < G ? voff : kBufferNone);
      mma(1);
    }
    ready(1, i + 1, 1, kBufferNone);
    mma(0);
    mma(1);
  }
};

// One wave's 32 columns of [16, K] x W, W[k][n]: column 32 t + 2 (lane mod 16) + j
// in acc[j], so a row's loads are a whole line; D groups of 16 k in flight (4: 94 us
// a step of 8 rows, 8: 98, 2: 91.5; what is requested early holds up the epilogue's
// own accesses).
struct ColProduct {
  static constexpr int D = 2;
  uint2 r[D][4];
  __amdgpu_buffer_rsrc_t rs;
  uint32_t voff, ld;  // bytes
  int G;

  __device__ __forceinline__ void start(const float* W, int K, int N, int t, int tiles) {
    const int lane = here() & 63;
    rs = raw_buffer(W);
    G = K >> 4;
    ld = 4u * (uint32_t)N;
    voff = t >= tiles ? kBufferNone : 4u * (uint32_t)((lane >> 4) * N + 32 * t + 2 * (lane & 15));
#pragma unroll
    for (int q = 0; q < D; ++q) load(q, q);
  }
  __device__ __forceinline__ void load(int q, int i) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
      r[q][s] =
          __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(rs, voff, (16u * i + 4u * s) * ld, 0));
  }
  __device__ __forceinline__ void run(const float* a, f32x4 (&acc)[2]) {
    const float* al = a + 4 * (here() & 63);
    acc[0] = acc[1] = f32x4{0.f, 0.f, 0.f, 0.f};
    f32q av[2];
    av[0] = *(const f32q*)al;
    auto mma = [&](int q) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[q & 1][s], __uint_as_float(r[q][s].x), acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[q & 1][s], __uint_as_float(r[q][s].y), acc[1], 0, 0, 0);
      }
    };
    int i = 0;
    auto step = [&](int q, bool more, bool last) {
      if (!last) av[(q + 1) & 1] = *(const f32q*)(al + 256 * (i + q + 1));
      __builtin_amdgcn_sched_barrier(0);
      mma(q);
      if (more) load(q, i + q + D);
      __builtin_amdgcn_sched_barrier(0);
    };
    static_assert(D % 2 == 0, "operand sets");
    for (; i + D < G; i += D)
#pragma unroll
      for (int q = 0; q < D; ++q) step(q, true, false);
#pragma unroll
    for (int q = 0; q < D; ++q) step(q, false, q + 1 == D);
  }
};

}  // namespace

template <int NB>
__global__ void __launch_bounds__(kThreads) fused_fp32_kernel(FusedFp32Args a, StreamIO io) {
  extern __shared__ __align__(16) float lds[];
  const int rows = a.st->rows, r0 = blockIdx.x * kRows;
  if (r0 >= rows) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int L = a.L, H = a.H, KH = NB * H, N = a.n_blocks;
  float* sH = lds;                   // residual stream, then its adjoint: [16][kLdRow]
  float* p = lds + kRows * kLdRow;   // operands, or row-major scratch
  float* q = p + a.buf;
  float* stage = q + a.buf;          // of the forward products: a piece a wave and matrix
  float* stage_f = stage + wave * 2 * RowProduct<2>::STAGE;
  float* stage_g = stage + wave * NB * RowProduct<2>::STAGE;
  const uint32_t bF = 4u * (uint32_t)(rows * kF), bH = 4u * (uint32_t)(rows * H), bKH = NB * bH;
  // where a lane works, formed anew in each stage
  struct Pos {
    // of a product: rows 4 g + e of the block (r + e of the step); columns n + 128 c,
    // or the adjoint's columns n2 + c
    int lane, g, n, n2, r;
    // byte offset of element e in an array of W columns
    __device__ uint32_t at(int e, int W) const { return 4u * (uint32_t)(r * W + n) + 4u * (uint32_t)(e * W); }
    __device__ uint32_t at2(int e, int W) const { return 4u * (uint32_t)(r * W + n2) + 4u * (uint32_t)(e * W); }
  };
  auto pos = [&] {
    Pos P;
    P.lane = here() & 63;
    P.g = P.lane >> 4;
    P.n = 16 * wave + (P.lane & 15);
    P.n2 = 32 * wave + 2 * (P.lane & 15);
    P.r = r0 + 4 * P.g;
    return P;
  };
  // row-wise passes: the wave's rows wave + 8 v, columns 4 lane ..
  auto row_of = [&](int v) { return r0 + wave + kWaves * v; };
  auto row_at = [&](int v, int lane) { return 4u * (uint32_t)(row_of(v) * kF + 4 * lane); };

  // The weights of the next product are on their way before the epilogue of the
  // one before.
  RowProduct<2> fw;
  RowProduct<NB> gt;
  ColProduct bw;
  constexpr int kHalf = 128;  // the second 16 columns of a wave lie so far on
  static_assert(kF == kLnRow && kF == 2 * kHalf && kWaves * 16 == kHalf, "two times 16 columns a wave");

  fw.start(a.w2, L, wave, kWaves, kHalf * L);
  for (int k = threadIdx.x; k < kRows * L; k += kThreads) {
    const int m = k / L, j = k - m * L;
    p[frag_at(m, j)] = r0 + m < rows ? a.y[(size_t)(r0 + m) * L + j] : 0.f;
  }
  f32q gm, bt;  // of the next LayerNorm
  auto affine = [&](int j) {
    const int lane = here() & 63;
    gm = *(const f32q*)(a.gamma.of(j) + 4 * lane);
    bt = *(const f32q*)(a.beta.of(j) + 4 * lane);
  };
  lds_barrier();
  {  // Eq. 16
    const Pos P = pos();
    f32x4 acc[2];
    const float bias[2] = {a.b2[P.n], a.b2[P.n + kHalf]};
    fw.run(p, stage_f, acc);
    if (N) {
      gt.start(a.w0.of(0), kF, wave, H / 16, H * kF);
      affine(0);
    } else {
      fw.start(a.wh, kF, wave, kWaves, kHalf * kF);
    }
    float* h = N ? a.h.of(0) : a.hn;
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const float v = acc[c][e] + bias[c];
        sH[(4 * P.g + e) * kLdRow + P.n + kHalf * c] = v;
        if (!N) q[frag_at(4 * P.g + e, P.n + kHalf * c)] = v;
        put(h, bF, P.at(e, kF), 4u * kHalf * c, v);
      }
  }
  lds_barrier();
  for (int j = 0; j < N; ++j) {
    {  // LayerNorm
      const int lane = here() & 63;
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        float mu, rs;
        const f32q z =
            ln_row_fwd(*(const f32q*)(sH + (wave + kWaves * v) * kLdRow + 4 * lane), gm, bt, &mu, &rs);
#pragma unroll
        for (int e = 0; e < 4; ++e) q[frag_at(wave + kWaves * v, 4 * lane + e)] = z[e];
        put4(a.z.of(j), bF, row_at(v, lane), z);
        if (row_of(v) < rows && lane == 0) {
          a.mean.of(j)[row_of(v)] = mu;
          a.rstd.of(j)[row_of(v)] = rs;
        }
      }
    }
    lds_barrier();
    if (16 * wave < H) {  // Eqs. 10-12
      const Pos P = pos();
      f32x4 acc[NB];
      float bias[NB];
      const float* b0 = a.b0.of(j);
#pragma unroll
      for (int b = 0; b < NB; ++b) bias[b] = b0[b * H + P.n];
      gt.run(q, stage_g, acc);
      fw.start(a.wo.of(j), H, wave, kWaves, kHalf * H);
      float *abr = a.abr.of(j), *gp = a.g.of(j);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float prod = 1.0f;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const float v = acc[b][e] + bias[b];
          put(abr, bKH, P.at(e, KH), 4u * b * H, v);
          prod = b == 0 ? v : prod * v;
        }
        const float v = gelu_f(prod);
        p[frag_at(4 * P.g + e, P.n)] = v;
        put(gp, bH, P.at(e, H), 0, v);
      }
    } else {
      fw.start(a.wo.of(j), H, wave, kWaves, kHalf * H);
    }
    lds_barrier();
    {  // Eq. 13
      const Pos P = pos();
      f32x4 acc[2];
      const float* bo = a.bo.of(j);
      const float bias[2] = {bo[P.n], bo[P.n + kHalf]};
      const bool last = j + 1 == N;
      fw.run(p, stage_f, acc);
      if (last) {
        fw.start(a.wh, kF, wave, kWaves, kHalf * kF);
      } else {
        gt.start(a.w0.of(j + 1), kF, wave, H / 16, H * kF);
        affine(j + 1);
      }
      float* h = last ? a.hn : a.h.of(j + 1);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          float* sh = sH + (4 * P.g + e) * kLdRow + P.n + kHalf * c;
          const float v = (acc[c][e] + bias[c]) + *sh;
          *sh = v;
          if (last) q[frag_at(4 * P.g + e, P.n + kHalf * c)] = v;
          put(h, bF, P.at(e, kF), 4u * kHalf * c, v);
        }
    }
    lds_barrier();
  }
  {  // logits
    const Pos P = pos();
    f32x4 acc[2];
    const float bias[2] = {a.bh[P.n], a.bh[P.n + kHalf]};
    fw.run(q, stage_f, acc);
    if (a.head.want_grad) bw.start(a.wh, 256, kF, wave, kF / 32);
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int c = 0; c < 2; ++c) p[(4 * P.g + e) * kLdRow + P.n + kHalf * c] = acc[c][e] + bias[c];
  }
  lds_barrier();
  // Eqs. 1, 2 and the coder, a wave a row
#pragma unroll 1
  for (int v = 0; v < 2; ++v) {
    const int lane = here() & 63;
    f32q d4 = f32q{0.f, 0.f, 0.f, 0.f};
    if (row_of(v) < rows) {
      const f32q zv = *(const f32q*)(p + (wave + kWaves * v) * kLdRow + 4 * lane);
      const float z[4] = {zv[0], zv[1], zv[2], zv[3]};
      float pr[4];
      int x = 0;
      const bool have_target = head_row(a.st, a.head, io, row_of(v), lane, z, pr, &x);
      if (have_target && a.head.want_grad) {
        const float ir = a.st->inv_rows;
#pragma unroll
        for (int e = 0; e < 4; ++e) d4[e] = (pr[e] - (4 * lane + e == x ? 1.0f : 0.0f)) * ir;
        put4(a.head.dz32, bF, row_at(v, lane), d4);
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) q[frag_at(wave + kWaves * v, 4 * lane + e)] = d4[e];
  }
  if (!a.head.want_grad) return;
  lds_barrier();
  {  // adjoint of the head
    const Pos P = pos();
    f32x4 acc[2];
    bw.run(q, acc);
    if (N) bw.start(a.wo.of(N - 1), kF, H, wave, H / 32);
    else bw.start(a.w2, kF, L, wave, L / 32);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        sH[(4 * P.g + e) * kLdRow + P.n2 + c] = acc[c][e];
        p[frag_at(4 * P.g + e, P.n2 + c)] = acc[c][e];
      }
      put2(a.dhn, bF, P.at2(e, kF), 0, acc[0][e], acc[1][e]);
    }
  }
  // (the global stores too: what the forward pass stored is read back, by other waves)
  __syncthreads();
  for (int j = N - 1; j >= 0; --j) {
    if (32 * wave < H) {  // p: adjoint of the block's output -> q: of the branches
      const Pos P = pos();
      float2 v[4][NB];
      const float* abr = a.abr.of(j);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int b = 0; b < NB; ++b) v[e][b] = get2(abr, bKH, P.at2(e, KH), 4u * b * H);
      f32x4 acc[2];
      bw.run(p, acc);
      bw.start(a.w0.of(j), KH, kF, wave, kF / 32);
      float* da = a.da.of(j);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float o[NB][2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          float x[NB], prod = 1.0f;
#pragma unroll
          for (int b = 0; b < NB; ++b) {
            x[b] = c ? v[e][b].y : v[e][b].x;
            prod = b == 0 ? x[b] : prod * x[b];
          }
          const float dp = acc[c][e] * gelu_grad_f(prod);
#pragma unroll
          for (int b = 0; b < NB; ++b) {
            o[b][c] = dp;
#pragma unroll
            for (int k = 0; k < NB; ++k)
              if (k != b) o[b][c] *= x[k];
            q[frag_at(4 * P.g + e, b * H + P.n2 + c)] = o[b][c];
          }
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) put2(da, bKH, P.at2(e, KH), 4u * b * H, o[b][0], o[b][1]);
      }
    } else {
      bw.start(a.w0.of(j), KH, kF, wave, kF / 32);
    }
    f32q x[2];
    float mu[2], rs[2];
    {
      const int lane = here() & 63;
      const float* h = a.h.of(j);
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        x[v] = __builtin_bit_cast(f32q, __builtin_amdgcn_raw_buffer_load_b128(rows_of(h, bF), row_at(v, lane), 0, 0));
        mu[v] = row_of(v) < rows ? a.mean.of(j)[row_of(v)] : 0.f;
        rs[v] = row_of(v) < rows ? a.rstd.of(j)[row_of(v)] : 0.f;
      }
      gm = *(const f32q*)(a.gamma.of(j) + 4 * lane);
    }
    lds_barrier();
    {  // q -> p: adjoint of the LayerNorm's output, row-major
      const Pos P = pos();
      f32x4 acc[2];
      bw.run(q, acc);
      if (j) bw.start(a.wo.of(j - 1), kF, H, wave, H / 32);
      else bw.start(a.w2, kF, L, wave, L / 32);
      float* dz = a.dz.of(j);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
#pragma unroll
        for (int c = 0; c < 2; ++c) p[(4 * P.g + e) * kLdRow + P.n2 + c] = acc[c][e];
        put2(dz, bF, P.at2(e, kF), 0, acc[0][e], acc[1][e]);
      }
    }
    lds_barrier();
    {  // LayerNorm's adjoint; -> sH and q
      const int lane = here() & 63;
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const int m = wave + kWaves * v;
        const f32q o = ln_row_bwd(x[v], mu[v], rs[v], gm, *(const f32q*)(p + m * kLdRow + 4 * lane),
                                  *(const f32q*)(sH + m * kLdRow + 4 * lane));
        *(f32q*)(sH + m * kLdRow + 4 * lane) = o;
#pragma unroll
        for (int e = 0; e < 4; ++e) q[frag_at(m, 4 * lane + e)] = o[e];
        put4(a.dh.of(j), bF, row_at(v, lane), o);
      }
    }
    lds_barrier();
    float* t = p;
    p = q;
    q = t;
  }
  if (32 * wave < L) {  // adjoint of Eq. 16
    const Pos P = pos();
    f32x4 acc[2];
    bw.run(p, acc);
#pragma unroll
    for (int e = 0; e < 4; ++e) put2(a.dy, 4u * (uint32_t)(rows * L), P.at2(e, L), 0, acc[0][e], acc[1][e]);
  }
}

static int fused_fp32_buf(int L, int H, int branches) {  // floats of an operand buffer
  return std::max(kRows * kLdRow, kRows * std::max(L, branches * H));
}
static int fused_fp32_lds(int L, int H, int branches) {
  return 4 * (kRows * kLdRow + 2 * fused_fp32_buf(L, H, branches) +
              kWaves * std::max(2, branches) * RowProduct<2>::STAGE);
}

bool fused_fp32_supported(int F, int L, int H, int branches) {
  return F == kF && L % 64 == 0 && L <= 256 && H % 64 == 0 && H <= 128 && branches >= 1 && branches <= 3 &&
         fused_fp32_lds(L, H, branches) <= 160 * 1024;
}

hipError_t launch_fused_fp32(FusedFp32Args a, int branches, const StreamIO& io, int max_rows, hipStream_t s) {
  a.buf = fused_fp32_buf(a.L, a.H, branches);
  const int smem = fused_fp32_lds(a.L, a.H, branches);
  const dim3 grid((max_rows + kRows - 1) / kRows);
  void (*kernel)(FusedFp32Args, StreamIO) = branches == 1   ? fused_fp32_kernel<1>
                                            : branches == 2 ? fused_fp32_kernel<2>
                                                            : fused_fp32_kernel<3>;
  static LdsLimit lds[3];
  if (smem > 64 * 1024)
    if (const hipError_t e = lds[branches - 1].raise((const void*)kernel, kLdsBytes); e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, grid, dim3(kThreads), smem, s, a, io);
  return hipGetLastError();
}

}  // namespace edpc
