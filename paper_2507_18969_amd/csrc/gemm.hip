// BF16 matrix products on 4-wave tiles (gfx950 MFMA); see gemm.h for the
// contract, gemm_fp32.hip for the FP32 products, gemm_wide.hip for the wide
// tiles.
#include "gemm_epi.h"
#include "lds_limit.h"

namespace edpc {

// 4 waves of 64, arranged 2 x 2 over the tile
constexpr int kThreads = 256;

template <int MB>
struct Mfma;
template <>
struct Mfma<32> {  // v_mfma_f32_32x32x16_bf16
  static constexpr int KSTEP = 16;
  static constexpr int NACC = 16;
  typedef f32x16 Acc;
  typedef bf16x8 Frag;
  __device__ static Acc mma(Frag a, Frag b, Acc c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};
template <>
struct Mfma<16> {  // v_mfma_f32_16x16x32_bf16
  static constexpr int KSTEP = 32;
  static constexpr int NACC = 4;
  typedef f32x4 Acc;
  typedef bf16x8 Frag;
  __device__ static Acc mma(Frag a, Frag b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};

// Row / column of accumulator register r of this lane inside an MB x MB block.
template <int MB>
__device__ __forceinline__ int acc_row(int r, int lane) {
  if constexpr (MB == 32) return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
  else return 4 * (lane >> 4) + r;
}
template <int MB>
__device__ __forceinline__ int acc_col(int lane) {
  return lane & (MB - 1);
}

// ---------------------------------------------------------------------------
// Operand tile staging.  LDS layout: row-major [ROWS][BK + 8], so that one
// lane reads its 8 consecutive k values with a single 16-byte access.  An
// operand stored row-contiguous in memory (k slowest) is moved in 8 x 8 blocks
// that each thread transposes in registers, so LDS still gets 16-byte stores.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void transpose8x8_bf16(const uint4* in, uint4* out) {
  // in[i] holds 8 bf16 of row i (columns 0..7); out[j] gets column j (rows 0..7)
  const uint32_t* w = (const uint32_t*)in;  // w[4 * i + q] = (col 2q, col 2q+1) of row i
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int q = j >> 1;
    const uint32_t sel = (j & 1) ? 0x07060302u : 0x05040100u;
    uint32_t o[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      o[k] = __builtin_amdgcn_perm(w[4 * (2 * k + 1) + q], w[4 * (2 * k) + q], sel);
    out[j] = make_uint4(o[0], o[1], o[2], o[3]);
  }
}

// 8 x 8 block b of a row-contiguous BF16 operand tile with 16 chunks of 8 k
// (BK = 128): row block rb, chunk kb.  The 16 lanes of an LDS store pass take
// 2 adjacent row blocks x 8 chunks: a 272-byte row is 17 16-byte bank groups,
// so the two row blocks start 8 groups apart and the 16 stores fill all 16
// groups of gfx950's 64-bank LDS (one row block x 16 chunks would fill 2).  A
// wave covers 8 row blocks x 8 chunks (ROWS >= 64; 4 x 16 at ROWS = 32), so
// each global load reads whole 128-byte lines (half lines at ROWS = 32, as
// before).
template <int ROWS>
__device__ __forceinline__ void blk_of(int b, int& rb, int& kb) {
  constexpr int U4 = ROWS / 16 < 4 ? ROWS / 16 : 4;  // row-block pairs a wave covers
  const int g = b >> 4, u = (g % U4) + U4 * (g / (2 * U4)), v = (g / U4) & 1;
  rb = 2 * u + ((b >> 3) & 1);
  kb = 8 * v + (b & 7);
}

template <int ROWS, int BK>
struct Stage {
  static constexpr int VEC = 8;                          // elements per 16-byte vector
  static constexpr int NVEC = ROWS * BK / VEC;           // vectors per tile
  static constexpr int PER_THREAD = (NVEC + kThreads - 1) / kThreads;
  static constexpr int NBLK = (ROWS / 8) * (BK / 8);     // 8 x 8 blocks (row-contiguous)
  static_assert(BK == 128 && ROWS % 16 == 0, "blk_of: 16 chunks, row blocks in pairs");
  static constexpr int BLK_PER_THREAD = (NBLK + kThreads - 1) / kThreads;
  static constexpr int NREG = PER_THREAD > 8 * BLK_PER_THREAD ? PER_THREAD : 8 * BLK_PER_THREAD;
  static constexpr int STRIDE = BK + 8;                  // LDS row stride (elements)
  static constexpr int LDS_ELEMS = ROWS * STRIDE;
  uint4 reg[NREG];

  // Global -> registers.  kmajor: src[row * ld + k]; else src[k * ld + row].
  template <bool KMAJOR>
  __device__ __forceinline__ void load(const bf16_t* src, int ld, int row0, int rows_valid, int k0,
                                       int K) {
    if constexpr (!KMAJOR) {
#pragma unroll
      for (int p = 0; p < BLK_PER_THREAD; ++p) {
        const int b = threadIdx.x + p * kThreads;
        int rb, kb;
        blk_of<ROWS>(b, rb, kb);
        const int gr = row0 + rb * 8;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int gk = k0 + kb * 8 + i;
          reg[8 * p + i] = ld_global16_or_zero(src + (long long)gk * ld + gr,
                                               b < NBLK && gr < rows_valid && gk < K);
        }
      }
    } else {
#pragma unroll
      for (int p = 0; p < PER_THREAD; ++p) {
        const int v = threadIdx.x + p * kThreads;
        const int row = v / (BK / VEC), kq = v % (BK / VEC);
        const int gr = row0 + row, gk = k0 + kq * VEC;
        reg[p] = ld_global16_or_zero(src + (long long)gr * ld + gk,
                                     v < NVEC && gr < rows_valid && gk < K);
      }
    }
  }

  template <bool KMAJOR>
  __device__ __forceinline__ void store(bf16_t* lds) {
    if constexpr (!KMAJOR) {
#pragma unroll
      for (int p = 0; p < BLK_PER_THREAD; ++p) {
        const int b = threadIdx.x + p * kThreads;
        if (b >= NBLK) continue;
        int rb, kb;
        blk_of<ROWS>(b, rb, kb);
        uint4 t[8];
        transpose8x8_bf16(&reg[8 * p], t);
#pragma unroll
        for (int j = 0; j < 8; ++j) *(uint4*)(lds + (rb * 8 + j) * STRIDE + kb * 8) = t[j];
      }
    } else {
#pragma unroll
      for (int p = 0; p < PER_THREAD; ++p) {
        const int v = threadIdx.x + p * kThreads;
        if (v >= NVEC) continue;
        const int row = v / (BK / VEC), kq = v % (BK / VEC);
        *(uint4*)(lds + row * STRIDE + kq * 8) = reg[p];
      }
    }
  }
};

template <int MB>
__device__ __forceinline__ bf16x8 frag_read(const bf16_t* lds, int stride, int row_base, int kk,
                                            int lane) {
  const int r = lane % MB, kg = lane / MB;
  return __builtin_bit_cast(bf16x8, *(const uint4*)(lds + (row_base + r) * stride + kk + 8 * kg));
}

template <int BM_, int BN_, int MB_, int TM_, int TN_>
struct TileCfg {
  static constexpr int BM = BM_, BN = BN_, MB = MB_, TM = TM_, TN = TN_;
};

// One output tile (m0, n0) of C = A * B_i for i < NB.
template <class T, bool AK, bool BKM, int NB>
struct TileCompute {
  static constexpr int BK = 128;
  static constexpr int MB = T::MB, TM = T::TM, TN = T::TN;
  typedef Mfma<MB> Op;
  typedef Stage<T::BM, BK> SA;
  typedef Stage<T::BN, BK> SB;
  // two register stages unless that would hold more than 16 vectors a thread
  static constexpr int ST = (SA::NREG + NB * SB::NREG) <= 16 ? 2 : 1;
  typename Op::Acc acc[NB][TM][TN];

  __device__ __forceinline__ void run(const bf16_t* A, int lda, const bf16_t* B, int ldb,
                                      long long bstride, int M, int N, int K, int m0, int n0,
                                      char* smem) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    bf16_t* lds_a = (bf16_t*)smem;
    bf16_t* lds_b = lds_a + SA::LDS_ELEMS;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int r = 0; r < Op::NACC; ++r) acc[b][i][j][r] = 0.0f;

    // ST register stages: tiles k0 .. k0 + (ST-1)*BK are in flight together
    SA sa[ST];
    SB sb[ST][NB];
#pragma unroll
    for (int q = 0; q < ST; ++q) {
      if (q * BK < K) {
        sa[q].template load<AK>(A, lda, m0, M, q * BK, K);
#pragma unroll
        for (int b = 0; b < NB; ++b)
          sb[q][b].template load<BKM>(B + b * bstride, ldb, n0, N, q * BK, K);
      }
    }
    for (int k0 = 0; k0 < K; k0 += ST * BK) {
#pragma unroll
      for (int q = 0; q < ST; ++q) {
        const int kq = k0 + q * BK;
        if (kq < K) {
          __syncthreads();
          sa[q].template store<AK>(lds_a);
#pragma unroll
          for (int b = 0; b < NB; ++b)
            sb[q][b].template store<BKM>(lds_b + b * SB::LDS_ELEMS);
          __syncthreads();
          if (kq + ST * BK < K) {
            sa[q].template load<AK>(A, lda, m0, M, kq + ST * BK, K);
#pragma unroll
            for (int b = 0; b < NB; ++b)
              sb[q][b].template load<BKM>(B + b * bstride, ldb, n0, N, kq + ST * BK, K);
          }
          // keep the loads' consumers (the transposes of the next stores)
          // below the products, so that the loads stay in flight under them
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int kk = 0; kk < BK; kk += Op::KSTEP) {
            typename Op::Frag fa[TM];
#pragma unroll
            for (int i = 0; i < TM; ++i)
              fa[i] = frag_read<MB>(lds_a, SA::STRIDE, (wm * TM + i) * MB, kk, lane);
#pragma unroll
            for (int b = 0; b < NB; ++b) {
#pragma unroll
              for (int j = 0; j < TN; ++j) {
                typename Op::Frag fb = frag_read<MB>(lds_b + b * SB::LDS_ELEMS, SB::STRIDE,
                                                     (wn * TN + j) * MB, kk, lane);
#pragma unroll
                for (int i = 0; i < TM; ++i) acc[b][i][j] = Op::mma(fa[i], fb, acc[b][i][j]);
              }
            }
          }
        }
      }
    }
  }

  static constexpr int smem_bytes() {
    return (SA::LDS_ELEMS + NB * SB::LDS_ELEMS) * 2;
  }
};

template <class T, bool AK, bool BKM, int EPI, int NB>
__global__ void __launch_bounds__(kThreads) gemm_kernel(GemmArgs g) {
  typedef TileCompute<T, AK, BKM, NB> TC;
  extern __shared__ __align__(16) char smem[];
  const int M = g.m_rows ? g.st->rows : g.M;
  const int K = g.k_rows ? g.st->rows : g.K;
  const int N = g.N;
  const int tile = xcd_tile(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  const int m0 = (tile / gridDim.x) * T::BM, n0 = (tile % gridDim.x) * T::BN;
  if (m0 >= M) return;
  TC tc;
  tc.run((const bf16_t*)g.A, g.lda, (const bf16_t*)g.B, g.ldb, g.b_branch_stride, M, N, K, m0, n0,
         smem);

  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave >> 1, wn = wave & 1;
#pragma unroll
  for (int i = 0; i < T::TM; ++i)
#pragma unroll
    for (int j = 0; j < T::TN; ++j)
#pragma unroll
      for (int r = 0; r < TC::Op::NACC; ++r) {
        const int m = m0 + (wm * T::TM + i) * T::MB + acc_row<T::MB>(r, lane);
        const int n = n0 + (wn * T::TN + j) * T::MB + acc_col<T::MB>(lane);
        if (m >= M || n >= N) continue;
        float v[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) v[b] = tc.acc[b][i][j][r];
        EpiOperands<EPI, NB> p;
        p.load(g, m, n);
        epi_element<EPI, NB>(g, m, n, v, p);
      }
}

template <class T>
__global__ void __launch_bounds__(kThreads) wgrad_kernel(const WgradProblem* __restrict__ probs,
                                                         int n_probs, const StepState* st) {
  typedef TileCompute<T, false, false, 1> TC;
  extern __shared__ __align__(16) char smem[];
  const int tile = xcd_tile(blockIdx.x, (int)gridDim.x);
  int p = 0;
  while (p + 1 < n_probs && tile >= probs[p + 1].tile_begin) ++p;
  const WgradProblem pr = probs[p];
  const int t = tile - pr.tile_begin;
  const int m0 = (t / pr.tiles_n) * T::BM, n0 = (t % pr.tiles_n) * T::BN;
  const int K = st->rows;
  TC tc;
  tc.run((const bf16_t*)pr.dout, pr.M, (const bf16_t*)pr.in, pr.N, 0, pr.M, pr.N, K, m0, n0, smem);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave >> 1, wn = wave & 1;
#pragma unroll
  for (int i = 0; i < T::TM; ++i)
#pragma unroll
    for (int j = 0; j < T::TN; ++j)
#pragma unroll
      for (int r = 0; r < TC::Op::NACC; ++r) {
        const int m = m0 + (wm * T::TM + i) * T::MB + acc_row<T::MB>(r, lane);
        const int n = n0 + (wn * T::TN + j) * T::MB + acc_col<T::MB>(lane);
        if (m < pr.M && n < pr.N) gl(pr.dw)[(long long)m * pr.N + n] = tc.acc[0][i][j][r];
      }
}

// ---------------------------------------------------------------------------
// Dispatch
// ---------------------------------------------------------------------------
typedef TileCfg<32, 32, 16, 1, 1> T32x32;
typedef TileCfg<64, 32, 16, 2, 1> T64x32;
typedef TileCfg<32, 64, 16, 1, 2> T32x64;
typedef TileCfg<64, 64, 32, 1, 1> T64x64;
typedef TileCfg<128, 64, 32, 2, 1> T128x64;
typedef TileCfg<64, 128, 32, 1, 2> T64x128;
typedef TileCfg<128, 128, 32, 2, 2> T128x128;

template <class T, bool AK, bool BKM, int EPI, int NB>
static hipError_t launch_one(const GemmArgs& g, int grid_m_max, hipStream_t s) {
  typedef TileCompute<T, AK, BKM, NB> TC;
  dim3 grid((g.N + T::BN - 1) / T::BN, (grid_m_max + T::BM - 1) / T::BM);
  if (grid.x == 0 || grid.y == 0) return hipSuccess;
  constexpr int smem = TC::smem_bytes();
  static_assert(smem <= 160 * 1024, "tile does not fit in LDS");
  if constexpr (smem > 64 * 1024) {
    static LdsLimit lds;
    if (const hipError_t e = lds.raise((const void*)gemm_kernel<T, AK, BKM, EPI, NB>, smem); e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((gemm_kernel<T, AK, BKM, EPI, NB>), grid, dim3(kThreads), smem, s, g);
  return hipGetLastError();
}

template <class T>
static hipError_t launch_t(bool ak, bool bk, EpiKind epi, int nb, const GemmArgs& g, int gm,
                           hipStream_t s) {
  if (ak && bk) {  // forward dense layers
    if (epi == EPI_STORE) return launch_one<T, true, true, EPI_STORE, 1>(g, gm, s);
    if (epi == EPI_GATE_FWD) {
      if (nb == 1) return launch_one<T, true, true, EPI_GATE_FWD, 1>(g, gm, s);
      if (nb == 2) return launch_one<T, true, true, EPI_GATE_FWD, 2>(g, gm, s);
      if (nb == 3) return launch_one<T, true, true, EPI_GATE_FWD, 3>(g, gm, s);
    }
  } else if (ak && !bk) {  // adjoint of the input
    if (epi == EPI_STORE) return launch_one<T, true, false, EPI_STORE, 1>(g, gm, s);
    if (epi == EPI_GATE_BWD) return launch_one<T, true, false, EPI_GATE_BWD, 1>(g, gm, s);
  }
  return hipErrorInvalidValue;
}

static hipError_t launch_p(int tile, bool ak, bool bk, EpiKind epi, int nb, const GemmArgs& g,
                           int gm, hipStream_t s) {
  switch (tile) {
    case TILE_32x32: return launch_t<T32x32>(ak, bk, epi, nb, g, gm, s);
    case TILE_64x32: return launch_t<T64x32>(ak, bk, epi, nb, g, gm, s);
    case TILE_32x64: return launch_t<T32x64>(ak, bk, epi, nb, g, gm, s);
    case TILE_64x64: return launch_t<T64x64>(ak, bk, epi, nb, g, gm, s);
    case TILE_128x64: return launch_t<T128x64>(ak, bk, epi, nb, g, gm, s);
    case TILE_64x128: return launch_t<T64x128>(ak, bk, epi, nb, g, gm, s);
    case TILE_128x128: return launch_t<T128x128>(ak, bk, epi, nb, g, gm, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_gemm(int tile, bool bf16, bool a_kmajor, bool b_kmajor, EpiKind epi, int nb,
                       const GemmArgs& g, int grid_m_max, hipStream_t s) {
  if (tile >= TILE_W128x128) {
    if (!wide_tile_supported(tile, bf16, epi, nb)) return hipErrorInvalidValue;
    return launch_gemm_wide(tile, a_kmajor, b_kmajor, epi, nb, g, grid_m_max, s);
  }
  return bf16 ? launch_p(tile, a_kmajor, b_kmajor, epi, nb, g, grid_m_max, s)
              : launch_gemm_fp32(tile, a_kmajor, b_kmajor, epi, nb, g, grid_m_max, s);
}

template <class T>
static hipError_t launch_w(const WgradProblem* d_probs, int n_probs, int total_tiles,
                           const StepState* st, hipStream_t s) {
  typedef TileCompute<T, false, false, 1> TC;
  if (total_tiles == 0) return hipSuccess;
  constexpr int smem = TC::smem_bytes();
  static_assert(smem <= 160 * 1024, "tile does not fit in LDS");
  if constexpr (smem > 64 * 1024) {
    static LdsLimit lds;
    if (const hipError_t e = lds.raise((const void*)wgrad_kernel<T>, smem); e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((wgrad_kernel<T>), dim3(total_tiles), dim3(kThreads), smem, s,
                     d_probs, n_probs, st);
  return hipGetLastError();
}

static hipError_t launch_wp(int tile, const WgradProblem* p, int n, int tt, const StepState* st,
                            hipStream_t s) {
  switch (tile) {
    case TILE_32x32: return launch_w<T32x32>(p, n, tt, st, s);
    case TILE_64x32: return launch_w<T64x32>(p, n, tt, st, s);
    case TILE_32x64: return launch_w<T32x64>(p, n, tt, st, s);
    case TILE_64x64: return launch_w<T64x64>(p, n, tt, st, s);
    case TILE_128x64: return launch_w<T128x64>(p, n, tt, st, s);
    case TILE_64x128: return launch_w<T64x128>(p, n, tt, st, s);
    case TILE_128x128: return launch_w<T128x128>(p, n, tt, st, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_wgrad(int tile, const WgradProblem* d_probs, int n_probs, int total_tiles,
                        const StepState* st, float* part, hipStream_t s) {
  return tile >= TILE_W128x128 ? launch_wgrad_wide(tile, d_probs, n_probs, total_tiles, st, part, s)
                               : launch_wp(tile, d_probs, n_probs, total_tiles, st, s);
}

}  // namespace edpc
