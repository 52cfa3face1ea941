// FP32 matrix products on the gfx950 MFMA; see gemm.h for the contract.
//
// What bounds them: at the sizes of the 8- and 1024-stream models a product is
// a chain of K / 4 MFMA steps on each of a few waves a CU, so the time is the
// launch, the first loads, and whatever keeps the chain waiting.  Hence vector
// LDS stores without conflicts (F32Operand), operands read one set of steps
// ahead, loads without branches that stay in flight across chunks, one
// barrier a chunk.  Measured per launch, before and after (MI355X): 8 rows,
// gated K 256 10.2 to 6.3 us, head K 256 7.2 to 4.5; 1024 rows, gated K 512
// 18.3 to 10.5 (51 TFLOP/s; the chain alone is 3.4 us), adjoint K 512 12.9 to
// 9.8; 16384 rows of the largest model, gated 778 to 635 us (108 TFLOP/s),
// adjoint 780 to 677.  The LDS reads are next: 4-byte operands for every step.
#include "gemm_epi.h"
#include "grad_sums.h"
#include "lds_limit.h"

#include <algorithm>

namespace edpc {

constexpr int kF32Threads = 256;  // 4 waves

template <int MB>
struct F32Mfma;
template <>
struct F32Mfma<32> {  // v_mfma_f32_32x32x2_f32
  static constexpr int KSTEP = 2, NACC = 16;
  typedef f32x16 Acc;
  __device__ static Acc mma(float a, float b, Acc c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
};
template <>
struct F32Mfma<16> {  // v_mfma_f32_16x16x4_f32
  static constexpr int KSTEP = 4, NACC = 4;
  typedef f32x4 Acc;
  __device__ static Acc mma(float a, float b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

// Row / column of accumulator register r of this lane inside an MB x MB block.
template <int MB>
__device__ __forceinline__ int f32_acc_row(int r, int lane) {
  if constexpr (MB == 32) return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
  else return 4 * (lane >> 4) + r;
}
template <int MB>
__device__ __forceinline__ int f32_acc_col(int lane) {
  return lane & (MB - 1);
}

// One operand tile of ROWS rows and BK k values.
//
// An MFMA step takes, of each operand, one value a lane: row lane % MB at
// k = kk + lane / MB.  gfx950's LDS serves 64 four-byte banks, and both
// layouts below give the 64 lanes 64 different banks, with every store a
// 16-byte vector:
// * K-major operands (src[row * ld + k]) stay row-major in LDS with 4 words
//   of padding a row, [ROWS][BK + 4].  Row r starts at bank 4 r, so 16 rows
//   fill the banks with 4 consecutive k values each.  For MB = 32 rows r and
//   r + 16 start at the same bank, and a step takes only two k values: rows
//   with bit 4 set keep the halves of each 4-value vector swapped, which
//   puts their two values on the two banks that the other row leaves free.
//   (Transposing such a tile into a k-major layout, as for the other kind,
//   takes four 4-byte stores a vector, 4-way conflicted: 18.3 against 11.5 us
//   for the gated product of 1024 rows, K = 512, 2 x 256 outputs.)
// * The others (src[k * ld + row]) stay k-major, [BK][ROWS + PAD], with a row
//   stride of MB (mod 2 MB) words, so that the 64 / MB k values of a step
//   start on different multiples of MB banks.
template <int ROWS, int BK, int MB, bool KMAJOR>
struct F32Operand {
  static constexpr int PAD = KMAJOR ? 4 : (3 * MB - ROWS % (2 * MB)) % (2 * MB);
  static constexpr int STRIDE = KMAJOR ? BK + PAD : ROWS + PAD;
  static constexpr int ELEMS = KMAJOR ? ROWS * STRIDE : BK * STRIDE;
  static constexpr int VROW = (KMAJOR ? BK : ROWS) / 4;  // vectors per LDS row
  static constexpr int NVEC = ROWS * BK / 4;
  static constexpr int PER = (NVEC + kF32Threads - 1) / kF32Threads;
  static_assert(STRIDE % 4 == 0 && BK % 4 == 0 && ROWS % 4 == 0, "16-byte vectors");

  struct Regs {
    uint4 v[PER];
  };
  // This thread's byte offsets from the chunk's first element (row row0 at
  // k0): they are the same in every chunk, so a load is a uniform base plus a
  // 32-bit offset.  Rows past the operand's end are read from its last rows:
  // they only reach outputs that are not stored.
  struct Offsets {
    uint32_t o[PER];
  };
  __device__ static __forceinline__ Offsets offsets(int ld, int row0, int rows_valid) {
    Offsets f;
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int v = min((int)threadIdx.x + p * kF32Threads, NVEC - 1);
      const int a = v / VROW, b = 4 * (v % VROW);
      f.o[p] = 4u * (uint32_t)(KMAJOR ? min(a, rows_valid - 1 - row0) * ld + b
                                      : a * ld + min(b, rows_valid - 4 - row0));  // rows in fours
    }
    return f;
  }
  // Chunk k0 .. k0 + BK - 1 of the rows from row0; k values past K are zero.
  // No branch: the compiler then counts the loads in flight exactly.
  __device__ static __forceinline__ void load(Regs& g, const Offsets& f, const float* src, int ld,
                                              int row0, int k0, int K) {
    const __amdgpu_buffer_rsrc_t rs =
        raw_buffer(src + (KMAJOR ? (long long)row0 * ld + k0 : (long long)k0 * ld + row0));
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int v = threadIdx.x + p * kF32Threads;
      const int k = k0 + (KMAJOR ? 4 * (v % VROW) : v / VROW);
      g.v[p] = __builtin_bit_cast(
          uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, k < K ? f.o[p] : kBufferNone, 0, 0));
    }
  }
  __device__ static __forceinline__ void store(const Regs& g, float* lds) {
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int v = threadIdx.x + p * kF32Threads;
      if (NVEC % kF32Threads && v >= NVEC) continue;
      const int a = v / VROW, b = 4 * (v % VROW);
      uint4 x = g.v[p];
      if constexpr (KMAJOR && MB == 32)
        if (a & 16) x = make_uint4(x.z, x.w, x.x, x.y);
      *(uint4*)(lds + a * STRIDE + b) = x;
    }
  }
  // LDS offset of this lane's value of step kk of the block whose first row
  // is `row` (a multiple of MB): lane_base(kk) is one of two values that do
  // not depend on kk beyond kk % 4, the rest is a constant.
  __device__ static __forceinline__ int lane_base(int lane, int half) {
    const int r = lane % MB, k = lane / MB;
    if constexpr (!KMAJOR) return k * STRIDE + r;
    else if constexpr (MB == 16) return r * STRIDE + k;
    else return r * STRIDE + ((k + 2 * half) ^ ((r & 16) >> 3));
  }
  __device__ static constexpr int step_off(int row, int kk) {
    if (!KMAJOR) return kk * STRIDE + row;
    return row * STRIDE + (MB == 32 ? (kk & ~3) : kk);
  }
};

// Tile of BM x BN outputs: WM x WN waves, each TM x TN blocks of MB x MB
// (the remaining waves of the 4 only move operands).  K runs in chunks of BK
// through NBUF LDS buffers, ST chunks in registers.
template <int MB_, int TM_, int TN_, int WM_, int WN_, int BK_, int NBUF_, int ST_>
struct F32Tile {
  static constexpr int MB = MB_, TM = TM_, TN = TN_, WM = WM_, WN = WN_, BK = BK_, NBUF = NBUF_,
                       ST = ST_;
  static constexpr int BM = MB * TM * WM, BN = MB * TN * WN;
  static_assert(WM * WN <= kF32Threads / 64 && (NBUF == 1 || NBUF == 2), "tile");
};

template <class T, bool AK, bool BKM, int NB>
struct F32Compute {
  typedef F32Mfma<T::MB> Op;
  typedef F32Operand<T::BM, T::BK, T::MB, AK> OA;
  typedef F32Operand<T::BN, T::BK, T::MB, BKM> OB;
  static constexpr int BUF = OA::ELEMS + NB * OB::ELEMS;  // floats per LDS buffer
  static constexpr int SMEM = T::NBUF * BUF * 4;
  // MFMA steps per operand set (see run) and sets per chunk: a quarter of the
  // chunk, or an eighth where that is more than 24 registers a set
  static constexpr int STEPS = T::BK / Op::KSTEP;
  static constexpr int G = STEPS / 4 * (T::TM + NB * T::TN) <= 24 ? STEPS / 4 : STEPS / 8;
  static constexpr int SETS = STEPS / G;
  static_assert(SETS % 2 == 0 && SETS * G == STEPS, "operand sets");
  typename Op::Acc acc[NB][T::TM][T::TN];

  __device__ __forceinline__ void run(const float* A, int lda, const float* B, int ldb,
                                      long long bstride, int M, int N, int K, int m0, int n0,
                                      float* smem) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / T::WN, wn = wave % T::WN;
    const bool computes = T::WM * T::WN == kF32Threads / 64 || wave < T::WM * T::WN;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int i = 0; i < T::TM; ++i)
#pragma unroll
        for (int j = 0; j < T::TN; ++j)
#pragma unroll
          for (int r = 0; r < Op::NACC; ++r) acc[b][i][j][r] = 0.0f;

    if (K <= 0) return;
    typename OA::Regs ra[T::ST];
    typename OB::Regs rb[T::ST][NB];
    const typename OA::Offsets oa = OA::offsets(lda, m0, M);
    const typename OB::Offsets ob = OB::offsets(ldb, n0, N);
    auto load = [&](int q, int c) {
      OA::load(ra[q], oa, A, lda, m0, c * T::BK, K);
#pragma unroll
      for (int b = 0; b < NB; ++b) OB::load(rb[q][b], ob, B + b * bstride, ldb, n0, c * T::BK, K);
    };
    auto store = [&](int q, float* buf) {
      OA::store(ra[q], buf);
#pragma unroll
      for (int b = 0; b < NB; ++b) OB::store(rb[q][b], buf + OA::ELEMS + b * OB::ELEMS);
    };
    const int a0 = OA::lane_base(lane, 0) + wm * T::TM * OA::step_off(T::MB, 0);
    const int a1 = OA::lane_base(lane, 1) + wm * T::TM * OA::step_off(T::MB, 0);
    const int b0 = OA::ELEMS + OB::lane_base(lane, 0) + wn * T::TN * OB::step_off(T::MB, 0);
    const int b1 = OA::ELEMS + OB::lane_base(lane, 1) + wn * T::TN * OB::step_off(T::MB, 0);
    // MFMA operands, in two sets of G steps: one is read from LDS while the
    // other feeds the products (read where they are used, the compiler waits
    // for each pair: the products then stand still for an LDS latency a step)
    float fa[2][G][T::TM], fb[2][G][NB][T::TN];
    auto read = [&](const float* buf, int set) {
#pragma unroll
      for (int s = 0; s < G; ++s) {
        const int kk = (set * G + s) * Op::KSTEP;
        const bool odd = (kk & 2) != 0;
#pragma unroll
        for (int i = 0; i < T::TM; ++i)
          fa[set & 1][s][i] = buf[(odd ? a1 : a0) + OA::step_off(i * T::MB, kk)];
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int j = 0; j < T::TN; ++j)
            fb[set & 1][s][b][j] =
                buf[b * OB::ELEMS + (odd ? b1 : b0) + OB::step_off(j * T::MB, kk)];
      }
    };
    auto mma = [&](int set) {
#pragma unroll
      for (int s = 0; s < G; ++s)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int j = 0; j < T::TN; ++j)
#pragma unroll
            for (int i = 0; i < T::TM; ++i)
              acc[b][i][j] = Op::mma(fa[set & 1][s][i], fb[set & 1][s][b][j], acc[b][i][j]);
    };

    const int nc = (K + T::BK - 1) / T::BK;
#pragma unroll
    for (int q = 0; q < T::ST; ++q)
      load(q, q);
    store(0, smem);
    load(0, T::ST);
    lds_barrier();
    if (computes) read(smem, 0);
    for (int cb = 0;; cb += T::ST) {
#pragma unroll
      for (int q = 0; q < T::ST; ++q) {
        const int c = cb + q;
        const int nq = (q + 1) % T::ST;
        const float* cur = smem + (T::NBUF == 2 ? (c & 1) * BUF : 0);
        float* nxt = smem + (T::NBUF == 2 ? ((c + 1) & 1) * BUF : 0);
        auto refill = [&] {  // chunk c + 1 (zeros past the last) to LDS, its registers to a later one
          store(nq, nxt);
          load(nq, c + 1 + T::ST);
        };
#pragma unroll
        for (int set = 0; set < SETS; ++set) {
          if (set + 1 < SETS) {
            if (computes) read(cur, set + 1);
          } else {
            // every wave has this chunk's last operands in registers
            lds_barrier();
            if constexpr (T::NBUF == 1) {
              refill();
              lds_barrier();
            }
            if (computes) read(nxt, 0);
          }
          __builtin_amdgcn_sched_barrier(0);
          if (computes) mma(set);
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (T::NBUF == 2)
            if (set == 0) refill();
        }
        if (c + 1 == nc) return;  // (straight out: the loads in flight are the same on every way round)
      }
    }
  }
};

template <class T, bool AK, bool BKM, int EPI, int NB>
__global__ void __launch_bounds__(kF32Threads) gemm_fp32_kernel(GemmArgs g) {
  typedef F32Compute<T, AK, BKM, NB> FC;
  typedef typename FC::Op Op;
  extern __shared__ __align__(16) char smem[];
  const int M = g.m_rows ? g.st->rows : g.M;
  const int K = g.k_rows ? g.st->rows : g.K;
  const int N = g.N;
  const int tile = xcd_tile(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
  const int m0 = (tile / gridDim.x) * T::BM, n0 = (tile % gridDim.x) * T::BN;
  if (m0 >= M) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / T::WN, wn = wave % T::WN;
  auto row = [&](int i, int r) { return m0 + (wm * T::TM + i) * T::MB + f32_acc_row<T::MB>(r, lane); };
  auto col = [&](int j) { return n0 + (wn * T::TN + j) * T::MB + f32_acc_col<T::MB>(lane); };
  // small tiles read the epilogue's operands before the sum, under the loads
  // of the first chunks
  constexpr int PER = T::TM * T::TN * Op::NACC;
  constexpr bool kAhead = PER <= 4;
  EpiOperands<EPI, NB> pre[kAhead ? PER : 1];
  const bool live = wave < T::WM * T::WN;
  FC fc;
  if constexpr (kAhead) {
#pragma unroll
    for (int r = 0; r < Op::NACC; ++r)
      if (live && row(0, r) < M && col(0) < N) pre[r].load(g, row(0, r), col(0));
  }
  fc.run((const float*)g.A, g.lda, (const float*)g.B, g.ldb, g.b_branch_stride, M, N, K, m0, n0,
         (float*)smem);
  if (!live) return;
#pragma unroll
  for (int i = 0; i < T::TM; ++i)
#pragma unroll
    for (int j = 0; j < T::TN; ++j)
#pragma unroll
      for (int r = 0; r < Op::NACC; ++r) {
        const int m = row(i, r), n = col(j);
        if (m >= M || n >= N) continue;
        float v[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) v[b] = fc.acc[b][i][j][r];
        if constexpr (kAhead) {
          epi_element<EPI, NB>(g, m, n, v, pre[r]);
        } else {
          EpiOperands<EPI, NB> p;
          p.load(g, m, n);
          epi_element<EPI, NB>(g, m, n, v, p);
        }
      }
}

// Weight-gradient tiles; the workgroups past them take the embedding gradient and
// the column sums, which are independent of the tiles and would leave most of the
// chip idle in launches of their own (8 streams of a small model: 14.3 us
// in three launches, 5.3 in this one; 333 rows of a mid one 42.3 and 20.9; 1024
// rows 67.7 and 47.7).  Its price: every tile's kernel has the registers of the widest
// embedding gradient, two waves a SIMD where the 32 x 32 tile alone would have six.
template <class T>
__global__ void __launch_bounds__(kF32Threads) wgrad_fp32_kernel(const WgradProblem* __restrict__ probs,
                                                                 int n_probs, int tiles, int emb_blocks,
                                                                 const StepState* st, GradSums gs) {
  typedef F32Compute<T, false, false, 1> FC;
  extern __shared__ __align__(16) char smem[];
  if ((int)blockIdx.x >= tiles) {
    const int i = blockIdx.x - tiles;
    if (i >= emb_blocks) {
      const int c = i - emb_blocks;
      colsum_block(st, gs.jobs, gs.n_jobs, gs.total_cols, gs.col_partial, c % gs.col_blocks, c / gs.col_blocks,
                   (float*)smem);
    } else if (gs.E == 16) {
      emb_grad_block<16>(st->rows, gs.ctx, gs.dx, gs.C, gs.chunk_rows, gs.sub_rows, gs.emb_partial, i, smem);
    } else if (gs.E == 32) {
      emb_grad_block<32>(st->rows, gs.ctx, gs.dx, gs.C, gs.chunk_rows, gs.sub_rows, gs.emb_partial, i, smem);
    } else {
      emb_grad_block<64>(st->rows, gs.ctx, gs.dx, gs.C, gs.chunk_rows, gs.sub_rows, gs.emb_partial, i, smem);
    }
    return;
  }
  const int tile = xcd_tile(blockIdx.x, tiles);
  const int p = find_entry(probs, n_probs, tile, [](const WgradProblem& q) { return q.tile_begin; });
  const WgradProblem pr = probs[p];
  const int t = tile - pr.tile_begin;
  const int m0 = (t / pr.tiles_n) * T::BM, n0 = (t % pr.tiles_n) * T::BN;
  FC fc;
  fc.run((const float*)pr.dout, pr.M, (const float*)pr.in, pr.N, 0, pr.M, pr.N, st->rows, m0, n0,
         (float*)smem);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / T::WN, wn = wave % T::WN;
#pragma unroll
  for (int i = 0; i < T::TM; ++i)
#pragma unroll
    for (int j = 0; j < T::TN; ++j)
#pragma unroll
      for (int r = 0; r < FC::Op::NACC; ++r) {
        const int m = m0 + (wm * T::TM + i) * T::MB + f32_acc_row<T::MB>(r, lane);
        const int n = n0 + (wn * T::TN + j) * T::MB + f32_acc_col<T::MB>(lane);
        if (m < pr.M && n < pr.N) gl(pr.dw)[(long long)m * pr.N + n] = fc.acc[0][i][j][r];
      }
}

// ---------------------------------------------------------------------------
// Dispatch
// ---------------------------------------------------------------------------
template <class T, bool AK, bool BKM, int EPI, int NB>
static hipError_t launch_one(const GemmArgs& g, int grid_m_max, hipStream_t s) {
  typedef F32Compute<T, AK, BKM, NB> FC;
  const dim3 grid((g.N + T::BN - 1) / T::BN, (grid_m_max + T::BM - 1) / T::BM);
  if (grid.x == 0 || grid.y == 0) return hipSuccess;
  static_assert(FC::SMEM <= 160 * 1024, "tile does not fit in LDS");
  if constexpr (FC::SMEM > 64 * 1024) {
    static LdsLimit lds;
    if (const hipError_t e = lds.raise((const void*)gemm_fp32_kernel<T, AK, BKM, EPI, NB>, FC::SMEM); e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((gemm_fp32_kernel<T, AK, BKM, EPI, NB>), grid, dim3(kF32Threads), FC::SMEM, s, g);
  return hipGetLastError();
}

template <class T>
static hipError_t launch_fwd(EpiKind epi, int nb, const GemmArgs& g, int gm, hipStream_t s) {
  if (epi == EPI_STORE) return launch_one<T, true, true, EPI_STORE, 1>(g, gm, s);
  if (epi == EPI_GATE_FWD) {
    if (nb == 1) return launch_one<T, true, true, EPI_GATE_FWD, 1>(g, gm, s);
    if (nb == 2) return launch_one<T, true, true, EPI_GATE_FWD, 2>(g, gm, s);
    if (nb == 3) return launch_one<T, true, true, EPI_GATE_FWD, 3>(g, gm, s);
  }
  return hipErrorInvalidValue;
}
template <class T>
static hipError_t launch_adj(EpiKind epi, const GemmArgs& g, int gm, hipStream_t s) {
  if (epi == EPI_STORE) return launch_one<T, true, false, EPI_STORE, 1>(g, gm, s);
  if (epi == EPI_GATE_BWD) return launch_one<T, true, false, EPI_GATE_BWD, 1>(g, gm, s);
  return hipErrorInvalidValue;
}

// The sums of a product depend on the MFMA alone (one chain of steps per
// output, in k order), so the tile ids fall into two classes, 16 x 16 x 4
// (ids of 32 x 32 to 32 x 64 tiles) and 32 x 32 x 2 (64 x 64 and up), and any
// tile of a class may serve any id of it: the choice below is by the size of
// the product.  Times in us, this tile against the other, MI355X.
typedef F32Tile<16, 1, 1, 1, 1, 128, 2, 2> T16x16;
typedef F32Tile<16, 1, 1, 2, 2, 64, 2, 2> T32x32;
typedef F32Tile<32, 1, 1, 2, 2, 32, 2, 2> T64x64;
typedef F32Tile<32, 2, 1, 2, 2, 64, 1, 1> T128x64;
typedef F32Tile<32, 2, 2, 2, 2, 32, 2, 1> T128x128;

hipError_t launch_gemm_fp32(int tile, bool ak, bool bk, EpiKind epi, int nb, const GemmArgs& g,
                            int gm, hipStream_t s) {
  if (!ak) return hipErrorInvalidValue;
  auto tiles = [&](int t) {
    return (long long)((gm + t - 1) / t) * ((g.N + t - 1) / t);
  };
  if (tile < TILE_64x64) {
    // As long as the 16 x 16 blocks have a CU each (64 tiles of 32 x 32), one wave of
    // products a work-group reads less per CU; past that CUs share two and the larger
    // tile, with half the operands a product, is the better one.  All products of
    // steps of 16 to 640 rows, time of 16 x 16 over 32 x 32: 16 to 64 tiles 0.94 (gated
    // K 512 of two branches, 256 rows: 9.8 against 10.7), 80 to 104 tiles 1.04 (333
    // rows: 11.5 against 10.8), 128 tiles 1.06, 160 to 208 1.2, 320 1.4.  Two kinds of
    // product hold out longer: gated ones of a long K (K 1024: 80 and 96 tiles 0.96, the
    // adjoint 0.92, 128 tiles 1.01 and 0.94, 176 tiles 1.17), and plain forward ones of few
    // columns (K 512 and 1024, 128 or 256 columns: 80 to 104 tiles 0.95, 128 tiles 0.99 to
    // 1.02, 160 tiles 1.13).
    const bool later = epi == EPI_STORE ? bk && g.K >= 512 && g.N <= 256 : g.K >= 1024;
    if (tiles(32) <= (later ? 127 : 64))
      return bk ? launch_fwd<T16x16>(epi, nb, g, gm, s) : launch_adj<T16x16>(epi, g, gm, s);
    return bk ? launch_fwd<T32x32>(epi, nb, g, gm, s) : launch_adj<T32x32>(epi, g, gm, s);
  }
  // Enough tiles to fill the card several times: larger ones.  16384 rows of
  // the largest model: gated K 2048 635 against 699 on 64 x 64 (4000 rows: 182
  // against 177), adjoint K 1024 677 against 733, gated adjoint 368 against
  // 375; the plain forward products stay (K 512: 411 against 438).
  const bool many = tiles(128) >= 512;
  if (bk) {
    if (many && epi == EPI_GATE_FWD) return launch_fwd<T128x64>(epi, nb, g, gm, s);
    return launch_fwd<T64x64>(epi, nb, g, gm, s);
  }
  return many ? launch_adj<T128x128>(epi, g, gm, s) : launch_adj<T64x64>(epi, g, gm, s);
}

template <class T>
static hipError_t launch_w(const WgradProblem* d_probs, int n_probs, int tiles, const StepState* st,
                           const GradSums& gs, int max_rows, hipStream_t s) {
  typedef F32Compute<T, false, false, 1> FC;
  const size_t smem = std::max((size_t)FC::SMEM, emb_lds_bytes(gs.sub_rows, gs.C, gs.E));
  const int emb_blocks = (max_rows + gs.chunk_rows - 1) / gs.chunk_rows;
  const int wgs = tiles + emb_blocks + gs.col_blocks * ((max_rows + kColChunk - 1) / kColChunk);
  if (wgs == 0) return hipSuccess;
  static_assert(FC::SMEM <= 160 * 1024, "tile does not fit in LDS");
  if (smem > 64 * 1024) {
    static LdsLimit lds;
    if (const hipError_t e = lds.raise((const void*)wgrad_fp32_kernel<T>, kLdsBytes); e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((wgrad_fp32_kernel<T>), dim3(wgs), dim3(kF32Threads), smem, s, d_probs, n_probs, tiles,
                     emb_blocks, st, gs);
  return hipGetLastError();
}

hipError_t launch_wgrad_fp32(int tile, const WgradProblem* p, int n, int tt, const StepState* st,
                             const GradSums& gs, int max_rows, hipStream_t s) {
  switch (tile) {  // the table is laid out in tiles of this shape
    case TILE_32x32: return launch_w<T32x32>(p, n, tt, st, gs, max_rows, s);
    case TILE_64x32: return launch_w<F32Tile<16, 2, 1, 2, 2, 64, 2, 2>>(p, n, tt, st, gs, max_rows, s);
    case TILE_32x64: return launch_w<F32Tile<16, 1, 2, 2, 2, 64, 2, 2>>(p, n, tt, st, gs, max_rows, s);
    case TILE_64x64: return launch_w<T64x64>(p, n, tt, st, gs, max_rows, s);
    case TILE_128x64: return launch_w<F32Tile<32, 2, 1, 2, 2, 32, 2, 2>>(p, n, tt, st, gs, max_rows, s);
    case TILE_64x128: return launch_w<F32Tile<32, 1, 2, 2, 2, 32, 2, 2>>(p, n, tt, st, gs, max_rows, s);
    case TILE_128x128: return launch_w<T128x128>(p, n, tt, st, gs, max_rows, s);
  }
  return hipErrorInvalidValue;
}

}  // namespace edpc
