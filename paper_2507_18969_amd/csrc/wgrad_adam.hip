// Weight gradients of the row-block step, each tile followed by Adam on its
// parameters and the rewrite of their fragment copies (gfx950 MFMA).
#include "adam.h"
#include "gemm.h"

namespace edpc {

// dW[m][n] = sum over rows k of dout[k][m] in[k][n]: both operands are stored
// with k slowest, so chunks of 64 k go to LDS as they lie and the MFMA operands
// are read transposed (ds_read_b64_tr_b16: 16 lanes, a 4 x 16 block, each lane
// one column of 4).  4 waves as 2 x 2 blocks of MB x MB.  The instruction (MB)
// and ascending k fix the sums, whatever the tile.
//
// A tile's time is that of its memory: 36 bytes a parameter for Adam, and
// 256 MB bytes of operands a chunk, from L2.  So Adam's operands are read before
// the sum, under its first chunks, the tile is the smallest that the instruction
// allows (more workgroups, two or three on a CU), and a chunk costs one barrier.
// 1.83 million parameters (448 tiles), 1024 rows: 21.5 us, and 14.3 at 16 rows,
// against 33.2 and 17.5 us for 128 x 64 tiles transposed in registers that read
// Adam's operands after the sum.  (Adam's reads after the sum: 22.1 and 15.1 us;
// four chunks ahead instead of two: the same.)
template <int MB>
struct WaTile {
  static constexpr int EDGE = 2 * MB;
  static constexpr int T = 256;               // threads
  static constexpr int BK = 64;               // k per chunk
  static constexpr int CPR = EDGE / 8;        // 16-byte pieces a row of a chunk
  static constexpr int RP = T / CPR;          // rows a pass
  static constexpr int PASS = BK / RP;
  static constexpr int ST = 2;                // chunks in flight in registers
  // LDS row stride, bytes.  192: the 4 rows of a transposed read start 0, 192,
  // 128, 64 bytes into the banks, so 32 lanes of 8 bytes hit every bank once.
  static constexpr int ROW = EDGE == 64 ? 192 : 96;
  static constexpr int OPER = BK * ROW;       // one operand's chunk
  static constexpr int LDG = EDGE + 4, LDT = EDGE + 8;
  static constexpr int EPI = EDGE * LDG * 4 + EDGE * LDT * 2;
  static constexpr int LDS = 4 * OPER > EPI ? 4 * OPER : EPI;
  // Row of a chunk that thread t moves: 8 lanes a row, and rows 2 apart in the
  // 16 lanes of a store (2 x 192 bytes is half the banks further on).
  __device__ static int row_of(int t) {
    const int u = t / CPR;
    return EDGE == 64 ? (u & ~3) | ((u & 1) << 1) | ((u >> 1) & 1) : u;
  }
};

template <int MB>
struct WaMma;
template <>
struct WaMma<32> {
  static constexpr int K = 16, N = 16;
  typedef f32x16 Acc;
  __device__ static Acc mma(bf16x8 a, bf16x8 b, Acc c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
  __device__ static int row(int r, int lane) { return 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3); }
};
template <>
struct WaMma<16> {
  static constexpr int K = 32, N = 4;
  typedef f32x4 Acc;
  __device__ static Acc mma(bf16x8 a, bf16x8 b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
  __device__ static int row(int r, int lane) { return 4 * (lane >> 4) + r; }
};

template <int MB>
__global__ void __launch_bounds__(256) wgrad_adam_kernel(const WgradProblem* __restrict__ probs, int n_probs,
                                                         const StepState* __restrict__ st, WgradAdam ad) {
  typedef WaTile<MB> W;
  constexpr int EDGE = W::EDGE;
  typedef WaMma<MB> Op;
  __shared__ __align__(16) char smem[W::LDS];
  if ((int)blockIdx.x >= ad.tiles) {  // an element-range Adam item
    const int it = blockIdx.x - ad.tiles;
    const int j = find_entry(ad.ejobs, ad.n_ejobs, it, [](const AdamJob& a) { return a.item_begin; });
    const AdamJob jb = ad.ejobs[j];
    adam_elements(st, jb, it - jb.item_begin, ad.p, ad.g, ad.m, ad.v, ad.ac, ad.ac.lr / st->bc1,
                  1.0f / st->bc2);
    return;
  }
  const int tile = xcd_tile(blockIdx.x, ad.tiles);
  const WgradProblem pr =
      probs[find_entry(probs, n_probs, tile, [](const WgradProblem& p) { return p.tile_begin; })];
  const int t = tile - pr.tile_begin;
  const int m0 = (t / pr.tiles_n) * EDGE, n0 = (t % pr.tiles_n) * EDGE;
  const int K = st->rows;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave >> 1, wn = wave & 1;

  // staging: the thread's pieces of a chunk, byte offsets from the operand
  const int srow = W::row_of(threadIdx.x), spiece = threadIdx.x % W::CPR;
  const auto ra = raw_buffer(pr.dout), rb = raw_buffer(pr.in);
  const bool oka = m0 + 8 * spiece < pr.M, okb = n0 + 8 * spiece < pr.N;
  uint4 sa[W::ST][W::PASS], sb[W::ST][W::PASS];
  auto load = [&](int q, int c) {
#pragma unroll
    for (int p = 0; p < W::PASS; ++p) {
      const int k = c * W::BK + p * W::RP + srow;
      const uint32_t oa = (uint32_t)(k * pr.M + m0 + 8 * spiece) * 2u;
      const uint32_t ob = (uint32_t)(k * pr.N + n0 + 8 * spiece) * 2u;
      sa[q][p] = __builtin_bit_cast(
          uint4, __builtin_amdgcn_raw_buffer_load_b128(ra, k < K && oka ? oa : kBufferNone, 0, 0));
      sb[q][p] = __builtin_bit_cast(
          uint4, __builtin_amdgcn_raw_buffer_load_b128(rb, k < K && okb ? ob : kBufferNone, 0, 0));
    }
  };
  const int soff = srow * W::ROW + 16 * spiece;
  auto store = [&](int q, char* buf) {
#pragma unroll
    for (int p = 0; p < W::PASS; ++p) {
      *(uint4*)(buf + soff + p * W::RP * W::ROW) = sa[q][p];
      *(uint4*)(buf + W::OPER + soff + p * W::RP * W::ROW) = sb[q][p];
    }
  };
  // operands: lane's 8 k from kb, of column (lane mod MB) of a block
  const int lk = 8 * (lane / MB) + ((lane & 15) >> 2), lc = (lane & 16 & (MB - 1)) + 4 * (lane & 3);
  const int fa0 = lk * W::ROW + 2 * (wm * MB + lc);
  const int fb0 = W::OPER + lk * W::ROW + 2 * (wn * MB + lc);
  auto frag = [&](const char* p) { return lds_frag_tr(p, p + 4 * W::ROW); };
  constexpr int KS = W::BK / Op::K;
  typename Op::Acc acc;
#pragma unroll
  for (int r = 0; r < Op::N; ++r) acc[r] = 0.0f;

  const int nc = (K + W::BK - 1) / W::BK;
#pragma unroll
  for (int q = 0; q < W::ST; ++q) load(q, q);

  // Adam's operands: items of 8 consecutive columns of a row
  constexpr int CH = EDGE / 8, ITEMS = EDGE * CH, PER = (ITEMS + W::T - 1) / W::T;
  const size_t base = (size_t)(pr.dw - ad.g);  // element offset of the matrix
  float P[PER][8], Mo[PER][8], V[PER][8];
  size_t o[PER];
  bool ok[PER];
  int rl[PER], cl[PER];
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    const int idx = (int)threadIdx.x + k * W::T;
    rl[k] = idx / CH;
    cl[k] = 8 * (idx % CH);
    ok[k] = idx < ITEMS && m0 + rl[k] < pr.M && n0 + cl[k] < pr.N;
    // an item outside the matrix loads its element 0 and stores nothing
    o[k] = ok[k] ? (size_t)(m0 + rl[k]) * pr.N + n0 + cl[k] : 0;
    adam8_load(ad.p + base + o[k], ad.m + base + o[k], ad.v + base + o[k], P[k], Mo[k], V[k]);
  }

  store(0, smem);
  load(0, W::ST);
  lds_barrier();
  static_assert(W::ST % 2 == 0, "buffer parity");
  for (int c = 0; c < nc;) {
#pragma unroll
    for (int q = 0; q < W::ST; ++q) {
      const char* cur = smem + (q & 1) * 2 * W::OPER;
      bf16x8 fa[KS], fb[KS];
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        fa[s] = frag(cur + fa0 + s * Op::K * W::ROW);
        fb[s] = frag(cur + fb0 + s * Op::K * W::ROW);
      }
      store((q + 1) % W::ST, smem + ((q + 1) & 1) * 2 * W::OPER);  // chunk c + 1 (zeros past the last)
      load((q + 1) % W::ST, c + 1 + W::ST);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < KS; ++s) acc = Op::mma(fa[s], fb[s], acc);
      __builtin_amdgcn_sched_barrier(0);
      lds_barrier();
      if (++c >= nc) break;
    }
  }

  float* sG = (float*)smem;
  bf16_t* sT = (bf16_t*)(smem + EDGE * W::LDG * 4);
  const float lr_bc = ad.ac.lr / st->bc1;
  const float inv_bc2 = 1.0f / st->bc2;
#pragma unroll
  for (int r = 0; r < Op::N; ++r)
    sG[(wm * MB + Op::row(r, lane)) * W::LDG + wn * MB + (lane & (MB - 1))] = acc[r];
  lds_barrier();
#pragma unroll
  for (int k = 0; k < PER; ++k) {
    if (!ok[k]) continue;
    float gv[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) gv[e] = sG[rl[k] * W::LDG + cl[k] + e];
    st_global16(pr.dw + o[k], __builtin_bit_cast(uint4, make_float4(gv[0], gv[1], gv[2], gv[3])));
    st_global16(pr.dw + o[k] + 4, __builtin_bit_cast(uint4, make_float4(gv[4], gv[5], gv[6], gv[7])));
    // (rounded as the kernels that wrote the containers so far were compiled)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (MB == 16 || e == 0) adam1<true>(P[k][e], Mo[k][e], V[k][e], gv[e], lr_bc, inv_bc2, ad.ac);
      else adam1(P[k][e], Mo[k][e], V[k][e], gv[e], lr_bc, inv_bc2, ad.ac);
    }
    adam8_store(ad.p + base + o[k], ad.m + base + o[k], ad.v + base + o[k], P[k], Mo[k], V[k]);
    const uint4 pk = pack_bf16x8(P[k]);
    const int row = m0 + rl[k], col = n0 + cl[k];
    // nt fragment (nb = row/16, kb = col/32), lane = row%16 + 16*((col%32)/8)
    st_global16(pr.nt + ((size_t)(row >> 4) * (pr.N / 32) + (col >> 5)) * 64 + (row & 15) +
                    16 * ((col & 31) >> 3),
                pk);
    *(uint4*)&sT[rl[k] * W::LDT + cl[k]] = pk;
  }
  lds_barrier();
  // nn fragment (nb = col/16, kb = row/32), lane = col%16 + 16*((row%32)/8):
  // 8 consecutive rows of one column
#pragma unroll
  for (int idx = threadIdx.x; idx < (EDGE / 8) * EDGE; idx += W::T) {
    const int rblk = idx / EDGE, c = idx % EDGE;
    const int row = m0 + 8 * rblk, col = n0 + c;
    if (row >= pr.M || col >= pr.N) continue;
    uint32_t w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
      w[k] = (uint32_t)sT[(8 * rblk + 2 * k) * W::LDT + c] |
             ((uint32_t)sT[(8 * rblk + 2 * k + 1) * W::LDT + c] << 16);
    st_global16(pr.nn + ((size_t)(col >> 4) * (pr.M / 32) + (row >> 5)) * 64 + (col & 15) +
                    16 * ((row & 31) >> 3),
                make_uint4(w[0], w[1], w[2], w[3]));
  }
}

hipError_t launch_wgrad_adam(int edge, const WgradProblem* p, int n, int tiles, int elem_items,
                             const StepState* st, const WgradAdam& ad_in, hipStream_t s) {
  WgradAdam ad = ad_in;
  ad.tiles = tiles;
  const dim3 grid(tiles + elem_items);
  if (grid.x == 0) return hipSuccess;
  if (edge == 64)
    hipLaunchKernelGGL(wgrad_adam_kernel<32>, grid, dim3(256), 0, s, p, n, st, ad);
  else
    hipLaunchKernelGGL(wgrad_adam_kernel<16>, grid, dim3(256), 0, s, p, n, st, ad);
  return hipGetLastError();
}

}  // namespace edpc
