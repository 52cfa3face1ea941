// Row-wise / element-wise kernels of one model step and the coder lanes.
#include "adam.h"
#include "grad_sums.h"
#include "head_row.h"
#include "ln_row.h"

#include <algorithm>

namespace edpc {

static inline unsigned blocks_for(size_t n, unsigned per) { return (unsigned)((n + per - 1) / per); }

// ---------------------------------------------------------------------------
// Step state
// ---------------------------------------------------------------------------
__global__ void step_set_kernel(StepState* st, int step) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    st->step = step;
    st->base = step;
  }
}

void k_step_set(StepState* st, int step, hipStream_t s) {
  hipLaunchKernelGGL(step_set_kernel, dim3(1), dim3(64), 0, s, st, step);
}

__device__ __forceinline__ void explicit_state(StepState* st, int rows, uint32_t tau, float beta1,
                                              float beta2) {
  st->step = -1;
  st->rows = rows;
  st->inv_rows = rows > 0 ? 1.0f / (float)rows : 0.0f;
  st->model = 1;
  st->tau = tau;
  st->bc1 = adam_bias_correction(beta1, tau);
  st->bc2 = adam_bias_correction(beta2, tau);
}

__global__ void step_explicit_kernel(StepState* st, int rows, uint32_t tau, float beta1,
                                     float beta2) {
  if (threadIdx.x == 0 && blockIdx.x == 0) explicit_state(st, rows, tau, beta1, beta2);
}

void k_step_explicit(StepState* st, int rows, uint32_t tau, float beta1, float beta2,
                     hipStream_t s) {
  hipLaunchKernelGGL(step_explicit_kernel, dim3(1), dim3(64), 0, s, st, rows, tau, beta1, beta2);
}

// ---------------------------------------------------------------------------
// Context window gather and byte embedding
// ---------------------------------------------------------------------------
// X[r][c E + e] = Emb[byte c of row r's context][e], features f, f + step, ..
__device__ __forceinline__ void embed_row(const uint8_t* bytes, const float* __restrict__ emb, int F, int E,
                                          float* __restrict__ x32, bf16_t* __restrict__ x16, size_t r, int f,
                                          int step) {
  for (; f < F; f += step) {
    const int c = f / E, e = f - c * E;
    const float4 val = *(const float4*)(emb + bytes[c] * E + e);
    if (x32) *(float4*)(x32 + r * F + f) = val;
    if (x16)
      *(ushort4*)(x16 + r * F + f) = make_ushort4(f2bf(val.x), f2bf(val.y), f2bf(val.z), f2bf(val.w));
  }
}

// A workgroup takes `per` rows with n threads each: one row, or from 2048 rows on as
// many as fit (below 1024 features one row leaves threads idle, which costs nothing
// while there are CUs to spare: a BF16 prediction of 100000 rows of 64 features 279 us,
// 259 so, of 256 features 433 and 418; 7 rows of 256 44.9 us, 45.1 together).  Up to 512
// rows, wide ones are shared out over workgroups of 1024 features (blockIdx.y): one would
// wait for its rounds of loads in turn (5 rows of 16384 features 145.4 us a prediction,
// 139.8 so; 3000 rows 347 and 357).
__global__ void __launch_bounds__(256) embed_kernel(const StepState* __restrict__ st,
                                                    const uint8_t* __restrict__ ctx,
                                                    const float* __restrict__ emb, int C, int E, int per, int n,
                                                    float* __restrict__ x32, bf16_t* __restrict__ x16) {
  const int i = per > 1 ? threadIdx.x / n : 0, r = blockIdx.x * per + i;
  if (i >= per || r >= st->rows) return;
  embed_row(ctx + (size_t)r * C, emb, C * E, E, x32, x16, r, 1024 * blockIdx.y + 4 * (threadIdx.x - i * n),
            1024 * gridDim.y);
}

void k_embed(const StepState* st, const uint8_t* ctx, const float* emb, int C, int E, float* x32,
             bf16_t* x16, int max_rows, hipStream_t s) {
  const int n = max_rows < 2048 ? 256 : std::min(256, C * E / 4), per = 256 / n;
  const unsigned share = max_rows <= 512 ? blocks_for(C * E, 1024) : 1;
  hipLaunchKernelGGL(embed_kernel, dim3(blocks_for(max_rows, per), share), dim3(256), 0, s, st, ctx, emb, C, E, per,
                     n, x32, x16);
}

// First launch of a coding step of the layer-by-layer sequence: the step state
// (formed and written by the first workgroup; no other reads it here: a row is
// active if its own stream is long enough), the row's context and target from
// its stream, and the embedding.  As launches of their own the three took 6.7 us
// of a 116 us step of 8 streams, this one 3.8.
__global__ void __launch_bounds__(256) embed_streams_kernel(StepState* st, Schedule sc, int mode, int step,
                                                            StreamIO io, int C, int E, bool decoding,
                                                            const float* __restrict__ emb,
                                                            uint8_t* __restrict__ ctx,
                                                            uint8_t* __restrict__ tgt,
                                                            float* __restrict__ x32,
                                                            bf16_t* __restrict__ x16) {
  __shared__ uint8_t bytes[256];
  if (mode == 2) step += st->base;
  const int r = blockIdx.x;
  const uint32_t s = io.slot[r];
  const bool live = sc.lens_sorted[r] > (int64_t)step;
  if (live) {
    const uint8_t* base = decoding ? io.dst : io.src;
    const uint64_t o = io.off[s];
    const int c = threadIdx.x;
    if (c < C) {
      const uint8_t v = base[io_at(io, o, (uint64_t)(step - C + c))];
      bytes[c] = v;
      ctx[(size_t)r * C + c] = v;
    }
    if (!decoding && c == 0) tgt[r] = io.src[io_at(io, o, (uint64_t)step)];
    __syncthreads();
    embed_row(bytes, emb, C * E, E, x32, x16, r, 4 * threadIdx.x, 1024);
  }
  if (r == 0) {
    const int rows = active_rows(sc, step);
    if (threadIdx.x == 0) write_step_state(st, sc, step, rows);
  }
}

void k_embed_streams(StepState* st, const Schedule& sc, int mode, int step, const StreamIO& io, int C,
                     int E, bool decoding, const float* emb, uint8_t* ctx, uint8_t* tgt, float* x32,
                     bf16_t* x16, int max_rows, hipStream_t s) {
  hipLaunchKernelGGL(embed_streams_kernel, dim3(max_rows), dim3(256), 0, s, st, sc, mode, step, io, C, E,
                     decoding, emb, ctx, tgt, x32, x16);
}

// Inputs of a step on explicit contexts in one launch: the step state, contexts
// and targets, and the slots, which come as kernel arguments (three copies and a
// launch otherwise, the one of the slots from host memory).
__global__ void __launch_bounds__(256) stage_kernel(StepState* st, int rows, uint32_t tau, float beta1,
                                                    float beta2, const uint8_t* __restrict__ src_ctx,
                                                    uint8_t* __restrict__ ctx, int n_ctx,
                                                    const uint8_t* __restrict__ src_tgt,
                                                    uint8_t* __restrict__ tgt, InlineSlots slots,
                                                    uint32_t* __restrict__ slot) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n_ctx) ctx[i] = src_ctx[i];
  if (i >= rows) return;
  if (src_tgt) tgt[i] = src_tgt[i];
  slot[i] = slots.v[i];
  if (i == 0) explicit_state(st, rows, tau, beta1, beta2);
}

void k_stage(StepState* st, int rows, uint32_t tau, float beta1, float beta2, const uint8_t* src_ctx,
             uint8_t* ctx, int C, const uint8_t* src_tgt, uint8_t* tgt, const InlineSlots& slots,
             uint32_t* slot, hipStream_t s) {
  hipLaunchKernelGGL(stage_kernel, dim3(blocks_for((size_t)rows * C, 256)), dim3(256), 0, s, st, rows, tau,
                     beta1, beta2, src_ctx, ctx, rows * C, src_tgt, tgt, slots, slot);
}

// 16-byte accesses, streaming (non-temporal) where NT.
template <bool NT>
__device__ __forceinline__ float4 load4(const float* p) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  if constexpr (!NT) return *(const float4*)p;
  const f4 v = __builtin_nontemporal_load((const f4*)p);
  return make_float4(v.x, v.y, v.z, v.w);
}
template <bool NT>
__device__ __forceinline__ void store4(float* p, float4 x) {
  typedef float f4 __attribute__((ext_vector_type(4)));
  if constexpr (!NT) {
    *(float4*)p = x;
  } else {
    const f4 v = {x.x, x.y, x.z, x.w};
    __builtin_nontemporal_store(v, (f4*)p);
  }
}

// Which accesses to a per-stream matrix and its Adam moments are streaming.
// The state is read and written once a step (and the matrix read once more by
// the forward product), so caching pays only for what stays in the 256 MB
// memory-side cache until the next step, beside what else a step touches:
// all of it up to 160 MB (700 slots of 128 x 128: 39.3 us against 42.0 with the
// moments streaming; 1024 slots, 201 MB: no difference in a step), the matrices
// up to 256 MB (4096 slots of 128 x 128: 203 against 236 us with all of it
// streaming, 292 with all of it cached), else nothing (16384 slots of
// 256 x 256: 4.85 against 4.99 ms, the forward product 716 against 758 us).
enum FdmCache : int {
  FDM_CACHED = 0,      // all of it fits
  FDM_STREAM_ADAM = 1,  // the matrices do
  FDM_STREAM = 2       // not even they
};
constexpr size_t kFdmCachedBytes = (size_t)160 << 20;
static FdmCache fdm_cache(int rows, int Lin, int Lout) {
  const size_t bytes = (size_t)rows * Lin * Lout * sizeof(float);
  return 3 * bytes <= kFdmCachedBytes ? FDM_CACHED : bytes <= ((size_t)256 << 20) ? FDM_STREAM_ADAM : FDM_STREAM;
}

// Rows of U_s whose loads are issued together in the FDM kernels, and the most
// workgroups that share a slot in the adjoint.
constexpr int kFdmBatch = 4;
constexpr int kFdmSplit = 4;

// ---------------------------------------------------------------------------
// Feature Distribution Matrix (Eq. 15): y_s = x'_s U_s, one workgroup per row.
// U_s is [Lin, Lout] (square for the FDM itself; the low-rank ablation's
// per-stream factors A_s [F, F'] and B_s [F', F] use the same kernels).
// Thread (g, t): t covers columns 4t..4t+3, group g rows l = g, g+G, ...
// ---------------------------------------------------------------------------
template <bool NT>
__global__ void __launch_bounds__(256) fdm_fwd_kernel(const StepState* __restrict__ st,
                                                      const float* __restrict__ x1,
                                                      const float* __restrict__ U,
                                                      const uint32_t* __restrict__ slot, int Lin,
                                                      int Lout, float* __restrict__ y32,
                                                      bf16_t* __restrict__ y16) {
  const int r = blockIdx.x;
  if (r >= st->rows) return;
  __shared__ float xs[256];
  __shared__ float part[1024];
  const int tpr = Lout >> 2, G = 256 / tpr;
  const int t = threadIdx.x % tpr, g = threadIdx.x / tpr;
  for (int l = threadIdx.x; l < Lin; l += 256) xs[l] = x1[(size_t)r * Lin + l];
  __syncthreads();
  const float* Us = U + (size_t)slot[r] * Lin * Lout;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  auto add = [&](float xv, float4 u) {
    acc = make_float4(fmaf(xv, u.x, acc.x), fmaf(xv, u.y, acc.y), fmaf(xv, u.z, acc.z), fmaf(xv, u.w, acc.w));
  };
  if (g < G) {
    // rows l = g, g + G, ... in order; loads issued kFdmBatch rows at a time
    int l = g;
    for (; l + (kFdmBatch - 1) * G < Lin; l += kFdmBatch * G) {
      float4 u[kFdmBatch];
#pragma unroll
      for (int q = 0; q < kFdmBatch; ++q) u[q] = load4<NT>(Us + (size_t)(l + q * G) * Lout + 4 * t);
#pragma unroll
      for (int q = 0; q < kFdmBatch; ++q) {
        add(xs[l + q * G], u[q]);
      }
    }
    for (; l < Lin; l += G) {
      const float4 u = load4<NT>(Us + (size_t)l * Lout + 4 * t);
      add(xs[l], u);
    }
    *(float4*)(part + g * Lout + 4 * t) = acc;
  }
  __syncthreads();
  for (int k = threadIdx.x; k < Lout; k += 256) {
    float y = 0.f;
    for (int gg = 0; gg < G; ++gg) y += part[gg * Lout + k];
    if (y32) y32[(size_t)r * Lout + k] = y;
    if (y16) y16[(size_t)r * Lout + k] = f2bf(y);
  }
}

void k_fdm_fwd(const StepState* st, const float* x1, const float* U, const uint32_t* slot, int Lin,
               int Lout, float* y32, bf16_t* y16, int max_rows, hipStream_t s) {
  const bool nt = fdm_cache(max_rows, Lin, Lout) == FDM_STREAM;
  hipLaunchKernelGGL(nt ? fdm_fwd_kernel<true> : fdm_fwd_kernel<false>, dim3(max_rows), dim3(256), 0,
                     s, st, x1, U, slot, Lin, Lout, y32, y16);
}

// Adjoint of Eq. 15 fused with the Adam step on U_s:
//   dx'_s = U_s dy_s (with U before the update), dU_s = x'_s (x) dy_s.
// Bound by memory: 24 bytes an element of U_s.  The rows of U_s are independent,
// so `split` workgroups share a slot; one workgroup a slot leaves the last
// round of workgroups short and too few loads in flight (slots of 128 x 128, one and
// four workgroups: 8 slots 17.2 and 6.8 us, 300 slots 27.7 and 21.9, 700 slots 46.2 and
// 43.4, 1024 slots 65.2 and 66.2, 3000 slots 179 and 173).
template <int CACHE>
__global__ void __launch_bounds__(256) fdm_bwd_kernel(
    const StepState* __restrict__ st, const float* __restrict__ x1, const float* __restrict__ dy,
    float* __restrict__ U, float* __restrict__ mU, float* __restrict__ vU,
    float* __restrict__ dU_keep, const uint32_t* __restrict__ slot, int Lin, int Lout, AdamCfg ac,
    bool update, float* __restrict__ dx1_32, bf16_t* __restrict__ dx1_16, int split) {
  constexpr bool NTU = CACHE == FDM_STREAM, NTM = CACHE != FDM_CACHED;
  const int r = blockIdx.x / split;
  if (r >= st->rows) return;
  __shared__ float xs[256];
  __shared__ float ds[256];
  const int tpr = Lout >> 2, G = 256 / tpr;
  const int t = threadIdx.x % tpr, g = threadIdx.x / tpr;
  const int per = Lin / split, lb = (int)(blockIdx.x % split) * per, le = lb + per;  // this workgroup's rows
  for (int l = lb + threadIdx.x; l < le; l += 256) xs[l] = x1[(size_t)r * Lin + l];
  for (int k = threadIdx.x; k < Lout; k += 256) ds[k] = dy[(size_t)r * Lout + k];
  __syncthreads();
  if (g >= G) return;
  const size_t base_s = (size_t)slot[r] * Lin * Lout;
  const float4 d4 = *(const float4*)(ds + 4 * t);
  const float lr_bc = ac.lr / st->bc1;
  const float inv_bc2 = 1.0f / st->bc2;
  // one row l of U_s: dx'[l] (from U before the update), dU, Adam
  auto row = [&](int l, float4 u, float4 m, float4 v) {
    const size_t idx = base_s + (size_t)l * Lout + 4 * t;
    float part = fmaf(u.w, d4.w, fmaf(u.z, d4.z, fmaf(u.x, d4.x, u.y * d4.y)));
    for (int o = tpr >> 1; o >= 1; o >>= 1) part += __shfl_xor(part, o, 64);
    if (t == 0) {
      if (dx1_32) dx1_32[(size_t)r * Lin + l] = part;
      if (dx1_16) dx1_16[(size_t)r * Lin + l] = f2bf(part);
    }
    const float xv = xs[l];
    const float gr[4] = {xv * d4.x, xv * d4.y, xv * d4.z, xv * d4.w};
    if (dU_keep) *(float4*)(dU_keep + idx) = make_float4(gr[0], gr[1], gr[2], gr[3]);
    if (update) {
      float* up = (float*)&u;
      float* mp = (float*)&m;
      float* vp = (float*)&v;
#pragma unroll
      for (int j = 0; j < 4; ++j) adam1<true>(up[j], mp[j], vp[j], gr[j], lr_bc, inv_bc2, ac);
      store4<NTU>(U + idx, u);
      store4<NTM>(mU + idx, m);
      store4<NTM>(vU + idx, v);
    }
  };
  // rows l = lb + g, lb + g + G, ...; the loads of kFdmBatch rows are issued
  // before any of them is used, so that each thread keeps 3 kFdmBatch 16-byte
  // loads in flight
  const float4 z4 = make_float4(0.f, 0.f, 0.f, 0.f);
  int l = lb + g;
  for (; l + (kFdmBatch - 1) * G < le; l += kFdmBatch * G) {
    float4 u[kFdmBatch], m[kFdmBatch], v[kFdmBatch];
#pragma unroll
    for (int q = 0; q < kFdmBatch; ++q) {
      const size_t idx = base_s + (size_t)(l + q * G) * Lout + 4 * t;
      u[q] = load4<NTU>(U + idx);
      m[q] = update ? load4<NTM>(mU + idx) : z4;
      v[q] = update ? load4<NTM>(vU + idx) : z4;
    }
#pragma unroll
    for (int q = 0; q < kFdmBatch; ++q) row(l + q * G, u[q], m[q], v[q]);
  }
  for (; l < le; l += G) {
    const size_t idx = base_s + (size_t)l * Lout + 4 * t;
    row(l, load4<NTU>(U + idx), update ? load4<NTM>(mU + idx) : z4,
        update ? load4<NTM>(vU + idx) : z4);
  }
}

void k_fdm_bwd(const StepState* st, const float* x1, const float* dy, float* U, float* mU,
               float* vU, float* dU_keep, const uint32_t* slot, int Lin, int Lout, AdamCfg ac,
               bool update, float* dx1_32, bf16_t* dx1_16, int max_rows, hipStream_t s) {
  const int G = 1024 / Lout;  // rows of U_s per pass of a workgroup
  const int split = std::max(1, std::min(kFdmSplit, Lin / (kFdmBatch * G)));
  const FdmCache c = fdm_cache(max_rows, Lin, Lout);
  hipLaunchKernelGGL(c == FDM_CACHED        ? fdm_bwd_kernel<FDM_CACHED>
                     : c == FDM_STREAM_ADAM ? fdm_bwd_kernel<FDM_STREAM_ADAM>
                                            : fdm_bwd_kernel<FDM_STREAM>,
                     dim3((unsigned)max_rows * split), dim3(256), 0, s, st, x1, dy, U, mU, vU, dU_keep,
                     slot, Lin, Lout, ac, update, dx1_32, dx1_16, split);
}

// ---------------------------------------------------------------------------
// LayerNorm (Eq. 9): one wave per row, biased variance, eps 1e-5.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) ln_fwd_kernel(const StepState* __restrict__ st,
                                                     const float* __restrict__ h,
                                                     const float* __restrict__ gamma,
                                                     const float* __restrict__ beta, int F,
                                                     float* __restrict__ z32,
                                                     bf16_t* __restrict__ z16,
                                                     float* __restrict__ mean,
                                                     float* __restrict__ rstd) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= st->rows) return;
  const float* hr = h + (size_t)r * F;
  float s = 0.f;
  for (int f = 4 * lane; f < F; f += 256) {
    const float4 x = *(const float4*)(hr + f);
    s += (x.x + x.y) + (x.z + x.w);
  }
  const float mu = wave_sum(s) / (float)F;
  float q = 0.f;
  for (int f = 4 * lane; f < F; f += 256) {
    const float4 x = *(const float4*)(hr + f);
    const float a = x.x - mu, b = x.y - mu, c = x.z - mu, d = x.w - mu;
    q += (a * a + b * b) + (c * c + d * d);
  }
  const float var = wave_sum(q) / (float)F;
  const float rs = 1.0f / sqrtf(var + 1e-5f);
  if (lane == 0) {
    mean[r] = mu;
    rstd[r] = rs;
  }
  for (int f = 4 * lane; f < F; f += 256) {
    const float4 x = *(const float4*)(hr + f);
    const float4 gm = *(const float4*)(gamma + f);
    const float4 bt = *(const float4*)(beta + f);
    float4 z;
    z.x = (x.x - mu) * rs * gm.x + bt.x;
    z.y = (x.y - mu) * rs * gm.y + bt.y;
    z.z = (x.z - mu) * rs * gm.z + bt.z;
    z.w = (x.w - mu) * rs * gm.w + bt.w;
    if (z32) *(float4*)(z32 + (size_t)r * F + f) = z;
    if (z16)
      *(ushort4*)(z16 + (size_t)r * F + f) = make_ushort4(f2bf(z.x), f2bf(z.y), f2bf(z.z), f2bf(z.w));
  }
}

// Rows of 256 (ln_row.h).
__global__ void __launch_bounds__(256) ln_fwd_256_kernel(const StepState* __restrict__ st,
                                                         const float* __restrict__ h,
                                                         const float* __restrict__ gamma,
                                                         const float* __restrict__ beta,
                                                         float* __restrict__ z32,
                                                         bf16_t* __restrict__ z16,
                                                         float* __restrict__ mean,
                                                         float* __restrict__ rstd) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= st->rows) return;
  const size_t o = (size_t)r * kLnRow + 4 * lane;
  float mu, rs;
  const f32q z = ln_row_fwd(*(const f32q*)(h + o), *(const f32q*)(gamma + 4 * lane),
                            *(const f32q*)(beta + 4 * lane), &mu, &rs);
  if (lane == 0) {
    mean[r] = mu;
    rstd[r] = rs;
  }
  if (z32) *(f32q*)(z32 + o) = z;
  if (z16) *(ushort4*)(z16 + o) = make_ushort4(f2bf(z[0]), f2bf(z[1]), f2bf(z[2]), f2bf(z[3]));
}

// Register-resident variant for F = 256 * NV, NV > 1: each lane holds NV float4.
template <int NV>
__global__ void __launch_bounds__(256) ln_fwd_reg_kernel(const StepState* __restrict__ st,
                                                         const float* __restrict__ h,
                                                         const float* __restrict__ gamma,
                                                         const float* __restrict__ beta,
                                                         float* __restrict__ z32,
                                                         bf16_t* __restrict__ z16,
                                                         float* __restrict__ mean,
                                                         float* __restrict__ rstd) {
  constexpr int F = 256 * NV;
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= st->rows) return;
  const float* hr = h + (size_t)r * F;
  float4 x[NV];
  float s = 0.f;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    x[v] = *(const float4*)(hr + 4 * (lane + 64 * v));
    s += (x[v].x + x[v].y) + (x[v].z + x[v].w);
  }
  const float mu = wave_sum(s) / (float)F;
  float q = 0.f;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const float a = x[v].x - mu, b = x[v].y - mu, c = x[v].z - mu, d = x[v].w - mu;
    q += (a * a + b * b) + (c * c + d * d);
  }
  const float var = wave_sum(q) / (float)F;
  const float rs = 1.0f / sqrtf(var + 1e-5f);
  if (lane == 0) {
    mean[r] = mu;
    rstd[r] = rs;
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int f = 4 * (lane + 64 * v);
    const float4 gm = *(const float4*)(gamma + f);
    const float4 bt = *(const float4*)(beta + f);
    float4 z;
    z.x = (x[v].x - mu) * rs * gm.x + bt.x;
    z.y = (x[v].y - mu) * rs * gm.y + bt.y;
    z.z = (x[v].z - mu) * rs * gm.z + bt.z;
    z.w = (x[v].w - mu) * rs * gm.w + bt.w;
    if (z32) *(float4*)(z32 + (size_t)r * F + f) = z;
    if (z16)
      *(ushort4*)(z16 + (size_t)r * F + f) = make_ushort4(f2bf(z.x), f2bf(z.y), f2bf(z.z), f2bf(z.w));
  }
}

void k_ln_fwd(const StepState* st, const float* h, const float* gamma, const float* beta, int F,
              float* z32, bf16_t* z16, float* mean, float* rstd, int max_rows, hipStream_t s) {
  const dim3 g(blocks_for(max_rows, 4)), b(256);
  switch (F % 256 == 0 ? F / 256 : 0) {
    case 1: hipLaunchKernelGGL(ln_fwd_256_kernel, g, b, 0, s, st, h, gamma, beta, z32, z16, mean, rstd); return;
    case 2: hipLaunchKernelGGL(ln_fwd_reg_kernel<2>, g, b, 0, s, st, h, gamma, beta, z32, z16, mean, rstd); return;
    case 4: hipLaunchKernelGGL(ln_fwd_reg_kernel<4>, g, b, 0, s, st, h, gamma, beta, z32, z16, mean, rstd); return;
    case 8: hipLaunchKernelGGL(ln_fwd_reg_kernel<8>, g, b, 0, s, st, h, gamma, beta, z32, z16, mean, rstd); return;
    default:
      hipLaunchKernelGGL(ln_fwd_kernel, g, b, 0, s, st, h, gamma, beta, F, z32, z16, mean, rstd);
  }
}

// dh = dh_next + rstd * (dxhat - mean(dxhat) - xhat * mean(dxhat * xhat)),
// dxhat = dz * gamma, xhat = (h - mean) * rstd.
__global__ void __launch_bounds__(256) ln_bwd_kernel(
    const StepState* __restrict__ st, const float* __restrict__ h, const float* __restrict__ mean,
    const float* __restrict__ rstd, const float* __restrict__ gamma, const float* __restrict__ dz,
    const float* __restrict__ dh_next, int F, float* __restrict__ dh32,
    bf16_t* __restrict__ dh16) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= st->rows) return;
  const float mu = mean[r], rs = rstd[r];
  const float* hr = h + (size_t)r * F;
  const float* dzr = dz + (size_t)r * F;
  float s1 = 0.f, s2 = 0.f;
  for (int f = 4 * lane; f < F; f += 256) {
    const float4 x = *(const float4*)(hr + f);
    const float4 d = *(const float4*)(dzr + f);
    const float4 gm = *(const float4*)(gamma + f);
    const float dx0 = d.x * gm.x, dx1 = d.y * gm.y, dx2 = d.z * gm.z, dx3 = d.w * gm.w;
    s1 += (dx0 + dx1) + (dx2 + dx3);
    s2 += (dx0 * ((x.x - mu) * rs) + dx1 * ((x.y - mu) * rs)) +
          (dx2 * ((x.z - mu) * rs) + dx3 * ((x.w - mu) * rs));
  }
  const float m1 = wave_sum(s1) / (float)F;
  const float m2 = wave_sum(s2) / (float)F;
  for (int f = 4 * lane; f < F; f += 256) {
    const float4 x = *(const float4*)(hr + f);
    const float4 d = *(const float4*)(dzr + f);
    const float4 gm = *(const float4*)(gamma + f);
    const float4 dn = *(const float4*)(dh_next + (size_t)r * F + f);
    float4 o;
    o.x = dn.x + rs * (d.x * gm.x - m1 - ((x.x - mu) * rs) * m2);
    o.y = dn.y + rs * (d.y * gm.y - m1 - ((x.y - mu) * rs) * m2);
    o.z = dn.z + rs * (d.z * gm.z - m1 - ((x.z - mu) * rs) * m2);
    o.w = dn.w + rs * (d.w * gm.w - m1 - ((x.w - mu) * rs) * m2);
    *(float4*)(dh32 + (size_t)r * F + f) = o;
    if (dh16)
      *(ushort4*)(dh16 + (size_t)r * F + f) = make_ushort4(f2bf(o.x), f2bf(o.y), f2bf(o.z), f2bf(o.w));
  }
}

// Rows of 256 (ln_row.h).
__global__ void __launch_bounds__(256) ln_bwd_256_kernel(
    const StepState* __restrict__ st, const float* __restrict__ h, const float* __restrict__ mean,
    const float* __restrict__ rstd, const float* __restrict__ gamma, const float* __restrict__ dz,
    const float* __restrict__ dh_next, float* __restrict__ dh32, bf16_t* __restrict__ dh16) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= st->rows) return;
  const size_t o = (size_t)r * kLnRow + 4 * lane;
  const f32q v = ln_row_bwd(*(const f32q*)(h + o), mean[r], rstd[r], *(const f32q*)(gamma + 4 * lane),
                            *(const f32q*)(dz + o), *(const f32q*)(dh_next + o));
  *(f32q*)(dh32 + o) = v;
  if (dh16) *(ushort4*)(dh16 + o) = make_ushort4(f2bf(v[0]), f2bf(v[1]), f2bf(v[2]), f2bf(v[3]));
}

template <int NV>
__global__ void __launch_bounds__(256) ln_bwd_reg_kernel(
    const StepState* __restrict__ st, const float* __restrict__ h, const float* __restrict__ mean,
    const float* __restrict__ rstd, const float* __restrict__ gamma, const float* __restrict__ dz,
    const float* __restrict__ dh_next, float* __restrict__ dh32, bf16_t* __restrict__ dh16) {
  constexpr int F = 256 * NV;
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= st->rows) return;
  const float mu = mean[r], rs = rstd[r];
  float xh[NV][4], dx[NV][4];
  float s1 = 0.f, s2 = 0.f;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int f = 4 * (lane + 64 * v);
    const float4 x = *(const float4*)(h + (size_t)r * F + f);
    const float4 d = *(const float4*)(dz + (size_t)r * F + f);
    const float4 gm = *(const float4*)(gamma + f);
    xh[v][0] = (x.x - mu) * rs; xh[v][1] = (x.y - mu) * rs;
    xh[v][2] = (x.z - mu) * rs; xh[v][3] = (x.w - mu) * rs;
    dx[v][0] = d.x * gm.x; dx[v][1] = d.y * gm.y; dx[v][2] = d.z * gm.z; dx[v][3] = d.w * gm.w;
    s1 += (dx[v][0] + dx[v][1]) + (dx[v][2] + dx[v][3]);
    s2 += (dx[v][0] * xh[v][0] + dx[v][1] * xh[v][1]) + (dx[v][2] * xh[v][2] + dx[v][3] * xh[v][3]);
  }
  const float m1 = wave_sum(s1) / (float)F;
  const float m2 = wave_sum(s2) / (float)F;
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int f = 4 * (lane + 64 * v);
    const float4 dn = *(const float4*)(dh_next + (size_t)r * F + f);
    float4 o;
    o.x = dn.x + rs * (dx[v][0] - m1 - xh[v][0] * m2);
    o.y = dn.y + rs * (dx[v][1] - m1 - xh[v][1] * m2);
    o.z = dn.z + rs * (dx[v][2] - m1 - xh[v][2] * m2);
    o.w = dn.w + rs * (dx[v][3] - m1 - xh[v][3] * m2);
    *(float4*)(dh32 + (size_t)r * F + f) = o;
    if (dh16)
      *(ushort4*)(dh16 + (size_t)r * F + f) = make_ushort4(f2bf(o.x), f2bf(o.y), f2bf(o.z), f2bf(o.w));
  }
}

// The LayerNorm adjoint with the column sums folded in.  The 4 waves of a
// workgroup share each row (thread t takes columns t, t + 256, ...), so a
// thread's share of the column sums over the group's rows stays in CPT x 3
// registers; the row statistics of the adjoint are summed over the 4 waves
// through LDS, in wave order.  Rows r0 .. r0 + kLnFoldRows - 1 in order.
template <int CPT>
__global__ void __launch_bounds__(256) ln_bwd_fold_kernel(
    const StepState* __restrict__ st, const float* __restrict__ h, const float* __restrict__ mean,
    const float* __restrict__ rstd, const float* __restrict__ gamma, const float* __restrict__ dz,
    const float* __restrict__ dh_next, float* __restrict__ dh32, bf16_t* __restrict__ dh16,
    float* __restrict__ part) {
  constexpr int F = 256 * CPT;
  __shared__ float red[2][4][2];  // per-row wave partials, alternating by row
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int rows = st->rows;
  const int r0 = blockIdx.x * kLnFoldRows;
  if (r0 >= rows) return;
  const int r1 = min(rows, r0 + kLnFoldRows);
  float gm[CPT], sb[CPT], sg[CPT], so[CPT];
#pragma unroll
  for (int u = 0; u < CPT; ++u) {
    gm[u] = gamma[t + 256 * u];
    sb[u] = sg[u] = so[u] = 0.f;
  }
  for (int r = r0; r < r1; ++r) {
    const int buf = (r - r0) & 1;
    const float mu = mean[r], rs = rstd[r];
    float xh[CPT], d[CPT], dn[CPT];
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
      const size_t o = (size_t)r * F + t + 256 * u;
      xh[u] = (h[o] - mu) * rs;
      d[u] = dz[o];
      dn[u] = dh_next[o];
      const float dx = d[u] * gm[u];
      s1 += dx;
      s2 += dx * xh[u];
    }
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    if (lane == 0) {
      red[buf][w][0] = s1;
      red[buf][w][1] = s2;
    }
    // (the next row's barrier keeps the row after next from rewriting
    // red[buf] before every thread has read it)
    __syncthreads();
    const float m1 = ((red[buf][0][0] + red[buf][1][0]) + (red[buf][2][0] + red[buf][3][0])) / (float)F;
    const float m2 = ((red[buf][0][1] + red[buf][1][1]) + (red[buf][2][1] + red[buf][3][1])) / (float)F;
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
      const size_t o = (size_t)r * F + t + 256 * u;
      const float dx = d[u] * gm[u];
      const float v = dn[u] + rs * (dx - m1 - xh[u] * m2);
      dh32[o] = v;
      if (dh16) dh16[o] = f2bf(v);
      sb[u] += d[u];
      sg[u] += d[u] * xh[u];
      so[u] += dn[u];
    }
  }
  float* pg = part + (size_t)blockIdx.x * 3 * F;
#pragma unroll
  for (int u = 0; u < CPT; ++u) {
    pg[t + 256 * u] = sb[u];
    pg[F + t + 256 * u] = sg[u];
    pg[2 * F + t + 256 * u] = so[u];
  }
}

bool ln_bwd_folds(int F) { return F == 256 || F == 512 || F == 1024 || F == 2048; }

size_t ln_fold_part_elems(int max_rows, int F) {
  return (size_t)((max_rows + kLnFoldRows - 1) / kLnFoldRows) * 3 * (size_t)F;
}

void k_ln_bwd(const StepState* st, const float* h, const float* mean, const float* rstd,
              const float* gamma, const float* dz, const float* dh_next, int F, float* dh32,
              bf16_t* dh16, float* part, int max_rows, hipStream_t s) {
  if (part && ln_bwd_folds(F)) {
    const dim3 g(blocks_for(max_rows, kLnFoldRows)), b(256);
    switch (F / 256) {
      case 1: hipLaunchKernelGGL(ln_bwd_fold_kernel<1>, g, b, 0, s, st, h, mean, rstd, gamma, dz, dh_next, dh32, dh16, part); return;
      case 2: hipLaunchKernelGGL(ln_bwd_fold_kernel<2>, g, b, 0, s, st, h, mean, rstd, gamma, dz, dh_next, dh32, dh16, part); return;
      case 4: hipLaunchKernelGGL(ln_bwd_fold_kernel<4>, g, b, 0, s, st, h, mean, rstd, gamma, dz, dh_next, dh32, dh16, part); return;
      case 8: hipLaunchKernelGGL(ln_bwd_fold_kernel<8>, g, b, 0, s, st, h, mean, rstd, gamma, dz, dh_next, dh32, dh16, part); return;
    }
  }
  const dim3 g(blocks_for(max_rows, 4)), b(256);
  switch (F % 256 == 0 ? F / 256 : 0) {
    case 1: hipLaunchKernelGGL(ln_bwd_256_kernel, g, b, 0, s, st, h, mean, rstd, gamma, dz, dh_next, dh32, dh16); return;
    case 2: hipLaunchKernelGGL(ln_bwd_reg_kernel<2>, g, b, 0, s, st, h, mean, rstd, gamma, dz, dh_next, dh32, dh16); return;
    case 4: hipLaunchKernelGGL(ln_bwd_reg_kernel<4>, g, b, 0, s, st, h, mean, rstd, gamma, dz, dh_next, dh32, dh16); return;
    case 8: hipLaunchKernelGGL(ln_bwd_reg_kernel<8>, g, b, 0, s, st, h, mean, rstd, gamma, dz, dh_next, dh32, dh16); return;
    default:
      hipLaunchKernelGGL(ln_bwd_kernel, g, b, 0, s, st, h, mean, rstd, gamma, dz, dh_next, F, dh32, dh16);
  }
}

// ---------------------------------------------------------------------------
// Head: softmax (Eq. 1) -> 16-bit integer CDF -> range-coder lane ->
// cross-entropy adjoint (Eq. 2).  One wave per row; lane l holds symbols
// 4l .. 4l+3.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) head_kernel(const StepState* __restrict__ st, HeadArgs a,
                                                   StreamIO io) {
  const int lane = threadIdx.x & 63;
  const int r = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= st->rows) return;
  const float4 z4 = *(const float4*)(a.logits + (size_t)r * 256 + 4 * lane);
  const float z[4] = {z4.x, z4.y, z4.z, z4.w};
  float p[4];
  int x = 0;
  const bool have_target = head_row(st, a, io, r, lane, z, p, &x);
  if (have_target && a.want_grad) {
    const float ir = st->inv_rows;
    float4 d4;
    d4.x = (p[0] - (4 * lane + 0 == x ? 1.0f : 0.0f)) * ir;
    d4.y = (p[1] - (4 * lane + 1 == x ? 1.0f : 0.0f)) * ir;
    d4.z = (p[2] - (4 * lane + 2 == x ? 1.0f : 0.0f)) * ir;
    d4.w = (p[3] - (4 * lane + 3 == x ? 1.0f : 0.0f)) * ir;
    if (a.dz32) *(float4*)(a.dz32 + (size_t)r * 256 + 4 * lane) = d4;
    if (a.dz16)
      *(ushort4*)(a.dz16 + (size_t)r * 256 + 4 * lane) =
          make_ushort4(f2bf(d4.x), f2bf(d4.y), f2bf(d4.z), f2bf(d4.w));
  }
}

void k_head(const StepState* st, HeadArgs a, StreamIO io, int max_rows, hipStream_t s) {
  hipLaunchKernelGGL(head_kernel, dim3(blocks_for(max_rows, 4)), dim3(256), 0, s, st, a, io);
}

// ---------------------------------------------------------------------------
// Column sums and embedding gradient by themselves (grad_sums.h)
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) colsum_partial_kernel(const StepState* __restrict__ st,
                                                             const ColsumJob* __restrict__ jobs,
                                                             int n_jobs, int total_cols,
                                                             float* __restrict__ partial) {
  __shared__ float part[256];
  colsum_block(st, jobs, n_jobs, total_cols, partial, blockIdx.x, blockIdx.y, part);
}

__global__ void colsum_reduce_kernel(const StepState* __restrict__ st,
                                     const ColsumJob* __restrict__ jobs, int n_jobs,
                                     int total_cols, const float* __restrict__ partial,
                                     int chunk) {
  const int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= total_cols) return;
  int j = 0;
  while (j + 1 < n_jobs && c >= jobs[j + 1].col_offset) ++j;
  const ColsumJob& jb = jobs[j];
  float s;
  if (jb.part) {
    const int ng = (st->rows + jb.part_rows - 1) / jb.part_rows;
    s = ordered_sum(jb.part + (c - jb.col_offset), (size_t)jb.part_ld, ng);
  } else {
    const int nch = (st->rows + chunk - 1) / chunk;
    s = ordered_sum(partial + c, (size_t)total_cols, nch);
  }
  gl(jb.dst)[c - jb.col_offset] = s * (jb.scale == 0.0f ? st->inv_rows : jb.scale);
}

size_t colsum_partial_elems(int max_rows, int total_cols) {
  return (size_t)((max_rows + kColChunk - 1) / kColChunk) * total_cols;
}

void k_colsum_partial(const StepState* st, const ColsumJob* jobs, int n_jobs, int total_blocks,
                      int total_cols, float* partial, int max_rows, hipStream_t s) {
  if (total_blocks == 0) return;
  dim3 grid(total_blocks, (max_rows + kColChunk - 1) / kColChunk);
  hipLaunchKernelGGL(colsum_partial_kernel, grid, dim3(256), 0, s, st, jobs, n_jobs, total_cols, partial);
}

void k_colsum(const StepState* st, const ColsumJob* jobs, int n_jobs, int total_blocks,
              int total_cols, float* partial, int max_rows, hipStream_t s) {
  if (total_blocks == 0) return;
  k_colsum_partial(st, jobs, n_jobs, total_blocks, total_cols, partial, max_rows, s);
  hipLaunchKernelGGL(colsum_reduce_kernel, dim3(blocks_for(total_cols, 256)), dim3(256), 0, s, st,
                     jobs, n_jobs, total_cols, (const float*)partial, kColChunk);
}

void k_colsum_reduce(const StepState* st, const ColsumJob* jobs, int n_jobs, int total_cols,
                     const float* partial, int chunk_rows, hipStream_t s) {
  if (total_cols == 0) return;
  hipLaunchKernelGGL(colsum_reduce_kernel, dim3(blocks_for(total_cols, 256)), dim3(256), 0, s, st,
                     jobs, n_jobs, total_cols, partial, chunk_rows);
}

template <int E>
__global__ void __launch_bounds__(256) emb_grad_partial_kernel(const StepState* __restrict__ st,
                                                               const uint8_t* __restrict__ ctx,
                                                               const float* __restrict__ dx, int C,
                                                               int chunk_rows, int sub_rows,
                                                               float* __restrict__ partial) {
  extern __shared__ __align__(16) char smem[];
  emb_grad_block<E>(st->rows, ctx, dx, C, chunk_rows, sub_rows, partial, blockIdx.x, smem);
}

__global__ void emb_grad_reduce_kernel(const StepState* __restrict__ st,
                                       const float* __restrict__ partial, int chunk_rows, int n,
                                       float* __restrict__ demb) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= n) return;
  const int nb = (st->rows + chunk_rows - 1) / chunk_rows;
  demb[k] = ordered_sum(partial + k, (size_t)n, nb);
}

void emb_grad_plan(int max_rows, int C, int E, int* chunk_rows, int* sub_rows) {
  const int F = C * E;
  int sub = 8192 / F;
  sub = sub < 1 ? 1 : (sub > 16 ? 16 : sub);
  int chunk = sub;
  while ((max_rows + chunk - 1) / chunk > 256) chunk += sub;
  *chunk_rows = chunk;
  *sub_rows = sub;
}

void k_emb_grad_reduce(const StepState* st, const float* partial, int chunk_rows, int E,
                       float* demb, hipStream_t s) {
  const int n = 256 * E;
  hipLaunchKernelGGL(emb_grad_reduce_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, st, partial,
                     chunk_rows, n, demb);
}

void k_emb_grad_partial(const StepState* st, const uint8_t* ctx, const float* dx, int C, int E,
                        float* partial, int chunk_rows, int sub_rows, int max_rows, hipStream_t s) {
  const int nb = (max_rows + chunk_rows - 1) / chunk_rows;
  const size_t smem = emb_lds_bytes(sub_rows, C, E);
#define EMB_CASE(EE)                                                                            \
  case EE:                                                                                      \
    if (smem > 65536)  /* the widest feature vectors need more than the default LDS */          \
      (void)hipFuncSetAttribute((const void*)emb_grad_partial_kernel<EE>,                       \
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);         \
    hipLaunchKernelGGL(emb_grad_partial_kernel<EE>, dim3(nb), dim3(256), smem, s, st, ctx, dx, C, \
                       chunk_rows, sub_rows, partial);                                          \
    break;
  switch (E) {
    EMB_CASE(16)
    EMB_CASE(32)
    EMB_CASE(64)
  }
#undef EMB_CASE
}

// ---------------------------------------------------------------------------
// Adam on the shared parameters (FP32 master, optional BF16 shadow).  A wave's 64
// elements belong to one tensor (tensors are 64-aligned).  kind[i / 64] = 0: the
// gradient is complete in g; k > 0: it is the in-order sum of the partials of job
// k - 1 (biases, LayerNorm, embedding), formed here instead of by two launches of
// their own, and written to g (FP32, the three launches against this one: 9.4 to
// 5.0 us at 8 streams of a small model, 16.8 to 10.4 us at 333 rows of a mid one).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) adam_kernel(const StepState* __restrict__ st, float* __restrict__ p,
                                                   float* __restrict__ g, float* __restrict__ m,
                                                   float* __restrict__ v, bf16_t* __restrict__ p16,
                                                   size_t n, AdamCfg ac, const uint8_t* __restrict__ kind,
                                                   const PartialJob* __restrict__ jobs) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;  // n a multiple of 64
  const float lr_bc = ac.lr / st->bc1;
  const float inv_bc2 = 1.0f / st->bc2;
  float gr = g[i];
  float m0 = m[i], v0 = v[i], p0 = p[i];
  const int k = __builtin_amdgcn_readfirstlane((int)kind[i >> 6]);
  if (k) {
    const PartialJob jb = jobs[k - 1];
    const size_t e = i - jb.off;
    if (e >= (size_t)jb.cols) return;  // padding
    gr = ordered_sum(jb.part + e, (size_t)jb.ld, (st->rows + jb.part_rows - 1) / jb.part_rows);
    g[i] = gr;
  }
  adam1(p0, m0, v0, gr, lr_bc, inv_bc2, ac);
  m[i] = m0;
  v[i] = v0;
  p[i] = p0;
  if (p16) p16[i] = f2bf(p0);
}

void k_adam(const StepState* st, float* p, float* g, float* m, float* v, bf16_t* p16, size_t n,
            AdamCfg ac, const uint8_t* kind, const PartialJob* jobs, hipStream_t s) {
  hipLaunchKernelGGL(adam_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, st, p, g, m, v, p16, n, ac,
                     kind, jobs);
}

// ---------------------------------------------------------------------------
// Initialisation (SplitMix64, Steele, Lea & Flood 2014)
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
  uint64_t z = x + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__device__ __forceinline__ float init_value(uint64_t counter, float bound) {
  const int k = (int)(splitmix64(counter) >> 40) - (1 << 23);
  const float a = (float)k * (1.0f / 8388608.0f);
  return a * bound;
}

// Tensors [0, n) of one launch, by increasing offset; elements begin .. end - 1
// of the flat buffers, padding between tensors included.
constexpr int kInitTensors = 64;
struct InitBatch {
  InitTensor t[kInitTensors];
  int n;
  size_t begin, end;
};

__global__ void __launch_bounds__(256) init_shared_kernel(InitBatch b, uint64_t seed, float* __restrict__ p,
                                                          float* __restrict__ m, float* __restrict__ v,
                                                          float* __restrict__ g, bf16_t* __restrict__ p16) {
  const size_t e = b.begin + (size_t)blockIdx.x * 256 + threadIdx.x;
  if (e >= b.end) return;
  int lo = 0, hi = b.n;  // the last tensor that starts at or before e
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (b.t[mid].off <= e) lo = mid; else hi = mid;
  }
  const InitTensor t = b.t[lo];
  const size_t j = e - t.off;
  const float x = j >= t.numel ? 0.0f : t.tid ? init_value(seed + ((uint64_t)t.tid << 40) + j, t.bound) : t.bound;
  p[e] = x;
  m[e] = v[e] = g[e] = 0.0f;
  if (p16) p16[e] = f2bf(x);
}

void k_init_shared(const InitTensor* t, int n, size_t total, uint64_t seed, float* p, float* m,
                   float* v, float* g, bf16_t* p16, hipStream_t s) {
  for (int i = 0; i < n; i += kInitTensors) {
    InitBatch b;
    b.n = std::min(kInitTensors, n - i);
    for (int k = 0; k < b.n; ++k) b.t[k] = t[i + k];
    b.begin = i == 0 ? 0 : t[i].off;
    b.end = i + b.n < n ? t[i + b.n].off : total;
    hipLaunchKernelGGL(init_shared_kernel, dim3(blocks_for(b.end - b.begin, 256)), dim3(256), 0, s, b,
                       seed, p, m, v, g, p16);
  }
}

// n a multiple of 4
__global__ void __launch_bounds__(256) init_streams_kernel(float* __restrict__ u, float* __restrict__ m,
                                                           float* __restrict__ v, size_t n, uint64_t counter,
                                                           float bound) {
  const size_t j = 4 * ((size_t)blockIdx.x * 256 + threadIdx.x);
  if (j >= n) return;
  *(float4*)(u + j) = make_float4(init_value(counter + j, bound), init_value(counter + j + 1, bound),
                                  init_value(counter + j + 2, bound), init_value(counter + j + 3, bound));
  const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
  *(float4*)(m + j) = z;
  *(float4*)(v + j) = z;
}

void k_init_streams(float* u, float* m, float* v, size_t n, uint64_t seed, uint32_t tid, float bound,
                    hipStream_t s) {
  hipLaunchKernelGGL(init_streams_kernel, dim3(blocks_for(n / 4, 256)), dim3(256), 0, s, u, m, v, n,
                     seed + ((uint64_t)tid << 40), bound);
}

__global__ void __launch_bounds__(256) zero_kernel(float* __restrict__ dst, size_t n) {
  for (size_t j = 4 * ((size_t)blockIdx.x * 256 + threadIdx.x); j < n; j += 4 * (size_t)gridDim.x * 256)
    *(float4*)(dst + j) = make_float4(0.f, 0.f, 0.f, 0.f);
}

void k_zero(float* dst, size_t n, hipStream_t s) {
  const size_t blocks = (n / 4 + 255) / 256;
  hipLaunchKernelGGL(zero_kernel, dim3((unsigned)std::min<size_t>(std::max<size_t>(blocks, 1), 65536)), dim3(256), 0, s,
                     dst, n);
}

__global__ void to_bf16_kernel(const float* src, bf16_t* dst, size_t n) {
  const size_t j = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j < n) dst[j] = f2bf(src[j]);
}
void k_to_bf16(const float* src, bf16_t* dst, size_t n, hipStream_t s) {
  if (n == 0) return;
  hipLaunchKernelGGL(to_bf16_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, src, dst, n);
}

// ---------------------------------------------------------------------------
// Coder lanes (one thread per stream)
// ---------------------------------------------------------------------------
// The first t bytes of each stream: frequency 256 each (Algorithm 1, "with
// equal probability"); also initialises the coder state.
__global__ void uniform_prefix_kernel(StreamIO io, int n_streams, int C, bool decoding) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n_streams) return;
  const uint64_t len = io.lens[s];
  const uint64_t n = len < (uint64_t)C ? len : (uint64_t)C;
  if (!decoding) {
    RcEnc e;
    rc_enc_init(e);
    uint8_t* out = io.pay + io.pay_off[s];
    const uint64_t cap = io.pay_cap[s];
    for (uint64_t i = 0; i < n; ++i) rc_encode(e, out, cap, 256u * io.src[io_at(io, io.off[s], i)], 256u);
    io.enc[s] = e;
  } else {
    RcDec d;
    const uint8_t* in = io.pay_in + io.pay_off[s];
    const uint64_t plen = io.pay_cap[s];
    rc_dec_init(d, in, plen);
    for (uint64_t i = 0; i < n; ++i) {
      // largest x with (range * 256x) >> 16 <= d
      uint32_t lo = 0, hi = 256;
      while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (((d.range * (uint64_t)(256u * mid)) >> 16) <= d.d) lo = mid; else hi = mid;
      }
      io.dst[io_at(io, io.off[s], i)] = (uint8_t)lo;
      rc_consume(d, in, plen, 256u * lo, 256u * lo + 256u);
    }
    io.dec[s] = d;
  }
}

void k_uniform_prefix(StreamIO io, int n_streams, int C, bool decoding, hipStream_t s) {
  hipLaunchKernelGGL(uniform_prefix_kernel, dim3(blocks_for(n_streams, 64)), dim3(64), 0, s, io,
                     n_streams, C, decoding);
}

__global__ void rc_finish_kernel(StreamIO io, int n_streams) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n_streams) return;
  RcEnc e = io.enc[s];
  rc_finish(e, io.pay + io.pay_off[s], io.pay_cap[s]);
  io.enc[s] = e;
}

void k_rc_finish(StreamIO io, int n_streams, hipStream_t s) {
  hipLaunchKernelGGL(rc_finish_kernel, dim3(blocks_for(n_streams, 64)), dim3(64), 0, s, io,
                     n_streams);
}

// Encoder with caller's tables, one wave per stream: lane l reads the symbol
// and the two table entries of step t0 + l, 64 steps at a time and the next 64
// while these are coded, and the coder itself is wave-uniform integer work.
// rc_encode (rangecoder.h) looks back at written bytes for a carry; here the
// last byte that is not 0xFF and the number of 0xFF after it are kept instead
// (a written byte is carried into at most once), so that a step touches no
// memory: finished bytes gather in a register, one a lane, and leave 64 at a
// time.  One thread per stream waits for two dependent loads a step, and as soon
// as one of its wave's 64 streams carries, for the bytes it reads back (3000
// streams x 40 steps: 44 to 16 us).
__global__ void __launch_bounds__(256) rc_table_encode_wave_kernel(
    const uint32_t* __restrict__ cum, const uint8_t* __restrict__ sym, size_t n_steps,
    size_t n_streams, uint8_t* __restrict__ out, size_t cap, uint64_t* __restrict__ out_lens) {
  const int lane = threadIdx.x & 63;
  const size_t s = (size_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (s >= n_streams) return;
  uint8_t* o = out + s * cap;
  uint64_t done = 0;     // bytes that have left the register
  int held = 0, buf = 0;  // bytes in it
  auto flush = [&] {
    if (lane < held && done + lane < cap) o[done + lane] = (uint8_t)buf;
    done += held;
    held = 0;
  };
  auto emit = [&](uint32_t b) {
    buf = lane == held ? (int)b : buf;
    if (++held == 64) flush();
  };
  bool have = false;  // a byte that may still be carried into,
  uint32_t last = 0;  // its value,
  uint64_t ffs = 0;   // and the 0xFF bytes after it
  auto push = [&](uint32_t b) {
    if (have && b == 0xFFu) {
      ++ffs;
      return;
    }
    if (have) emit(last);
    for (; ffs > 0; --ffs) emit(0xFFu);
    last = b;
    have = true;
  };
  auto carry = [&] {
    last = (last + 1) & 0xFFu;
    if (ffs == 0) return;
    emit(last);
    for (; ffs > 1; --ffs) emit(0u);
    last = 0;
    ffs = 0;
  };

  // steps past the last are read as the last one and not coded
  auto at = [&](size_t t) { return min(t, n_steps - 1) * n_streams + s; };
  uint64_t low = 0, range = kRcTop;
  uint32_t x_next = 0, lo_next = 0, hi_next = 0;
  auto entries = [&](size_t t0) {
    const uint32_t* c = cum + at(t0 + lane) * 257 + x_next;
    lo_next = c[0];
    hi_next = c[1];
  };
  if (n_steps > 0) {
    x_next = sym[at(lane)];
    entries(0);
    x_next = sym[at(64 + lane)];
  }
  for (size_t t0 = 0; t0 < n_steps; t0 += 64) {
    const int vlo = (int)lo_next, vhi = (int)hi_next;
    if (t0 + 64 < n_steps) {
      entries(t0 + 64);
      x_next = sym[at(t0 + 128 + lane)];
    }
    const int n = (int)min((size_t)64, n_steps - t0);
    for (int k = 0; k < n; ++k) {
      const uint32_t c0 = __builtin_amdgcn_readlane(vlo, k), c1 = __builtin_amdgcn_readlane(vhi, k);
      const uint64_t lo = (range * c0) >> 16, hi = (range * c1) >> 16;
      low += lo;
      range = hi - lo;
      if (low >= kRcTop) {
        carry();
        low -= kRcTop;
      }
      for (int q = 0; q < 4 && range < kRcBot; ++q) {
        push((uint32_t)(low >> 24));
        low = (low << 8) & 0xFFFFFFFFull;
        range <<= 8;
      }
    }
  }
  if (n_steps > 0) {
    uint64_t v = (low + 0xFFFFull) & ~0xFFFFull;
    if (v >= kRcTop) {
      carry();
      v -= kRcTop;
    }
    push((uint32_t)(v >> 24));
    push((uint32_t)(v >> 16) & 0xFFu);
    emit(last);
    for (; ffs > 0; --ffs) emit(0xFFu);
    flush();
  }
  if (lane == 0) out_lens[s] = done;
}

// The same, one thread per stream: for more streams than fill the chip with a wave
// each (rc_wave_streams).
__global__ void rc_table_encode_thread_kernel(
    const uint32_t* __restrict__ cum, const uint8_t* __restrict__ sym, size_t n_steps,
    size_t n_streams, uint8_t* __restrict__ out, size_t cap, uint64_t* __restrict__ out_lens) {
  const size_t s = (size_t)blockIdx.x * 64 + threadIdx.x;
  if (s >= n_streams) return;
  RcEnc e;
  rc_enc_init(e);
  uint8_t* o = out + s * cap;
  for (size_t t = 0; t < n_steps; ++t) {
    const uint32_t* c = cum + (t * n_streams + s) * 257;
    const uint32_t x = sym[t * n_streams + s];
    rc_encode(e, o, cap, c[x], c[x + 1] - c[x]);
  }
  rc_finish(e, o, cap);
  out_lens[s] = e.pos;
}

// Most streams that take a wave each.  8192 waves fill the chip; past that they
// come in turn, and their time is that of the instructions they issue, 64 times
// those of a thread per stream, whose own time is the latency of a step's
// dependent loads whatever the number of streams.  So the line is where the issue
// of all streams passes that latency, and it lies lower where a few steps leave
// little latency to hide.  Whole calls, us, a thread and a wave per stream:
//   encode  4 steps: 4000 streams 34.6 and 34.6, 8000 36.8 and 38.7, 128000 103 and 154
//          64 steps: 6000 101 and 70, 12000 104 and 101, 16000 108 and 122, 32000 141 and 203
//          (symbols that the tables say are likely; 10000 x 40 unlikely ones, more bytes
//          a step: 78 and 84)
//   decode  4 steps: 6000 35.7 and 35.9, 12000 39.8 and 44.2, 128000 114 and 190
//          16 steps: 8000 72 and 58, 12000 74 and 70, 16000 77 and 81, 64000 155 and 241
//          64 steps: 16000 283 and 237, 24000 349 and 329, 32000 365 and 433
static size_t rc_wave_streams(size_t n_steps, bool decode) {
  return n_steps < 16 ? 6000 : !decode ? 8000 : n_steps < 64 ? 12000 : 24000;
}

void k_rc_table_encode(const uint32_t* cum, const uint8_t* sym, size_t n_steps, size_t n_streams,
                       uint8_t* out, size_t cap, uint64_t* out_lens, hipStream_t s) {
  if (n_streams <= rc_wave_streams(n_steps, false))
    hipLaunchKernelGGL(rc_table_encode_wave_kernel, dim3(blocks_for(n_streams, 4)), dim3(256), 0, s, cum,
                       sym, n_steps, n_streams, out, cap, out_lens);
  else
    hipLaunchKernelGGL(rc_table_encode_thread_kernel, dim3(blocks_for(n_streams, 64)), dim3(64), 0, s, cum,
                       sym, n_steps, n_streams, out, cap, out_lens);
}

// Decoder with caller's tables, one wave per stream: the lanes hold the whole
// table of a step (lane l the entries l, l + 64, l + 128, l + 192), loaded
// kRcAhead steps ahead in contiguous 256-byte pieces, and find the symbol by
// counting the entries whose interval starts at or below the code value (the
// entries do not decrease).  The payload comes through a window of 64 bytes, one
// a lane, with the next window in flight.  A step is then a chain of integer
// instructions with no memory access in it; a binary search by one thread took 8
// dependent loads of 4 bytes each (3000 streams x 40 steps, 123 MB of tables:
// 108 to 33 us).
constexpr int kRcAhead = 4;

__global__ void __launch_bounds__(256) rc_table_decode_wave_kernel(
    const uint32_t* __restrict__ cum, const uint8_t* __restrict__ in,
    const uint64_t* __restrict__ in_lens, size_t cap, size_t n_steps, size_t n_streams,
    uint8_t* __restrict__ sym) {
  const int lane = threadIdx.x & 63;
  const size_t s = (size_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (s >= n_streams || n_steps == 0) return;
  const uint8_t* p = in + s * cap;
  const uint64_t len = in_lens[s] < cap ? in_lens[s] : cap;
  auto window = [&](uint64_t w) { return w + lane < len ? (uint32_t)p[w + lane] : 0u; };
  uint64_t wbase = 0, pos = 0;
  uint32_t cur = window(0), nxt = window(64);
  auto next_byte = [&]() -> uint64_t {
    if (pos - wbase == 64) {
      cur = nxt;
      wbase += 64;
      nxt = window(wbase + 64);
    }
    return (uint32_t)__builtin_amdgcn_readlane(cur, (int)(pos++ - wbase));
  };
  uint64_t d = 0, range = kRcTop;
  for (int k = 0; k < 4; ++k) d = (d << 8) | next_byte();

  uint32_t c[2][kRcAhead][4];
  auto tables = [&](int set, size_t t0) {  // steps past the last are read as the last one
#pragma unroll
    for (int q = 0; q < kRcAhead; ++q) {
      const uint32_t* row = cum + (min(t0 + q, n_steps - 1) * n_streams + s) * 257;
#pragma unroll
      for (int j = 0; j < 4; ++j) c[set][q][j] = row[lane + 64 * j];
    }
  };
  auto entry = [&](const uint32_t (&e)[4], int x) -> uint64_t {
    const int l = x & 63, j = x >> 6;
    const uint32_t a = __builtin_amdgcn_readlane(e[0], l), b = __builtin_amdgcn_readlane(e[1], l);
    const uint32_t f = __builtin_amdgcn_readlane(e[2], l), g = __builtin_amdgcn_readlane(e[3], l);
    const uint32_t lo = (j & 1) ? b : a, hi = (j & 1) ? g : f;
    return (j & 2) ? hi : lo;
  };
  tables(0, 0);
  for (size_t t0 = 0; t0 < n_steps; t0 += 2 * kRcAhead) {
#pragma unroll
    for (int set = 0; set < 2; ++set) {
      tables(set ^ 1, t0 + (set + 1) * kRcAhead);
#pragma unroll
      for (int q = 0; q < kRcAhead; ++q) {
        const size_t t = t0 + set * kRcAhead + q;
        if (t >= n_steps) return;
        int cnt = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j)
          cnt += __builtin_popcountll(__ballot(((range * c[set][q][j]) >> 16) <= d));
        const int x = max(cnt - 1, 0);
        const uint64_t lo = (range * entry(c[set][q], x)) >> 16;
        const uint64_t c1 = x < 255 ? entry(c[set][q], x + 1) : (uint64_t)cum[(t * n_streams + s) * 257 + 256];
        const uint64_t hi = (range * c1) >> 16;
        d -= lo;
        range = hi - lo;
        for (int k = 0; k < 4 && range < kRcBot; ++k) {
          d = (d << 8) | next_byte();
          range <<= 8;
        }
        if (lane == 0) sym[t * n_streams + s] = (uint8_t)x;
      }
    }
  }
}

// The same, one thread per stream, for many streams (rc_wave_streams).
__global__ void rc_table_decode_thread_kernel(
    const uint32_t* __restrict__ cum, const uint8_t* __restrict__ in,
    const uint64_t* __restrict__ in_lens, size_t cap, size_t n_steps, size_t n_streams,
    uint8_t* __restrict__ sym) {
  const size_t s = (size_t)blockIdx.x * 64 + threadIdx.x;
  if (s >= n_streams) return;
  const uint8_t* p = in + s * cap;
  const uint64_t len = in_lens[s] < cap ? in_lens[s] : cap;
  RcDec d;
  rc_dec_init(d, p, len);
  for (size_t t = 0; t < n_steps; ++t) {
    const uint32_t* c = cum + (t * n_streams + s) * 257;
    const uint32_t x = rc_find(d, c);
    rc_consume(d, p, len, c[x], c[x + 1]);
    sym[t * n_streams + s] = (uint8_t)x;
  }
}

void k_rc_table_decode(const uint32_t* cum, const uint8_t* in, const uint64_t* in_lens, size_t cap,
                       size_t n_steps, size_t n_streams, uint8_t* sym, hipStream_t s) {
  if (n_streams <= rc_wave_streams(n_steps, true))
    hipLaunchKernelGGL(rc_table_decode_wave_kernel, dim3(blocks_for(n_streams, 4)), dim3(256), 0, s, cum,
                       in, in_lens, cap, n_steps, n_streams, sym);
  else
    hipLaunchKernelGGL(rc_table_decode_thread_kernel, dim3(blocks_for(n_streams, 64)), dim3(64), 0, s, cum,
                       in, in_lens, cap, n_steps, n_streams, sym);
}

// CRC-32 (IEEE 802.3, reflected polynomial 0xEDB88320), one thread per stream.
__global__ void crc32_kernel(const uint8_t* __restrict__ data, const uint64_t* __restrict__ off,
                             const uint64_t* __restrict__ lens, int n, uint32_t* __restrict__ crc) {
  __shared__ uint32_t table[256];
  for (int i = threadIdx.x; i < 256; i += blockDim.x) {
    uint32_t c = (uint32_t)i;
    for (int k = 0; k < 8; ++k) c = (c & 1u) ? (0xEDB88320u ^ (c >> 1)) : (c >> 1);
    table[i] = c;
  }
  __syncthreads();
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  const uint8_t* p = data + off[s];
  const uint64_t len = lens[s];
  uint32_t c = 0xFFFFFFFFu;
  for (uint64_t i = 0; i < len; ++i) c = table[(c ^ p[i]) & 0xFFu] ^ (c >> 8);
  crc[s] = c ^ 0xFFFFFFFFu;
}

void k_crc32(const uint8_t* data, const uint64_t* off, const uint64_t* lens, int n, uint32_t* crc,
             hipStream_t s) {
  hipLaunchKernelGGL(crc32_kernel, dim3(blocks_for(n, 64)), dim3(64), 0, s, data, off, lens, n, crc);
}

__global__ void gather_payloads_kernel(const uint8_t* __restrict__ pay,
                                       const uint64_t* __restrict__ pay_off,
                                       const uint64_t* __restrict__ len,
                                       const uint64_t* __restrict__ dst_off,
                                       uint8_t* __restrict__ dst) {
  const int s = blockIdx.x;
  const uint8_t* src = pay + pay_off[s];
  uint8_t* d = dst + dst_off[s];
  const uint64_t n = len[s];
  for (uint64_t i = threadIdx.x; i < n; i += blockDim.x) d[i] = src[i];
}

void k_gather_payloads(const uint8_t* pay, const uint64_t* pay_off, const uint64_t* len,
                       const uint64_t* dst_off, uint8_t* dst, int n, hipStream_t s) {
  if (n == 0) return;
  hipLaunchKernelGGL(gather_payloads_kernel, dim3(n), dim3(256), 0, s, pay, pay_off, len, dst_off,
                     dst);
}

}  // namespace edpc

namespace edpc {

// One wave per stream.  A carry adds one to the last byte before the coder's
// write position that is not 0xFF and zeroes the 0xFF bytes after it, so the
// bytes before that byte are final.
__global__ void __launch_bounds__(64) pay_drain_kernel(const RcEnc* __restrict__ enc,
                                                       const uint8_t* __restrict__ pay,
                                                       const uint64_t* __restrict__ pay_off,
                                                       uint64_t* __restrict__ done, int n, int all,
                                                       uint8_t* __restrict__ out, uint32_t stride,
                                                       uint32_t* __restrict__ out_len) {
  const int s = blockIdx.x;
  if (s >= n) return;
  const uint8_t* p = pay + pay_off[s];
  const uint64_t pos = enc[s].pos, d0 = done[s];
  uint64_t fin = pos;
  if (!all) {
    fin = d0;
    for (uint64_t i = pos; i > d0; --i)  // wave-uniform scan, usually one step
      if (p[i - 1] != 0xFF) { fin = i - 1; break; }
  }
  if (fin > d0 + stride) fin = d0 + stride;
  const uint32_t cnt = (uint32_t)(fin > d0 ? fin - d0 : 0);
  uint8_t* o = out + (size_t)s * stride;
  for (uint32_t i = threadIdx.x; i < cnt; i += 64) o[i] = p[d0 + i];
  __syncthreads();
  if (threadIdx.x == 0) {
    out_len[s] = cnt;
    done[s] = d0 + cnt;
  }
}

void k_pay_drain(const RcEnc* enc, const uint8_t* pay, const uint64_t* pay_off, uint64_t* done,
                 int n, bool all, uint8_t* out, uint32_t stride, uint32_t* out_len, hipStream_t s) {
  if (n <= 0) return;
  hipLaunchKernelGGL(pay_drain_kernel, dim3(n), dim3(64), 0, s, enc, pay, pay_off, done, n,
                     all ? 1 : 0, out, stride, out_len);
}

}  // namespace edpc
