// Learned proxy: z = W2 gelu(W1 x + b1) + b2 on standardised pooled document features,
// p = softmax(z), answered iff max p > tau (the confident items of a two-stage cascade).
//
// Training step (BF16 compute, FP32 master weights, deterministic):
//   gather    : x = bf16((F[row] - mean) * inv_std) for the minibatch rows, also transposed
//   layer 1   : h1 = x W1^T on the BF16 MFMA projection kernel (FP32 out)
//   head      : one wavefront per row: a = gelu(h1 + b1), z = a W2^T + b2, softmax, CE loss,
//               dz = (p - y)/B, da = dz W2, dh1 = da * gelu'(h1 + b1) (FP32; dh1^T also in BF16)
//   dW1       : dh1^T x on the projection kernel (contraction over the batch)
//   reduce    : dW2 = dz^T a, db2 = sum dz, db1 = sum dh1, loss = mean CE (fixed order)
//   adam      : bias-corrected Adam on the FP32 masters; refresh the BF16 copy of W1
#include <algorithm>

#include "common.h"
#include "direct_loads.h"
#include "kernels.h"

namespace kvop {

// ---------------------------------------------------------------- standardiser
// mean and 1/std over n rows (two passes, FP32, rows added in order; std floor 1e-6)
//
// Bound: a column's sum is one chain of n dependent additions per pass, so it is kept in one
// lane and everything else is taken off its path: 16 columns per workgroup (128 CUs at
// d = 2048), one wavefront that only adds, four that stream the 64-byte row pieces into LDS by
// direct loads, 112 KiB in flight.  20 000 x 2048: 9335 us with one thread per column reading
// its own rows (8 workgroups, one load latency every few rows), now 226 us (5.6 ns a row and pass).
constexpr int kStatCols = 16, kStatRows = 256, kStatStages = 8, kStatLoaders = 4;

__global__ __launch_bounds__(64 * (1 + kStatLoaders)) void proxy_stats_kernel(const float* __restrict__ F, int64_t n,
                                                                             int d, float* __restrict__ mean,
                                                                             float* __restrict__ istd) {
  extern __shared__ __attribute__((aligned(16))) float stat_smem[];   // [stage][row][16 columns]
  constexpr int STAGE = kStatRows * kStatCols, OPS = kStatRows * kStatCols / 4 / (64 * kStatLoaders);
  // workgroup b runs on XCD b % 8: neighbouring column groups, which share 128-byte lines, go to
  // the same XCD's L2
  const int nb = gridDim.x, xcd = blockIdx.x & 7, per = nb >> 3, rem = nb & 7;
  const int cg = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + (blockIdx.x >> 3);
  const int c0 = cg * kStatCols, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, col = lane % kStatCols;
  const int nt = (int)((n + kStatRows - 1) / kStatRows);               // stages per pass
  auto issue = [&](int t) {                                            // stage t of either pass
    const int64_t r0 = (int64_t)(t < nt ? t : t - nt) * kStatRows;
    float* dst = stat_smem + (t % kStatStages) * STAGE;
#pragma unroll
    for (int i = 0; i < OPS; i++) {
      const int f = i * 64 * kStatLoaders + 64 * (wave - 1) + lane;    // 16-byte chunk: row f / 4, columns 4 (f % 4)
      const int64_t row = r0 + f / 4 < n ? r0 + f / 4 : n - 1;
      load_to_lds<16>(F + row * d + c0 + 4 * (f % 4), dst + (i * 64 * kStatLoaders + 64 * (wave - 1)) * 4);
    }
  };
  if (wave > 0) {
    for (int t = 0; t < kStatStages - 1 && t < 2 * nt; t++) issue(t);
    for (int t = 0; t < 2 * nt; t++) {
      vm_wait_behind<kStatStages - 2, OPS, 0>(2 * nt - 1 - t);
      __builtin_amdgcn_s_barrier();                                    // stage t visible, stage t - 1 consumed
      if (t + kStatStages - 1 < 2 * nt) issue(t + kStatStages - 1);
    }
    return;
  }
  float s = 0.f, mu = 0.f, q = 0.f;
  for (int t = 0; t < 2 * nt; t++) {
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");                                     // the reads below stay behind the barrier
    const float* x = stat_smem + (t % kStatStages) * STAGE + col;
    const bool second = t >= nt;
    const int64_t left = n - (int64_t)(second ? t - nt : t) * kStatRows;
    const int rows = left < kStatRows ? (int)left : kStatRows;
    // 32 rows are read ahead of the 32 being added
    auto walk = [&](auto add) __attribute__((always_inline)) {
      if (rows == kStatRows) {
        float cur[32], nxt[32];
#pragma unroll
        for (int r = 0; r < 32; r++) cur[r] = x[r * kStatCols];
#pragma unroll
        for (int g = 0; g < kStatRows / 32; g++) {
          if (g + 1 < kStatRows / 32) {
#pragma unroll
            for (int r = 0; r < 32; r++) nxt[r] = x[(32 * (g + 1) + r) * kStatCols];
          }
          asm volatile("" ::: "memory");
#pragma unroll
          for (int r = 0; r < 32; r++) add(cur[r]);
#pragma unroll
          for (int r = 0; r < 32; r++) cur[r] = nxt[r];
        }
      } else {
        for (int r = 0; r < rows; r++) add(x[r * kStatCols]);
      }
    };
    if (!second) {
      walk([&](float v) { s += v; });
      if (t == nt - 1) mu = s / (float)n;
    } else {
      walk([&](float v) {
        const float dv = v - mu;
        q = __builtin_fmaf(dv, dv, q);
      });
    }
  }
  if (lane < kStatCols) {
    const float sd = sqrtf(q / (float)n);
    mean[c0 + col] = mu;
    istd[c0 + col] = 1.0f / fmaxf(sd, 1e-6f);
  }
}

// features that do not start on a 16-byte boundary: one thread per column
__global__ void proxy_stats_unaligned_kernel(const float* __restrict__ F, int64_t n, int d, float* __restrict__ mean,
                                             float* __restrict__ istd) {
  int c = blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= d) return;
  float s = 0.f;
  for (int64_t r = 0; r < n; r++) s += F[r * d + c];
  float mu = s / (float)n;
  float q = 0.f;
  for (int64_t r = 0; r < n; r++) {
    float t = F[r * d + c] - mu;
    q = __builtin_fmaf(t, t, q);
  }
  float sd = sqrtf(q / (float)n);
  mean[c] = mu;
  istd[c] = 1.0f / fmaxf(sd, 1e-6f);
}

hipError_t proxy_stats(const float* F, int64_t n, int d, float* mean, float* istd, hipStream_t st) {
  if (n < 1 || d % kStatCols) return hipErrorInvalidValue;
  if (reinterpret_cast<uintptr_t>(F) & 15) {
    hipLaunchKernelGGL(proxy_stats_unaligned_kernel, dim3((d + 255) / 256), dim3(256), 0, st, F, n, d, mean, istd);
    return hipGetLastError();
  }
  constexpr size_t lds = (size_t)kStatStages * kStatRows * kStatCols * 4;
  static const hipError_t attr =
      hipFuncSetAttribute((const void*)proxy_stats_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(proxy_stats_kernel, dim3(d / kStatCols), dim3(64 * (1 + kStatLoaders)), lds, st, F, n, d, mean,
                     istd);
  return hipGetLastError();
}

// ---------------------------------------------------------------- gather (+ transpose)
// tile of 32 rows x 64 features per workgroup, four features per lane and load; xT (optional)
// receives the transpose, eight rows per store (B a multiple of 8 then)
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));   // features may start anywhere
__global__ __launch_bounds__(256) void proxy_gather_kernel(const float* __restrict__ F, int d,
                                                           const int32_t* __restrict__ rows, int B,
                                                           const float* __restrict__ mean,
                                                           const float* __restrict__ istd, bf16_t* __restrict__ x,
                                                           bf16_t* __restrict__ xT) {
  __shared__ bf16_t tile[32][64 + 2];
  const int r0 = blockIdx.y * 32, cc = 4 * (threadIdx.x % 16), c = blockIdx.x * 64 + cc;
  const f32x4 mu = *reinterpret_cast<const f32x4*>(mean + c), is = *reinterpret_cast<const f32x4*>(istd + c);
  f32x4_any v[2];
#pragma unroll
  for (int i = 0; i < 2; i++) {
    const int b = min(r0 + 16 * i + (int)threadIdx.x / 16, B - 1);
    const int64_t src = rows ? rows[b] : b;
    v[i] = *reinterpret_cast<const f32x4_any*>(F + src * d + c);
  }
#pragma unroll
  for (int i = 0; i < 2; i++) {
    const int rr = 16 * i + threadIdx.x / 16, b = r0 + rr;
    u32x2 pk;
    pk[0] = pack_bf16x2((v[i][0] - mu[0]) * is[0], (v[i][1] - mu[1]) * is[1]);
    pk[1] = pack_bf16x2((v[i][2] - mu[2]) * is[2], (v[i][3] - mu[3]) * is[3]);
    if (b < B) *reinterpret_cast<u32x2*>(x + (int64_t)b * d + c) = pk;
    *reinterpret_cast<uint32_t*>(&tile[rr][cc]) = pk[0];
    *reinterpret_cast<uint32_t*>(&tile[rr][cc + 2]) = pk[1];
  }
  if (!xT) return;
  __syncthreads();
  const int tc = threadIdx.x / 4, b8 = 8 * (threadIdx.x % 4);
  if (r0 + b8 < B) {
    u32x4 o;
#pragma unroll
    for (int q = 0; q < 4; q++) o[q] = (uint32_t)tile[b8 + 2 * q][tc] | ((uint32_t)tile[b8 + 2 * q + 1][tc] << 16);
    *reinterpret_cast<u32x4*>(xT + (int64_t)(blockIdx.x * 64 + tc) * B + r0 + b8) = o;
  }
}

hipError_t proxy_gather(const float* F, int d, const int32_t* rows, int B, const float* mean, const float* istd,
                        bf16_t* x, bf16_t* xT, hipStream_t st) {
  if (B <= 0) return hipSuccess;
  if (d % 64 || (xT && B % 8)) return hipErrorInvalidValue;
  dim3 grid(d / 64, (B + 31) / 32);
  hipLaunchKernelGGL(proxy_gather_kernel, grid, dim3(256), 0, st, F, d, rows, B, mean, istd, x, xT);
  return hipGetLastError();
}

// ---------------------------------------------------------------- per-row head
__device__ inline float gelu_f(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ inline float gelu_grad_f(float x) {
  return 0.5f * (1.0f + erff(x * 0.70710678118654752f)) + x * 0.39894228040143268f * expf(-0.5f * x * x);
}

// Inference over blocks of 16 MB rows in one pass over the features: each of the first MB
// wavefronts standardises 16 rows in registers (its A fragments, loaded PA slabs ahead) and
// multiplies them with slabs of W1 that two more wavefronts bring into LDS by direct loads; the
// hidden pre-activations then go through LDS to the per-row head below, in its order of
// additions.  The MFMA steps run over the depth in order, as the projection tiles do, so the
// results equal the separate passes (gather, projection, head) bit for bit.
//
// Bound by reading the features once (164 MB for 20 000 x 2048).  The rows per workgroup are the
// fewest that make one round of the 256 CUs (32 to 96): every workgroup streams all of W1 from
// L2, and a second round would cost as much again.  20 000 rows: 133 us as three passes (72
// gather, 48 projection, 13 head) when this was written, 56 us now.
constexpr int kInferLoaders = 2, kInferStages = 4, kInferAhead = 3;

template <int MB, int H>
__global__ __launch_bounds__(64 * (MB + kInferLoaders)) void proxy_infer_kernel(
    const float* __restrict__ F, int n, int d, const float* __restrict__ mean, const float* __restrict__ istd,
    const bf16_t* __restrict__ W1, const float* __restrict__ b1, const float* __restrict__ W2,
    const float* __restrict__ b2, float tau, int8_t* __restrict__ cls, float* __restrict__ conf,
    int8_t* __restrict__ answered) {
  extern __shared__ __attribute__((aligned(16))) uint8_t infer_smem[];
  constexpr int NB = H / 16, OPS = H * 8 / (64 * kInferLoaders), STAGE = H * 128, U = H / 64, EP = H + 4;
  static_assert(OPS * 64 * kInferLoaders == H * 8, "chunks per loader thread");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r0 = blockIdx.x * 16 * MB, nt = d / 64;
  // the standardiser in LDS: read from memory beside the features, every use of it would wait for
  // the features in flight (loads return in order)
  float* st_mean = reinterpret_cast<float*>(infer_smem + (size_t)kInferStages * STAGE);
  float* st_istd = st_mean + d;
  for (int c = threadIdx.x; c < d; c += blockDim.x) {
    st_mean[c] = mean[c];
    st_istd[c] = istd[c];
  }
  __syncthreads();
  if (wave >= MB) {
    // ---- W1 slabs: row j of the slab (64 deep) as eight 16-byte chunks, chunk c at slot c ^ (j / 2 & 7)
    const int lt = threadIdx.x - 64 * MB;
    auto issue = [&](int t) {
      uint8_t* dst = infer_smem + (t % kInferStages) * STAGE;
#pragma unroll
      for (int i = 0; i < OPS; i++) {
        const int f = i * 64 * kInferLoaders + lt, j = f / 8, c = (f % 8) ^ ((j >> 1) & 7);
        load_to_lds<16>(W1 + (int64_t)j * d + 64 * t + 8 * c, dst + (i * 64 * kInferLoaders + 64 * (wave - MB)) * 16);
      }
    };
    for (int t = 0; t < kInferStages - 1 && t < nt; t++) issue(t);
    for (int t = 0; t < nt; t++) {
      vm_wait_behind<kInferStages - 2, OPS, 0>(nt - 1 - t);
      __builtin_amdgcn_s_barrier();                    // slab t visible, slab t - 1 consumed
      if (t + kInferStages - 1 < nt) issue(t + kInferStages - 1);
    }
    __builtin_amdgcn_s_barrier();                      // the last slab is consumed
  } else {
    const int lrow = lane & 15, lg = lane >> 4;
    const float* fr = F + (int64_t)min(r0 + 16 * wave + lrow, n - 1) * d + 8 * lg;
    f32x4_any a[kInferAhead][4];
    auto load_a = [&](int t, f32x4_any (&v)[4]) {
#pragma unroll
      for (int q = 0; q < 4; q++) v[q] = *reinterpret_cast<const f32x4_any*>(fr + 64 * t + 32 * (q >> 1) + 4 * (q & 1));
    };
    f32x4 acc[NB];
#pragma unroll
    for (int j = 0; j < NB; j++) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < kInferAhead; u++) load_a(min(u, nt - 1), a[u]);
    for (int t0 = 0; t0 < nt; t0 += kInferAhead) {
#pragma unroll
      for (int u = 0; u < kInferAhead; u++) {
        const int t = t0 + u;
        if (t >= nt) break;
        asm volatile("" ::: "memory");                 // one slab's reads at a time (registers)
        u32x4 fa[2];
#pragma unroll
        for (int ks = 0; ks < 2; ks++)
#pragma unroll
          for (int hq = 0; hq < 2; hq++) {
            const int c = 64 * t + 32 * ks + 8 * lg + 4 * hq;
            const f32x4 mu = *reinterpret_cast<const f32x4*>(st_mean + c);
            const f32x4 is = *reinterpret_cast<const f32x4*>(st_istd + c);
            const f32x4_any v = a[u][2 * ks + hq];
            fa[ks][2 * hq] = pack_bf16x2((v[0] - mu[0]) * is[0], (v[1] - mu[1]) * is[1]);
            fa[ks][2 * hq + 1] = pack_bf16x2((v[2] - mu[2]) * is[2], (v[3] - mu[3]) * is[3]);
          }
        load_a(min(t + kInferAhead, nt - 1), a[u]);
        __builtin_amdgcn_s_barrier();                  // slab t visible
        asm volatile("" ::: "memory");
        const uint8_t* Bs = infer_smem + (t % kInferStages) * STAGE;
#pragma unroll
        for (int ks = 0; ks < 2; ks++)
#pragma unroll
          for (int j = 0; j < NB; j++) {
            const int row = 16 * j + lrow;
            const u32x4 fb = *reinterpret_cast<const u32x4*>(Bs + row * 128 + ((4 * ks + lg) ^ ((row >> 1) & 7)) * 16);
            acc[j] = mfma_bf16(__builtin_bit_cast(u16x8, fa[ks]), __builtin_bit_cast(u16x8, fb), acc[j]);
          }
      }
    }
    __builtin_amdgcn_s_barrier();                      // the last slab is consumed
    asm volatile("" ::: "memory");
    float* E = reinterpret_cast<float*>(infer_smem) + wave * 16 * EP;
#pragma unroll
    for (int j = 0; j < NB; j++)
#pragma unroll
      for (int r = 0; r < 4; r++) E[(4 * lg + r) * EP + 16 * j + lrow] = acc[j][r];
  }
  __syncthreads();
  // ---- head: one wavefront per row
  for (int rr = wave; rr < 16 * MB && r0 + rr < n; rr += MB + kInferLoaders) {
    const float* h1 = reinterpret_cast<const float*>(infer_smem) + rr * EP;
    float z0 = 0.f, z1 = 0.f;
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int j = lane + 64 * u;
      const float act = gelu_f(h1[j] + b1[j]);
      z0 = __builtin_fmaf(act, W2[j], z0);
      z1 = __builtin_fmaf(act, W2[H + j], z1);
    }
    z0 = wave_sum(z0) + b2[0];
    z1 = wave_sum(z1) + b2[1];
    const float m = fmaxf(z0, z1);
    const float e0 = expf(z0 - m), e1 = expf(z1 - m);
    const float p0 = e0 / (e0 + e1), p1 = e1 / (e0 + e1);
    if (lane == 0) {
      const int c = p1 > p0 ? 1 : 0;
      const float cf = c ? p1 : p0;
      cls[r0 + rr] = (int8_t)c;
      conf[r0 + rr] = cf;
      answered[r0 + rr] = cf > tau ? 1 : 0;
    }
  }
}

template <int MB, int H>
static hipError_t launch_infer(const float* F, int n, int d, const float* mean, const float* istd, const bf16_t* w1,
                               const float* b1, const float* W2, const float* b2, float tau, int8_t* cls, float* conf,
                               int8_t* answered, hipStream_t st) {
  static_assert((size_t)kInferStages * H * 128 >= (size_t)16 * MB * (H + 4) * 4, "pre-activations fit the slabs");
  const size_t lds = (size_t)kInferStages * H * 128 + 8 * (size_t)d;
  auto kern = proxy_infer_kernel<MB, H>;
  static const hipError_t attr =
      hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 160 << 10);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(kern, dim3((n + 16 * MB - 1) / (16 * MB)), dim3(64 * (MB + kInferLoaders)), lds, st, F, n, d, mean,
                     istd, w1, b1, W2, b2, tau, cls, conf, answered);
  return hipGetLastError();
}

// Fewer rows than this run the separate passes: a workgroup's stream of W1 takes its time whatever its
// rows (2048 -> 256: 28 us; 4096 rows 29 us in three passes, 38 in one; 8192 rows 42 and 41; 20 000
// rows 80 and 53).  From 8192 rows on one pass is the faster at every size it takes, 64 to 4096
// columns and 64 to 256 hidden units (8192 rows of 4096 -> 256 69 us and 66, of 64 -> 64 15 and 10);
// below, it depends on the size (4096 rows: 45 and 64, 15 and 9).  The standardiser has 32 KiB
// of LDS beside the slabs.
constexpr int kInferFusedRows = 8192;
static bool infer_sizes_ok(int d, int H) { return d % 64 == 0 && d <= 4096 && (H == 64 || H == 128 || H == 256); }
bool proxy_infer_fused(int n, int d, int H) { return n >= kInferFusedRows && infer_sizes_ok(d, H); }

hipError_t proxy_infer(const float* F, int n, int d, int H, const float* mean, const float* istd, const bf16_t* w1,
                       const float* b1, const float* W2, const float* b2, float tau, int8_t* cls, float* conf,
                       int8_t* answered, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  if (!infer_sizes_ok(d, H)) return hipErrorInvalidValue;
  const int mb = std::min(6, std::max(2, (n + 256 * 16 - 1) / (256 * 16)));
#define KVOP_INFER(MB)                                                                                                 \
  (H == 256   ? launch_infer<MB, 256>(F, n, d, mean, istd, w1, b1, W2, b2, tau, cls, conf, answered, st)               \
   : H == 128 ? launch_infer<MB, 128>(F, n, d, mean, istd, w1, b1, W2, b2, tau, cls, conf, answered, st)               \
              : launch_infer<MB, 64>(F, n, d, mean, istd, w1, b1, W2, b2, tau, cls, conf, answered, st))
  switch (mb) {
    case 2: return KVOP_INFER(2);
    case 3: return KVOP_INFER(3);
    case 4: return KVOP_INFER(4);
    case 5: return KVOP_INFER(5);
    default: return KVOP_INFER(6);
  }
#undef KVOP_INFER
}

// one wavefront per row; H <= 512 (H/64 hidden units per lane)
template <bool TRAIN>
__global__ __launch_bounds__(256) void proxy_head_kernel(const float* __restrict__ h1, int B, int H,
                                                         const float* __restrict__ b1, const float* __restrict__ W2,
                                                         const float* __restrict__ b2, const int32_t* __restrict__ labels,
                                                         const int32_t* __restrict__ rows, float tau,
                                                         int8_t* __restrict__ cls, float* __restrict__ conf,
                                                         int8_t* __restrict__ answered, float* __restrict__ a_out,
                                                         float* __restrict__ dz_out, float* __restrict__ dh1,
                                                         bf16_t* __restrict__ dh1T, float* __restrict__ loss_row) {
  int b = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (b >= B) return;
  constexpr int MAXU = 8;
  float pre[MAXU], act[MAXU];
  float z0 = 0.f, z1 = 0.f;
  const int U = H / 64;
#pragma unroll
  for (int u = 0; u < MAXU; u++) {
    if (u >= U) break;
    int j = lane + 64 * u;
    pre[u] = h1[(int64_t)b * H + j] + b1[j];
    act[u] = gelu_f(pre[u]);
    z0 += act[u] * W2[j];
    z1 += act[u] * W2[H + j];
  }
  z0 = wave_sum(z0) + b2[0];
  z1 = wave_sum(z1) + b2[1];
  float m = fmaxf(z0, z1);
  float e0 = expf(z0 - m), e1 = expf(z1 - m);
  float p0 = e0 / (e0 + e1), p1 = e1 / (e0 + e1);
  if constexpr (!TRAIN) {
    if (lane == 0) {
      int c = p1 > p0 ? 1 : 0;
      float cf = c ? p1 : p0;
      cls[b] = (int8_t)c;
      conf[b] = cf;
      answered[b] = cf > tau ? 1 : 0;
    }
  } else {
    int y = labels[rows ? rows[b] : b];
    float lse = m + logf(e0 + e1);
    float d0 = (p0 - (y == 0 ? 1.f : 0.f)) / (float)B;
    float d1 = (p1 - (y == 1 ? 1.f : 0.f)) / (float)B;
    if (lane == 0) {
      loss_row[b] = lse - (y == 1 ? z1 : z0);
      dz_out[2 * b] = d0;
      dz_out[2 * b + 1] = d1;
    }
#pragma unroll
    for (int u = 0; u < MAXU; u++) {
      if (u >= U) break;
      int j = lane + 64 * u;
      float da = d0 * W2[j] + d1 * W2[H + j];
      float g = da * gelu_grad_f(pre[u]);
      a_out[(int64_t)b * H + j] = act[u];
      dh1[(int64_t)b * H + j] = g;
      dh1T[(int64_t)j * B + b] = f2bf(g);
    }
  }
}

hipError_t proxy_head_infer(const float* h1, int n, int H, const float* b1, const float* W2, const float* b2,
                            float tau, int8_t* cls, float* conf, int8_t* answered, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  if (H % 64 || H > 512) return hipErrorInvalidValue;
  hipLaunchKernelGGL(proxy_head_kernel<false>, dim3((n + 3) / 4), dim3(256), 0, st, h1, n, H, b1, W2, b2, nullptr,
                     nullptr, tau, cls, conf, answered, nullptr, nullptr, nullptr, nullptr, nullptr);
  return hipGetLastError();
}

hipError_t proxy_head_train(const float* h1, int B, int H, const float* b1, const float* W2, const float* b2,
                            const int32_t* labels, const int32_t* rows, float* a, float* dz, float* dh1, bf16_t* dh1T,
                            float* loss_row, hipStream_t st) {
  if (B <= 0) return hipSuccess;
  if (H % 64 || H > 512) return hipErrorInvalidValue;
  hipLaunchKernelGGL(proxy_head_kernel<true>, dim3((B + 3) / 4), dim3(256), 0, st, h1, B, H, b1, W2, b2, labels, rows,
                     0.f, nullptr, nullptr, nullptr, a, dz, dh1, dh1T, loss_row);
  return hipGetLastError();
}

// ---------------------------------------------------------------- reductions over the batch
// Workgroup w < H / 16: db1, dW2[0], dW2[1] of hidden units 16 w .. 16 w + 15, 64 row groups of the
// batch side by side, added in a fixed order (rows rg, rg + 64, ..., then the groups); the last
// workgroup: db2 and the mean loss.  One thread per unit over the whole batch, as first
// written, took 169 us at 512 x 256 (one workgroup, a serial chain of loads); now 5 us.
__global__ __launch_bounds__(1024) void proxy_reduce_kernel(const float* __restrict__ a, const float* __restrict__ dz,
                                                            const float* __restrict__ dh1,
                                                            const float* __restrict__ loss_row, int B, int H,
                                                            float* __restrict__ g_b1, float* __restrict__ g_w2,
                                                            float* __restrict__ g_b2, float* __restrict__ loss) {
  __shared__ float part[16][16][3];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool tail = (int)blockIdx.x == H / 16;
  const int j = blockIdx.x * 16 + threadIdx.x % 16;
  float s[3] = {0.f, 0.f, 0.f};
  if (!tail) {
    for (int b = threadIdx.x / 16; b < B; b += 64) {
      const float av = a[(int64_t)b * H + j];
      s[0] += dh1[(int64_t)b * H + j];
      s[1] += dz[2 * b] * av;
      s[2] += dz[2 * b + 1] * av;
    }
  } else {
    for (int b = threadIdx.x; b < B; b += 1024) {
      s[0] += dz[2 * b];
      s[1] += dz[2 * b + 1];
      s[2] += loss_row[b];
    }
  }
#pragma unroll
  for (int k = 0; k < 3; k++) {
    if (tail) {
      s[k] = wave_sum(s[k]);
    } else {
      s[k] += __shfl_xor(s[k], 16, 64);
      s[k] += __shfl_xor(s[k], 32, 64);
    }
    if (lane < 16) part[wave][lane][k] = s[k];
  }
  __syncthreads();
  if (threadIdx.x >= 16) return;
  float t[3] = {0.f, 0.f, 0.f};
  for (int w = 0; w < 16; w++)
#pragma unroll
    for (int k = 0; k < 3; k++) t[k] += part[w][threadIdx.x][k];
  if (!tail) {
    g_b1[j] = t[0];
    g_w2[j] = t[1];
    g_w2[H + j] = t[2];
  } else if (threadIdx.x == 0) {
    g_b2[0] = t[0];
    g_b2[1] = t[1];
    if (loss) *loss = t[2] / (float)B;
  }
}

hipError_t proxy_reduce(const float* a, const float* dz, const float* dh1, const float* loss_row, int B, int H,
                        float* g_b1, float* g_w2, float* g_b2, float* loss, hipStream_t st) {
  if (H % 16) return hipErrorInvalidValue;
  hipLaunchKernelGGL(proxy_reduce_kernel, dim3(H / 16 + 1), dim3(1024), 0, st, a, dz, dh1, loss_row, B, H, g_b1, g_w2,
                     g_b2, loss);
  return hipGetLastError();
}

// ---------------------------------------------------------------- Adam
// p -= lr * mhat / (sqrt(vhat) + eps), mhat = m / (1 - b1^t), vhat = v / (1 - b2^t); the first
// n_w1 parameters (W1) are also written as BF16 for the next forward pass
__global__ void proxy_adam_kernel(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                                  float* __restrict__ v, int64_t n, int64_t n_w1, bf16_t* __restrict__ w1b, float lr,
                                  float beta1, float beta2, float eps, float c1, float c2) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float gi = g[i];
  float mi = beta1 * m[i] + (1.f - beta1) * gi;
  float vi = beta2 * v[i] + (1.f - beta2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
  p[i] = pi;
  if (i < n_w1) w1b[i] = f2bf(pi);
}

hipError_t proxy_adam(float* p, const float* g, float* m, float* v, int64_t n, int64_t n_w1, bf16_t* w1b, float lr,
                      float beta1, float beta2, float eps, int step, hipStream_t st) {
  float c1 = 1.f - powf(beta1, (float)step), c2 = 1.f - powf(beta2, (float)step);
  hipLaunchKernelGGL(proxy_adam_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, g, m, v, n, n_w1, w1b,
                     lr, beta1, beta2, eps, c1, c2);
  return hipGetLastError();
}

__global__ void f32_to_bf16_kernel(const float* __restrict__ s, bf16_t* __restrict__ d, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) d[i] = f2bf(s[i]);
}
hipError_t f32_to_bf16(const float* s, bf16_t* d, int64_t n, hipStream_t st) {
  hipLaunchKernelGGL(f32_to_bf16_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, s, d, n);
  return hipGetLastError();
}

}  // namespace kvop
