// Query-agnostic cache compression by expected attention: the offline choice of the rows a
// compressed cache profile keeps (Section 2.3; Section 5, "Offline").  Runs inside kv_build,
// per layer, on the pre-rotation queries, keys and values the QKV projection just produced.
//
// Per (document, query head): the document's queries define a Gaussian (mean mu, population
// covariance S); the rotation averaged over the n positions after the document (L .. L+n-1)
// maps it to mu_r = R mu, S_r = R S R^T; every rotated key k of the head's kv head gets the
// expected log-weight  mu_r.k / sqrt(D) + k^T S_r k / (2 D)  (the Gaussian's moment generating
// function at k / sqrt(D)).  Per (document, kv head): softmax of those over the document's keys,
// times the value norm, averaged over the group's query heads, normalised to total 1 and added
// to the row's running score (one accumulator per (row, kv head): no atomics, the result does
// not depend on scheduling).  Selection: per document, the k highest scores (equal scores:
// lower row first) listed in ascending row order, by a radix select over the score bits.
//
// Work layout of the log-weight kernel (256 threads = 4 wavefronts per document segment and query
// head): the covariance of the document's queries is formed on MFMA from row tiles that arrive by
// direct loads, goes through LDS once to apply the averaged rotation (each output element combines
// at most four inputs: the rotation mixes dimension j only with j +- D/2), and the quadratic forms
// run on FP32 MFMA, 32 keys per wavefront.  Bound by the FP32 matrix rate; both products use the
// covariance's symmetry (36 of 64 blocks at D = 128).  On the vector ALU, a key per lane with
// broadcast LDS reads of S_r, a layer of 63 000 rows x 16 heads took 1286 us (65 TFLOP/s of FP32
// products, the queries' tiles transposed element by element); now 404 us.
#include <algorithm>

#include "common.h"
#include "direct_loads.h"
#include "kernels.h"

namespace kvop {

namespace {

constexpr int kEaThreads = 256;
constexpr int kEaChunk = 64;  // document rows staged in LDS at a time

template <typename T>
__device__ inline float ld_f(const T* p);
template <>
__device__ inline float ld_f<float>(const float* p) { return *p; }
template <>
__device__ inline float ld_f<bf16_t>(const bf16_t* p) { return bf2f(*p); }
// eight consecutive elements as floats (16-byte aligned for BF16, 32-byte for FP32)
__device__ inline void ld8(const float* p, float (&x)[8]) {
  const f32x4 a = *reinterpret_cast<const f32x4*>(p), b = *reinterpret_cast<const f32x4*>(p + 4);
#pragma unroll
  for (int i = 0; i < 4; i++) { x[i] = a[i]; x[i + 4] = b[i]; }
}
__device__ inline void ld8(const bf16_t* p, float (&x)[8]) {
  const u32x4 v = *reinterpret_cast<const u32x4*>(p);
#pragma unroll
  for (int i = 0; i < 4; i++) {
    x[2 * i] = __builtin_bit_cast(float, v[i] << 16);
    x[2 * i + 1] = __builtin_bit_cast(float, v[i] & 0xffff0000u);
  }
}

__device__ inline float block_sum(float v, float* red) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}
__device__ inline float block_max(float v, float* red) {
  v = wave_max(v);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

// ---------------------------------------------------------------- expected log-weights
// two transposed reads of 16 rows, with their wait
template <int STEP> __device__ inline void ds_read_tr16_x2(uint32_t a0, uint32_t a1, u32x4& f0, u32x4& f1) {
  u32x2 y0, y1, y2, y3;
  asm volatile(
      "ds_read_b64_tr_b16 %0, %4\n\tds_read_b64_tr_b16 %1, %4 offset:%c6\n\t"
      "ds_read_b64_tr_b16 %2, %5\n\tds_read_b64_tr_b16 %3, %5 offset:%c6\n\ts_waitcnt lgkmcnt(0)"
      : "=&v"(y0), "=&v"(y1), "=&v"(y2), "=&v"(y3)
      : "v"(a0), "v"(a1), "i"(STEP)
      : "memory");
  f0 = u32x4{y0[0], y0[1], y1[0], y1[1]};
  f1 = u32x4{y2[0], y2[1], y3[0], y3[1]};
}
template <int STEP> __device__ inline void ds_read_tr16_x4(const uint32_t (&ad)[4], u32x4* f) {
  u32x2 y[8];
  ds_read_tr16_x8<STEP>(ad, y);
#pragma unroll
  for (int i = 0; i < 4; i++) f[i] = u32x4{y[2 * i][0], y[2 * i][1], y[2 * i + 1][0], y[2 * i + 1][1]};
}

// four consecutive elements as floats
__device__ inline f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ inline f32x4 ld4(const bf16_t* p) {
  const u32x2 v = *reinterpret_cast<const u32x2*>(p);
  f32x4 r;
  r[0] = __builtin_bit_cast(float, v[0] << 16);
  r[1] = __builtin_bit_cast(float, v[0] & 0xffff0000u);
  r[2] = __builtin_bit_cast(float, v[1] << 16);
  r[3] = __builtin_bit_cast(float, v[1] & 0xffff0000u);
  return r;
}

template <typename T, int D>
__global__ __launch_bounds__(kEaThreads) __attribute__((amdgpu_waves_per_eu(2))) void ea_logw_kernel(const T* __restrict__ qkv, int64_t ld, int H, int Hkv,
                                                             const int64_t* __restrict__ row_off,
                                                             const int32_t* __restrict__ items, int n_future,
                                                             const float* __restrict__ cos_tab,
                                                             const float* __restrict__ sin_tab,
                                                             float* __restrict__ e_out) {
  constexpr int H2 = D / 2, NB = D / 16, SP = D + 4;   // 16-wide blocks; pitch of the covariance (floats)
  // the covariance; before it the query rows: BF16 four stages of 64 rows, FP32 one of 64
  __shared__ __attribute__((aligned(16))) float region[D * SP > kEaChunk * D * 2 ? D * SP : kEaChunk * D * 2];
  __shared__ __attribute__((aligned(16))) float mu[D], mur[D];
  __shared__ float cb[H2], sb[H2];
  // work item: (document, first key, key count); the statistics always cover all the
  // document's rows, the keys are this item's segment
  const int32_t* it = items + 3 * (blockIdx.x / H);
  const int doc = it[0], k_lo = it[1], k_hi = it[1] + it[2], h = blockIdx.x % H, g = (h * Hkv) / H;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, lr = lane & 15, lg = lane >> 4;
  const int64_t r0 = row_off[doc];
  const int L = (int)(row_off[doc + 1] - r0);
  const T* Q = qkv + r0 * ld + (int64_t)h * D;
  const T* Kp = qkv + r0 * ld + (int64_t)(H + g) * D;
  const float invL = 1.0f / (float)L;
  // averaged rotation over the future positions
  if (tid < H2) {
    float c = 0.f, s = 0.f;
#pragma unroll 8
    for (int p = L; p < L + n_future; p++) {
      c += cos_tab[(int64_t)p * H2 + tid];
      s += sin_tab[(int64_t)p * H2 + tid];
    }
    cb[tid] = c / (float)n_future;
    sb[tid] = s / (float)n_future;
  }
  // ---- mean and covariance of the pre-rotation queries; covariance into region [D][SP]
  if constexpr (sizeof(T) == 2) {
    // BF16 queries: S = sum over rows of q q^T on MFMA (exact products, FP32 sums).  Row-major tiles
    // of 64 rows by direct loads, three in flight; a transposed read gives a lane eight rows of one
    // dimension, which serves as A and as B operand.  S is symmetric: wavefront w forms the
    // blocks (j, i <= j) of block rows w and NB - 1 - w, and by a product with ones the sums of
    // those dimensions.
    constexpr int CH = D / 8, NS = 4, OPS = kEaChunk * CH / kEaThreads, TILE = kEaChunk * D;   // elements
    constexpr int SH = CH >= 16 ? 0 : (CH == 8 ? 1 : 2);          // rows that share a 256-byte bank line
    constexpr int NR = NB == 8 ? 2 : 1;                           // block rows per wavefront
    static_assert(OPS * kEaThreads == kEaChunk * CH && NS * TILE * 2 <= (int)sizeof(region), "query tiles");
    auto swz = [](int r) { return CH >= 4 ? 2 * ((r >> SH) & (CH / 2 - 1)) : 0; };
    bf16_t* tiles = reinterpret_cast<bf16_t*>(region);
    const int nt = (L + kEaChunk - 1) / kEaChunk;
    auto issue = [&](int t) {
#pragma unroll
      for (int i = 0; i < OPS; i++) {
        const int f = i * kEaThreads + tid, r = f / CH, c = (f % CH) ^ swz(r);
        load_to_lds<16>(Q + (int64_t)min(t * kEaChunk + r, L - 1) * ld + 8 * c,
                        tiles + (t % NS) * TILE + (i * kEaThreads + 64 * w) * 8);
      }
    };
    f32x4 acc[NR][NB], ones[NR];
#pragma unroll
    for (int a = 0; a < NR; a++) {
      ones[a] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < NB; i++) acc[a][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int wu = __builtin_amdgcn_readfirstlane(w);
    int jr[NR];
    jr[0] = wu < NB ? wu : -1;
    if constexpr (NR == 2) jr[1] = NB - 1 - wu;
    const u32x4 one = u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
    for (int t = 0; t < NS - 1 && t < nt; t++) issue(t);
    for (int t = 0; t < nt; t++) {
      const int behind = nt - 1 - t;
      if (behind >= NS - 2) vm_wait<(NS - 2) * OPS>();
      else if (behind == 1) vm_wait<OPS>();
      else vm_wait<0>();
      __builtin_amdgcn_s_barrier();                    // tile t visible, tile t - 1 consumed
      if (t + NS - 1 < nt) issue(t + NS - 1);
      const uint8_t* tb = reinterpret_cast<const uint8_t*>(tiles + (t % NS) * TILE);
      const int left = L - t * kEaChunk;
      if (jr[0] < 0) continue;
#pragma unroll
      for (int hs = 0; hs < kEaChunk / 32; hs++) {
        // lane (lr, lg): rows 32 hs + 4 lg + 0..3 and + 16, dimension 16 i + lr
        u32x4 fr[NB];
        const int vr = 32 * hs + 4 * lg + (lr >> 2);
        uint32_t ad[NB];
#pragma unroll
        for (int i = 0; i < NB; i++) {
          const int c = (16 * i + 4 * (lr & 3)) >> 3;
          ad[i] = (uint32_t)reinterpret_cast<uintptr_t>(tb + vr * D * 2 + (c ^ swz(vr)) * 16 + (lr & 1) * 8);
        }
        if constexpr (NB == 2) {
          ds_read_tr16_x2<16 * D * 2>(ad[0], ad[1], fr[0], fr[1]);
        } else {
#pragma unroll
          for (int i = 0; i < NB; i += 4) {
            const uint32_t a4[4] = {ad[i], ad[i + 1], ad[i + 2], ad[i + 3]};
            ds_read_tr16_x4<16 * D * 2>(a4, fr + i);
          }
        }
        if (left < kEaChunk) {                         // rows past the document: zeros
          const int ra = 32 * hs + 4 * lg;
          u32x4 keep;
#pragma unroll
          for (int q = 0; q < 2; q++) {
            keep[q] = (ra + 2 * q < left ? 0xffffu : 0u) | (ra + 2 * q + 1 < left ? 0xffff0000u : 0u);
            keep[2 + q] = (ra + 16 + 2 * q < left ? 0xffffu : 0u) | (ra + 16 + 2 * q + 1 < left ? 0xffff0000u : 0u);
          }
#pragma unroll
          for (int i = 0; i < NB; i++) fr[i] &= keep;
        }
#pragma unroll
        for (int a = 0; a < NR; a++) {
          u32x4 fj = fr[0];
#pragma unroll
          for (int i = 1; i < NB; i++)
            if (jr[a] == i) fj = fr[i];                // uniform
          ones[a] = mfma_bf16(__builtin_bit_cast(u16x8, fj), __builtin_bit_cast(u16x8, one), ones[a]);
#pragma unroll
          for (int i = 0; i < NB; i++)
            if (i <= jr[a])
              acc[a][i] = mfma_bf16(__builtin_bit_cast(u16x8, fj), __builtin_bit_cast(u16x8, fr[i]), acc[a][i]);
        }
      }
    }
    __syncthreads();                                   // the tiles are consumed: region takes the covariance
#pragma unroll
    for (int a = 0; a < NR; a++)
      if (jr[a] >= 0 && lr == 0)
#pragma unroll
        for (int r = 0; r < 4; r++) mu[16 * jr[a] + 4 * lg + r] = ones[a][r] * invL;
    __syncthreads();
#pragma unroll
    for (int a = 0; a < NR; a++)
#pragma unroll
      for (int i = 0; i < NB; i++)
        if (i <= jr[a])
#pragma unroll
          for (int r = 0; r < 4; r++) {
            const int ra = 16 * jr[a] + 4 * lg + r, rb = 16 * i + lr;
            const float v = acc[a][i][r] * invL - mu[ra] * mu[rb];
            region[ra * SP + rb] = v;
            if (i < jr[a]) region[rb * SP + ra] = v;
          }
  } else {
    // FP32 queries: mean in a pass of its own (each dimension's rows split over 256 / D threads), then
    // centred products on the vector ALU, accumulated in the lane's block of the covariance
    constexpr int BR = D / 32, BC = D / 8, SPLIT = kEaThreads / D;
    const int a0 = w * (D / 4) + (lane >> 3) * BR, b0 = (lane & 7) * BC;
    {
      const int j = tid % D, part = tid / D;
      float s = 0.f;
#pragma unroll 4
      for (int i = part; i < L; i += SPLIT) s += ld_f(Q + (int64_t)i * ld + j);
      region[tid] = s;
      __syncthreads();
      if (tid < D) {
        float t = 0.f;
        for (int q = 0; q < SPLIT; q++) t += region[q * D + tid];
        mu[tid] = t / (float)L;
      }
      __syncthreads();
    }
    float acc[BR][BC];
#pragma unroll
    for (int a = 0; a < BR; a++)
#pragma unroll
      for (int b = 0; b < BC; b++) acc[a][b] = 0.f;
    for (int c0 = 0; c0 < L; c0 += kEaChunk) {
      for (int e = tid; e < kEaChunk * D; e += kEaThreads) {
        const int i = e / D, j = e % D;
        region[e] = (c0 + i < L) ? ld_f(Q + (int64_t)(c0 + i) * ld + j) - mu[j] : 0.f;
      }
      __syncthreads();
      const int n = min(kEaChunk, L - c0);
#pragma unroll 1
      for (int i = 0; i < n; i++) {
        const float* x = region + i * D;
        float xa[BR], xb[BC];
#pragma unroll
        for (int a = 0; a < BR; a++) xa[a] = x[a0 + a];
#pragma unroll
        for (int b = 0; b < BC; b++) xb[b] = x[b0 + b];
#pragma unroll
        for (int a = 0; a < BR; a++)
#pragma unroll
          for (int b = 0; b < BC; b++) acc[a][b] = fmaf(xa[a], xb[b], acc[a][b]);
      }
      __syncthreads();
    }
#pragma unroll
    for (int a = 0; a < BR; a++)
#pragma unroll
      for (int b = 0; b < BC; b++) region[(a0 + a) * SP + b0 + b] = acc[a][b] * invL;
  }
  __syncthreads();
  // ---- the rotated mean, and S_r = R S R^T in place, one 2x2 quad (a, a + D/2) x (b, b + D/2) at a
  // time: the rotation mixes dimension j only with j + D/2, so a quad's outputs depend only on its inputs
  if (tid < D) {
    const int j = tid % H2;
    mur[tid] = tid < H2 ? cb[j] * mu[tid] - sb[j] * mu[tid + H2] : sb[j] * mu[j] + cb[j] * mu[tid];
  }
  for (int qd = tid; qd < H2 * H2; qd += kEaThreads) {
    const int qa = qd / H2, qb = qd % H2;
    float* r0p = region + qa * SP;
    float* r1p = region + (qa + H2) * SP;
    const float s00 = r0p[qb], s01 = r0p[qb + H2], s10 = r1p[qb], s11 = r1p[qb + H2];
    const float ca = cb[qa], sa = sb[qa], cc = cb[qb], sc = sb[qb];
    const float t00 = ca * s00 - sa * s10, t01 = ca * s01 - sa * s11;  // rows: R S
    const float t10 = sa * s00 + ca * s10, t11 = sa * s01 + ca * s11;
    r0p[qb] = cc * t00 - sc * t01;                                     // columns: (R S) R^T
    r0p[qb + H2] = sc * t00 + cc * t01;
    r1p[qb] = cc * t10 - sc * t11;
    r1p[qb + H2] = sc * t10 + cc * t11;
  }
  __syncthreads();
  // ---- expected log-weight of every rotated key: Y = S_r K^T on FP32 MFMA (products and sums in
  // FP32), 32 keys per wavefront.  A lane holds dimensions 16 i + 4 lg + 0..3 of key lr (and of key
  // 16 + lr): they are the B operand of block i (its depth runs over 4 lg + s), and Y comes out
  // with the same dimensions in the same lane, so k . Y needs only a sum over the lane groups.
  // S_r is symmetric: k^T S_r k = sum over block rows j of k_j . (2 sum_{i<j} S_ji k_i + S_jj k_j).
  const float inv_sqrt_d = rsqrtf((float)D), inv_2d = 0.5f / (float)D;
  for (int c0 = k_lo + 32 * w; c0 < k_hi; c0 += 32 * (kEaThreads / 64)) {
    f32x4 kv[2][NB];
#pragma unroll
    for (int u = 0; u < 2; u++) {
      const int p = min(c0 + 16 * u + lr, k_hi - 1);
      const T* kr = Kp + (int64_t)p * ld + 4 * lg;
      const float* ct = cos_tab + (int64_t)p * H2 + 4 * lg;
      const float* st = sin_tab + (int64_t)p * H2 + 4 * lg;
#pragma unroll
      for (int i = 0; i < NB / 2; i++) {
        const f32x4 x1 = ld4(kr + 16 * i), x2 = ld4(kr + 16 * i + H2), cs = ld4(ct + 16 * i), sn = ld4(st + 16 * i);
        kv[u][i] = x1 * cs - x2 * sn;
        kv[u][i + NB / 2] = x2 * cs + x1 * sn;
      }
    }
    float e[2] = {0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NB; j++) {
      asm volatile("" ::: "memory");                   // one block row's reads at a time (registers)
      const float* srow = region + (16 * j + lr) * SP + 4 * lg;
      f32x4 y[2];
#pragma unroll
      for (int u = 0; u < 2; u++) y[u] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i <= j; i++) {
        if (i == j) {
#pragma unroll
          for (int u = 0; u < 2; u++) y[u] += y[u];
        }
        const f32x4 s4 = *reinterpret_cast<const f32x4*>(srow + 16 * i);
#pragma unroll
        for (int s = 0; s < 4; s++)
#pragma unroll
          for (int u = 0; u < 2; u++) y[u] = mfma_f32(s4[s], kv[u][i][s], y[u]);
      }
      const f32x4 m4 = *reinterpret_cast<const f32x4*>(mur + 16 * j + 4 * lg);
#pragma unroll
      for (int u = 0; u < 2; u++)
#pragma unroll
        for (int s = 0; s < 4; s++) e[u] = fmaf(kv[u][j][s], fmaf(y[u][s], inv_2d, m4[s] * inv_sqrt_d), e[u]);
    }
#pragma unroll
    for (int u = 0; u < 2; u++) {
      e[u] += __shfl_xor(e[u], 16, 64);
      e[u] += __shfl_xor(e[u], 32, 64);
      const int p = c0 + 16 * u + lr;
      if (lg == 0 && p < k_hi) e_out[(r0 + p) * H + h] = e[u];
    }
  }
}

// ---------------------------------------------------------------- contributions
template <typename T, int D>
__global__ __launch_bounds__(kEaThreads) void ea_contrib_kernel(const T* __restrict__ qkv, int64_t ld, int H, int Hkv,
                                                                const int64_t* __restrict__ row_off,
                                                                const int32_t* __restrict__ order,
                                                                const float* __restrict__ e_in,
                                                                float* __restrict__ acc) {
  constexpr int kKeep = 8192;
  __shared__ float red[4], keep[kKeep];
  __shared__ float mx[64], zs[64];
  const int doc = order[blockIdx.x / Hkv], g = blockIdx.x % Hkv, G = H / Hkv;
  const int tid = threadIdx.x;
  const int64_t r0 = row_off[doc];
  const int L = (int)(row_off[doc + 1] - r0);
  const T* V = qkv + r0 * ld + (int64_t)(H + Hkv + g) * D;
  for (int q = 0; q < G; q++) {
    const int h = g * G + q;
    float m = -INFINITY;
#pragma unroll 4
    for (int i = tid; i < L; i += kEaThreads) m = fmaxf(m, e_in[(r0 + i) * H + h]);
    m = block_max(m, red);
    float z = 0.f;
#pragma unroll 4
    for (int i = tid; i < L; i += kEaThreads) z += __expf(e_in[(r0 + i) * H + h] - m);
    z = block_sum(z, red);
    if (tid == 0) { mx[q] = m; zs[q] = z; }
  }
  __syncthreads();
  auto contrib = [&](int i) {
    float vn = 0.f;
    const T* v = V + (int64_t)i * ld;
#pragma unroll
    for (int j = 0; j < D; j += 8) {
      float x[8];
      ld8(v + j, x);
#pragma unroll
      for (int u = 0; u < 8; u++) vn = fmaf(x[u], x[u], vn);
    }
    float wsum = 0.f;
    for (int q = 0; q < G; q++) wsum += __expf(e_in[(r0 + i) * H + g * G + q] - mx[q]) / zs[q];
    return wsum / (float)G * sqrtf(vn);
  };
  // the first kKeep rows' contributions wait in LDS for the document's total
  float tot = 0.f;
  for (int i = tid; i < L; i += kEaThreads) {
    const float c = contrib(i);
    if (i < kKeep) keep[i] = c;
    tot += c;
  }
  tot = block_sum(tot, red);
  for (int i = tid; i < L; i += kEaThreads)
    acc[(r0 + i) * Hkv + g] += tot > 0.f ? (i < kKeep ? keep[i] : contrib(i)) / tot : 1.0f / (float)L;
}

__global__ void ea_finish_kernel(const float* __restrict__ acc, int Hkv, int rows, float* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows) return;
  float s = 0.f;
  for (int g = 0; g < Hkv; g++) s += acc[(int64_t)i * Hkv + g];
  out[i] = s;
}

__global__ void ea_zero_kernel(float* __restrict__ p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.f;
}

// ---------------------------------------------------------------- selection
// float -> unsigned key with the same order (all finite values and infinities)
__device__ inline uint32_t order_key(float f) {
  const uint32_t u = __builtin_bit_cast(uint32_t, f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// inclusive prefix sum over a wavefront
__device__ inline int wave_scan(int v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(v, o, 64);
    if (lane >= o) v += y;
  }
  return v;
}
__device__ inline int bits_below(uint64_t mask) {   // set bits of mask below this lane's
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

// sum over a wavefront, the same in every lane's view (register-to-register steps: a shuffle goes
// through LDS)
template <int CTRL, int ROWS> __device__ inline int dpp_add(int v) {
  return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false);
}
__device__ inline int wave_total(int v) {
  v = dpp_add<0x111, 0xf>(v);   // row_shr 1, 2, 4, 8: lane 15 of each row of 16 holds the row's sum
  v = dpp_add<0x112, 0xf>(v);
  v = dpp_add<0x114, 0xf>(v);
  v = dpp_add<0x118, 0xf>(v);
  v = dpp_add<0x142, 0xa>(v);   // row_bcast 15 into rows 1 and 3, row_bcast 31 into rows 2 and 3
  v = dpp_add<0x143, 0xc>(v);
  return __builtin_amdgcn_readlane(v, 63);
}

// NW wavefronts per document: the threshold bit by bit from the first bit in which the document's
// keys differ, ending as soon as exactly k keys lie at or above it, then one pass that writes
// the rows in order.  The keys stay in registers, 16 a lane; only documents over 4096 rows are read
// again in each pass.
// Bound by the chain of passes and, over many documents, by instructions.  So a document that fits
// one wavefront's registers gets one wavefront (no barriers, nothing computed four times over),
// a longer one a workgroup.  4096 documents of 512 rows in the median (2.7 M scores): 134 us with 33
// passes over memory and block reductions, 42 with a workgroup for every document, 41 with a
// wavefront for every document, now 23.
constexpr int kSelRegs = 16, kSelShort = kSelRegs * 64;
template <int NW>
__device__ __forceinline__ void select_rows(const float* __restrict__ scores, int L, int k, int32_t* __restrict__ out, int w) {
  constexpr int REGS = kSelRegs, ROW = 64 * NW, kSelRows = REGS * ROW;
  static_assert(REGS * NW <= 64, "a lane per register and wavefront in the prefix sums");
  __shared__ uint32_t red[2][NW];
  __shared__ int cnt[2][NW], tab[2][64];
  const int lane = threadIdx.x & 63, tid = 64 * w + lane;
  const bool many = L > kSelRows;
  uint32_t key[REGS];
  // f(register) for the registers that hold rows of the segment at c0, four (a branch) at a time
  auto regs = [&](int c0, auto f) __attribute__((always_inline)) {
#pragma unroll
    for (int g = 0; g < REGS; g += 4)
      if (c0 + g * ROW < L) {
#pragma unroll
        for (int j = g; j < g + 4; j++) f(j);
      }
  };
  auto load = [&](int c0) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < REGS; j++) key[j] = 0u;   // below every threshold tried
    // all loads first: a key formed beside its load would wait for it before the next load starts
    regs(c0, [&](int j) __attribute__((always_inline)) {
      key[j] = __builtin_bit_cast(uint32_t, scores[min(c0 + j * ROW + tid, L - 1)]);
    });
    __builtin_amdgcn_sched_barrier(0);
    regs(c0, [&](int j) __attribute__((always_inline)) {
      key[j] = c0 + j * ROW + tid < L ? order_key(__builtin_bit_cast(float, key[j])) : 0u;
    });
  };
  // f(row, register) over the document's rows, a whole wavefront at a time
  auto each = [&](auto f) __attribute__((always_inline)) {
    for (int c0 = 0; c0 < L; c0 += kSelRows) {
      if (many) load(c0);
      regs(c0, [&](int j) __attribute__((always_inline)) { f(c0 + j * ROW + tid, j); });
    }
  };
  load(0);

  // ---- the bits that all keys share
  uint32_t all = ~0u, any = 0u;
  each([&](int i, int j) __attribute__((always_inline)) {
    if (i < L) {
      all &= key[j];
      any |= key[j];
    }
  });
#pragma unroll
  for (int o = 32; o; o >>= 1) {
    all &= (uint32_t)__shfl_xor((int)all, o, 64);
    any |= (uint32_t)__shfl_xor((int)any, o, 64);
  }
  if constexpr (NW > 1) {
    if (lane == 0) {
      red[0][w] = all;
      red[1][w] = any;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NW; q++) {
      all &= red[0][q];
      any |= red[1][q];
    }
  }
  all = __builtin_amdgcn_readfirstlane(all);
  any = __builtin_amdgcn_readfirstlane(any);

  // ---- largest t with #(key >= t) >= k
  int par = 0;
  auto total = [&](int c) __attribute__((always_inline)) {   // of the lanes' counts
    c = wave_total(c);
    if constexpr (NW > 1) {
      if (lane == 0) cnt[par][w] = c;
      __syncthreads();
      c = 0;
#pragma unroll
      for (int q = 0; q < NW; q++) c += cnt[par][q];
      par ^= 1;
    }
    return __builtin_amdgcn_readfirstlane(c);
  };
  const int top = all == any ? -1 : 31 - __builtin_clz(all ^ any);
  uint32_t t = top < 0 ? all : all & ~((2u << top) - 1u);
  bool exact = false;
  for (int bit = top; bit >= 0 && !exact; bit--) {
    const uint32_t cand = t | (1u << bit);
    int c = 0;
    each([&](int, int j) __attribute__((always_inline)) { c += key[j] >= cand ? 1 : 0; });
    c = total(c);
    if (c >= k) t = cand;
    exact = c == k;
  }
  int need = 0;   // rows equal to t still to take, where not all of them are
  if (!exact) {
    int c = 0;
    each([&](int i, int j) __attribute__((always_inline)) { c += i < L && key[j] > t ? 1 : 0; });
    need = k - total(c);
  }

  // ---- rows in order: a register's rows of all wavefronts come before the next register's
  // lane j NW + w: the sum over the registers and wavefronts before (j, w), from each one's count
  int eq_before = 0, out_before = 0;
  auto prefix = [&](int v, int* before, int which) __attribute__((always_inline)) {
    if constexpr (NW > 1) {
      __syncthreads();
      v = tab[which][lane];
    }
    const int inc = wave_scan(v), base = *before + inc - v;
    *before += __builtin_amdgcn_readlane(inc, 63);
    return base;
  };
  auto put = [&](int& v, int j, int c, int which) __attribute__((always_inline)) {
    if constexpr (NW > 1) {
      if (lane == 0) tab[which][j * NW + w] = c;
    } else {
      v = lane == j ? c : v;
    }
  };
  for (int c0 = 0; c0 < L; c0 += kSelRows) {
    if (many) load(c0);
    if (NW > 1) {
      if (tid < 64) tab[0][tid] = tab[1][tid] = 0;   // registers past the document's end
      __syncthreads();
    }
    int eq_base = 0;
    if (!exact) {
      int v = 0;
      regs(c0, [&](int j) __attribute__((always_inline)) {
        put(v, j, __popcll(__ballot(c0 + j * ROW + tid < L && key[j] == t)), 0);
      });
      eq_base = prefix(v, &eq_before, 0);
    }
    auto taken = [&](int j) __attribute__((always_inline)) {
      const bool in = c0 + j * ROW + tid < L;
      if (exact) return in && key[j] >= t;
      const bool eq = in && key[j] == t;
      const int rank = __builtin_amdgcn_readlane(eq_base, j * NW + w) + bits_below(__ballot(eq));
      return in && (key[j] > t || (eq && rank < need));
    };
    int v = 0;
    regs(c0, [&](int j) __attribute__((always_inline)) { put(v, j, __popcll(__ballot(taken(j))), 1); });
    const int base = prefix(v, &out_before, 1);
    regs(c0, [&](int j) __attribute__((always_inline)) {
      const bool tk = taken(j);
      const int pos = __builtin_amdgcn_readlane(base, j * NW + w) + bits_below(__ballot(tk));
      if (tk) out[pos] = c0 + j * ROW + tid;
    });
    if (NW > 1 && many) __syncthreads();
  }
}

// order: the n_long documents of more than kSelShort rows, a workgroup each, then the others, a
// wavefront each (null: none is long)
__global__ __launch_bounds__(kEaThreads) void ea_select_kernel(const float* __restrict__ scores,
                                                               const int64_t* __restrict__ doc_off,
                                                               const int32_t* __restrict__ kcount,
                                                               const int64_t* __restrict__ out_off,
                                                               const int32_t* __restrict__ order, int n_docs, int n_long,
                                                               int32_t* __restrict__ idx) {
  constexpr int NW = kEaThreads / 64;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), b = blockIdx.x;
  const bool is_long = b < n_long;
  const int at = is_long ? b : n_long + (b - n_long) * NW + w;
  if (at >= n_docs) return;
  const int d = order ? order[at] : at;
  const int64_t s0 = doc_off[d];
  const int L = (int)(doc_off[d + 1] - s0), k = kcount[d];
  int32_t* out = idx + out_off[d];
  if (k >= L) {
    const int tid = is_long ? (int)threadIdx.x : (int)(threadIdx.x & 63), step = is_long ? kEaThreads : 64;
    for (int i = tid; i < L; i += step) out[i] = i;
    return;
  }
  if (k <= 0) return;
  if (is_long) select_rows<NW>(scores + s0, L, k, out, w);
  else select_rows<1>(scores + s0, L, k, out, 0);
}

template <typename T, int D>
hipError_t ea_layer_t(const void* qkv, int64_t ld, int H, int Hkv, const int64_t* row_off, const int32_t* order,
                      int nd, const int32_t* items, int n_items, int n_future, const float* cos_tab,
                      const float* sin_tab, float* e_ws, float* acc, hipStream_t st) {
  hipLaunchKernelGGL((ea_logw_kernel<T, D>), dim3(n_items * H), dim3(kEaThreads), 0, st, (const T*)qkv, ld, H, Hkv,
                     row_off, items, n_future, cos_tab, sin_tab, e_ws);
  hipLaunchKernelGGL((ea_contrib_kernel<T, D>), dim3(nd * Hkv), dim3(kEaThreads), 0, st, (const T*)qkv, ld, H, Hkv,
                     row_off, order, (const float*)e_ws, acc);
  return hipGetLastError();
}

}  // namespace

hipError_t ea_layer(int dt, int D, const void* qkv, int64_t ld, int H, int Hkv, const int64_t* row_off,
                    const int32_t* order, int nd, const int32_t* items, int n_items, int n_future,
                    const float* cos_tab, const float* sin_tab, float* e_ws, float* acc, hipStream_t st) {
  if (nd <= 0) return hipSuccess;
  if (H % Hkv || H / Hkv > 64) return hipErrorInvalidValue;
  if (dt == DT_F32) {
    if (D == 128) return ea_layer_t<float, 128>(qkv, ld, H, Hkv, row_off, order, nd, items, n_items, n_future, cos_tab, sin_tab, e_ws, acc, st);
    if (D == 64) return ea_layer_t<float, 64>(qkv, ld, H, Hkv, row_off, order, nd, items, n_items, n_future, cos_tab, sin_tab, e_ws, acc, st);
    if (D == 32) return ea_layer_t<float, 32>(qkv, ld, H, Hkv, row_off, order, nd, items, n_items, n_future, cos_tab, sin_tab, e_ws, acc, st);
  } else {
    if (D == 128) return ea_layer_t<bf16_t, 128>(qkv, ld, H, Hkv, row_off, order, nd, items, n_items, n_future, cos_tab, sin_tab, e_ws, acc, st);
    if (D == 64) return ea_layer_t<bf16_t, 64>(qkv, ld, H, Hkv, row_off, order, nd, items, n_items, n_future, cos_tab, sin_tab, e_ws, acc, st);
    if (D == 32) return ea_layer_t<bf16_t, 32>(qkv, ld, H, Hkv, row_off, order, nd, items, n_items, n_future, cos_tab, sin_tab, e_ws, acc, st);
  }
  return hipErrorInvalidValue;
}

hipError_t ea_zero(float* p, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(ea_zero_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, n);
  return hipGetLastError();
}

hipError_t ea_finish(const float* acc, int Hkv, int rows, float* out, hipStream_t st) {
  if (rows <= 0) return hipSuccess;
  hipLaunchKernelGGL(ea_finish_kernel, dim3((rows + 255) / 256), dim3(256), 0, st, acc, Hkv, rows, out);
  return hipGetLastError();
}

hipError_t ea_select(const float* scores, const int64_t* doc_off, const int32_t* kcount, const int64_t* out_off,
                     const int32_t* order, int n_docs, int n_long, int32_t* idx, hipStream_t st) {
  if (n_docs <= 0) return hipSuccess;
  constexpr int NW = kEaThreads / 64;
  hipLaunchKernelGGL(ea_select_kernel, dim3(n_long + (n_docs - n_long + NW - 1) / NW), dim3(kEaThreads), 0, st, scores,
                     doc_off, kcount, out_off, order, n_docs, n_long, idx);
  return hipGetLastError();
}

int ea_select_short() { return kSelShort; }

}  // namespace kvop
