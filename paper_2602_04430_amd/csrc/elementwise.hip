// Bandwidth-bound kernels around the projections and the attention: embedding gather,
// RMSNorm (FP32 statistics), rotary embedding, the cache writer of the prefill (with
// per-16-row FP8 block quantisation), pooled document features, the restricted logit
// heads, index-list validation and weight conversion.  One wavefront per row where a
// row reduction is needed; 16-byte accesses where the layout allows.
#include "common.h"
#include "kernels.h"

namespace kvop {

// eight values in 16- or 32-byte accesses
template <typename T> struct Vec8;
template <> struct Vec8<bf16_t> {
  __device__ static void load(const bf16_t* p, float* x) {
    const u32x4 v = *reinterpret_cast<const u32x4*>(p);
#pragma unroll
    for (int q = 0; q < 4; q++) {
      x[2 * q] = bf2f((bf16_t)(v[q] & 0xffffu));
      x[2 * q + 1] = bf2f((bf16_t)(v[q] >> 16));
    }
  }
  __device__ static void store(bf16_t* p, const float* x) {
    u32x4 v;
#pragma unroll
    for (int q = 0; q < 4; q++) v[q] = pack_bf16x2(x[2 * q], x[2 * q + 1]);
    *reinterpret_cast<u32x4*>(p) = v;
  }
};
template <> struct Vec8<float> {
  __device__ static void load(const float* p, float* x) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(p), b = *reinterpret_cast<const f32x4*>(p + 4);
#pragma unroll
    for (int q = 0; q < 4; q++) { x[q] = a[q]; x[4 + q] = b[q]; }
  }
  __device__ static void store(float* p, const float* x) {
    *reinterpret_cast<f32x4*>(p) = f32x4{x[0], x[1], x[2], x[3]};
    *reinterpret_cast<f32x4*>(p + 4) = f32x4{x[4], x[5], x[6], x[7]};
  }
};

// ---------------------------------------------------------------- embedding
// A wavefront per row, eight values per lane and access, a row's pieces in flight together.  Bound by
// the bytes written: 62 870 rows of 2048 took 219 us with a workgroup per row and a value per thread
// and access, now 148.
template <typename T>
__global__ __launch_bounds__(256) void embed_kernel(const T* __restrict__ E, const int32_t* __restrict__ tok, int S,
                                                    int n_rows, int d, int vocab, float* __restrict__ x) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= n_rows) return;
  int t = S > 0 ? tok[row % S] : tok[row];
  t = min(max(t, 0), vocab - 1);  // ids are validated by the callers; the clamp only guards the gather
  const T* e = E + (int64_t)t * d;
  float* o = x + (int64_t)row * d;
  for (int c0 = 8 * lane; c0 < d; c0 += 2048) {
    float v[4][8];
#pragma unroll
    for (int u = 0; u < 4; u++) Vec8<T>::load(e + min(c0 + 512 * u, d - 8), v[u]);
#pragma unroll
    for (int u = 0; u < 4; u++)
      if (c0 + 512 * u < d) Vec8<float>::store(o + c0 + 512 * u, v[u]);
  }
}

hipError_t embed_rows(int dt, const void* E, const int32_t* tok, int n_rows, int d, int vocab, float* x,
                      hipStream_t st) {
  if (n_rows <= 0) return hipSuccess;
  if (d % 8) return hipErrorInvalidValue;   // eight-value row pieces
  if (dt == DT_F32)
    hipLaunchKernelGGL(embed_kernel<float>, dim3((n_rows + 3) / 4), dim3(256), 0, st, (const float*)E, tok, 0, n_rows, d, vocab, x);
  else
    hipLaunchKernelGGL(embed_kernel<bf16_t>, dim3((n_rows + 3) / 4), dim3(256), 0, st, (const bf16_t*)E, tok, 0, n_rows, d, vocab, x);
  return hipGetLastError();
}

hipError_t embed_suffix(int dt, const void* E, const int32_t* suffix, int S, int n_rows, int d, int vocab, float* x,
                        hipStream_t st) {
  if (n_rows <= 0) return hipSuccess;
  if (d % 8) return hipErrorInvalidValue;   // eight-value row pieces
  if (dt == DT_F32)
    hipLaunchKernelGGL(embed_kernel<float>, dim3((n_rows + 3) / 4), dim3(256), 0, st, (const float*)E, suffix, S, n_rows, d, vocab, x);
  else
    hipLaunchKernelGGL(embed_kernel<bf16_t>, dim3((n_rows + 3) / 4), dim3(256), 0, st, (const bf16_t*)E, suffix, S, n_rows, d, vocab, x);
  return hipGetLastError();
}

// ---------------------------------------------------------------- RMSNorm
// One wavefront per row.  Rows of up to 8 x 256 values stay in registers between the sum of
// squares and the scaling (one read of x); the output is written 4 values per lane per store.
template <typename TO>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const float* __restrict__ x, int64_t ldx,
                                                      const float* __restrict__ g, int n_rows, int d, float eps,
                                                      TO* __restrict__ y, int64_t ldy) {
  int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  int lane = threadIdx.x & 63;
  if (row >= n_rows) return;
  const float* xr = x + (int64_t)row * ldx;
  TO* yr = y + (int64_t)row * ldy;
  constexpr int KEEP = 8;                     // 16-byte pieces per lane kept in registers
  f32x4 keep[KEEP], gain[KEEP];               // (the gains come with the row: one latency, not two)
  float ss = 0.f;
#pragma unroll
  for (int it = 0; it < KEEP; it++) {
    const int c = lane * 4 + 256 * it;
    if (c < d) {
      keep[it] = *reinterpret_cast<const f32x4*>(xr + c);
      gain[it] = *reinterpret_cast<const f32x4*>(g + c);
    }
  }
#pragma unroll
  for (int it = 0; it < KEEP; it++) {
    const int c = lane * 4 + 256 * it;
    if (c < d) {
      const f32x4 v = keep[it];
      ss += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
    }
  }
  for (int c = lane * 4 + 256 * KEEP; c < d; c += 256) {
    f32x4 v = *reinterpret_cast<const f32x4*>(xr + c);
    ss += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
  }
  ss = wave_sum(ss);
  float inv = 1.0f / sqrtf(ss / (float)d + eps);
  auto put = [&](int c, const f32x4& v, const f32x4& gg) {
    if constexpr (sizeof(TO) == 2) {
      u32x2 pk;
      pk[0] = pack_bf16x2(v[0] * inv * gg[0], v[1] * inv * gg[1]);
      pk[1] = pack_bf16x2(v[2] * inv * gg[2], v[3] * inv * gg[3]);
      *reinterpret_cast<u32x2*>(yr + c) = pk;
    } else {
      *reinterpret_cast<f32x4*>(yr + c) =
          f32x4{v[0] * inv * gg[0], v[1] * inv * gg[1], v[2] * inv * gg[2], v[3] * inv * gg[3]};
    }
  };
#pragma unroll
  for (int it = 0; it < KEEP; it++) {
    const int c = lane * 4 + 256 * it;
    if (c < d) put(c, keep[it], gain[it]);
  }
  for (int c = lane * 4 + 256 * KEEP; c < d; c += 256)
    put(c, *reinterpret_cast<const f32x4*>(xr + c), *reinterpret_cast<const f32x4*>(g + c));
}

hipError_t rmsnorm_rows(int dt, const float* x, int64_t ldx, const float* g, int n_rows, int d, float eps, void* y,
                        int64_t ldy, hipStream_t st) {
  if (n_rows <= 0) return hipSuccess;
  if (d % 4 || ldx % 4 || ldy % 4) return hipErrorInvalidValue;   // 16- and 8-byte row accesses
  dim3 grid((n_rows + 3) / 4);
  if (dt == DT_F32)
    hipLaunchKernelGGL(rmsnorm_kernel<float>, grid, dim3(256), 0, st, x, ldx, g, n_rows, d, eps, (float*)y, ldy);
  else
    hipLaunchKernelGGL(rmsnorm_kernel<bf16_t>, grid, dim3(256), 0, st, x, ldx, g, n_rows, d, eps, (bf16_t*)y, ldy);
  return hipGetLastError();
}

// ---------------------------------------------------------------- rotary embedding
// thread per (row, head, 8 consecutive pairs i..i+7): (x_i, x_{i+D/2}) ->
// (x_i c - x_{i+D/2} s, x_{i+D/2} c + x_i s), 16- or 32-byte accesses (D/2 a multiple of 8)
template <typename T>
__global__ __launch_bounds__(256) void rope_kernel(T* __restrict__ qkv, int64_t ld, int n_rows, int n_heads, int H,
                                                   int D, const int32_t* __restrict__ pos,
                                                   const float* __restrict__ cos_t, const float* __restrict__ sin_t,
                                                   T* __restrict__ q_alt, const int32_t* __restrict__ shift, int step) {
  const int half = D / 2, groups = half / 8;
  const int per_row = n_heads * groups;
  const int gid = blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= per_row * n_rows) return;
  const int row = gid / per_row, rem = gid - row * per_row;
  const int head = rem / groups, i = (rem - head * groups) * 8;
  T* v = qkv + (int64_t)row * ld + head * D;
  float x1[8], x2[8], c[8], s[8], y1[8], y2[8];
  Vec8<T>::load(v + i, x1);
  Vec8<T>::load(v + i + half, x2);
  const int p = pos[(int64_t)row * step];
  Vec8<float>::load(cos_t + (int64_t)p * half + i, c);
  Vec8<float>::load(sin_t + (int64_t)p * half + i, s);
  if (q_alt && head < H && shift[(int64_t)row * step] >= 0) {
    const int p2 = p - shift[(int64_t)row * step];
    float c2[8], s2[8];
    Vec8<float>::load(cos_t + (int64_t)p2 * half + i, c2);
    Vec8<float>::load(sin_t + (int64_t)p2 * half + i, s2);
#pragma unroll
    for (int e = 0; e < 8; e++) rope_pair(x1[e], x2[e], c2[e], s2[e], y1[e], y2[e]);
    T* va = q_alt + (int64_t)row * ld + head * D;
    Vec8<T>::store(va + i, y1);
    Vec8<T>::store(va + i + half, y2);
  }
#pragma unroll
  for (int e = 0; e < 8; e++) rope_pair(x1[e], x2[e], c[e], s[e], y1[e], y2[e]);
  Vec8<T>::store(v + i, y1);
  Vec8<T>::store(v + i + half, y2);
}

hipError_t rope_qk(int dt, void* qkv, int64_t ld, int n_rows, int H, int Hkv, int D, const int32_t* pos,
                   const float* cos_tab, const float* sin_tab, void* q_alt, const int32_t* alt_shift,
                   hipStream_t st, int step) {
  if (n_rows <= 0) return hipSuccess;
  if ((D / 2) % 8 || ld % 8) return hipErrorInvalidValue;
  const int64_t total = (int64_t)n_rows * (H + Hkv) * (D / 16);
  if (total > 0x7fffffff) return hipErrorInvalidValue;
  dim3 grid((unsigned)((total + 255) / 256));
  if (dt == DT_F32)
    hipLaunchKernelGGL(rope_kernel<float>, grid, dim3(256), 0, st, (float*)qkv, ld, n_rows, H + Hkv, H, D, pos, cos_tab,
                       sin_tab, (float*)q_alt, alt_shift, step);
  else
    hipLaunchKernelGGL(rope_kernel<bf16_t>, grid, dim3(256), 0, st, (bf16_t*)qkv, ld, n_rows, H + Hkv, H, D, pos,
                       cos_tab, sin_tab, (bf16_t*)q_alt, alt_shift, step);
  return hipGetLastError();
}

// Rows of a batch that repeat every src_rows rows before the rotation (every item's rows are
// the same suffix at layer 0): each row is copied from its source row r mod src_rows, the
// query and key heads (columns below rot_cols) rotated at the row's own position with the
// arithmetic of the projection's rotary epilogue (BF16) or of rope_kernel (FP32), so the rows
// equal what those write bit for bit; joins also get the queries rotated at position - shift into q_alt.
template <typename T>
__global__ __launch_bounds__(256) void rope_broadcast_kernel(const T* __restrict__ src, int src_rows,
                                                             T* __restrict__ dst, int64_t ld, int n_rows,
                                                             int n_cols, int rot_cols, int q_cols, int D,
                                                             const int32_t* __restrict__ pos,
                                                             const float* __restrict__ cos_t,
                                                             const float* __restrict__ sin_t, T* __restrict__ q_alt,
                                                             const int32_t* __restrict__ shift) {
  const int half = D / 2, gph = half / 8;
  const int per_row = (n_cols / D) * gph;
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (gid >= (int64_t)per_row * n_rows) return;
  const int row = (int)(gid / per_row), rem = (int)(gid - (int64_t)row * per_row);
  const int hh = rem / gph, i = (rem - hh * gph) * 8, col = hh * D + i;
  const T* sp = src + (int64_t)(row % src_rows) * ld + col;
  T* o = dst + (int64_t)row * ld + col;
  if (col >= rot_cols) {
    constexpr int NV = 8 * (int)sizeof(T) / 16;
#pragma unroll
    for (int q = 0; q < NV; q++) {
      reinterpret_cast<u32x4*>(o)[q] = reinterpret_cast<const u32x4*>(sp)[q];
      reinterpret_cast<u32x4*>(o + half)[q] = reinterpret_cast<const u32x4*>(sp + half)[q];
    }
    return;
  }
  float x1[8], x2[8];
  Vec8<T>::load(sp, x1);
  Vec8<T>::load(sp + half, x2);
  auto rotate_store = [&](int p, T* d) {
    float c[8], s[8], y1[8], y2[8];
    Vec8<float>::load(cos_t + (int64_t)p * half + i, c);
    Vec8<float>::load(sin_t + (int64_t)p * half + i, s);
#pragma unroll
    for (int e = 0; e < 8; e++) rope_pair(x1[e], x2[e], c[e], s[e], y1[e], y2[e]);
    Vec8<T>::store(d, y1);
    Vec8<T>::store(d + half, y2);
  };
  const int p = pos[row];
  if (q_alt && col < q_cols && shift[row] >= 0) rotate_store(p - shift[row], q_alt + (int64_t)row * ld + col);
  rotate_store(p, o);
}

hipError_t rope_broadcast(int dt, const void* src, int src_rows, void* dst, int64_t ld, int n_rows, int n_cols, int rot_cols,
                          int q_cols, int D, const int32_t* pos, const float* cos_tab, const float* sin_tab, void* q_alt,
                          const int32_t* shift, hipStream_t st) {
  if (n_rows <= 0) return hipSuccess;
  if (src_rows < 1 || D % 16 || n_cols % D || ld % 8 || (q_alt && !shift)) return hipErrorInvalidValue;
  const int64_t total = (int64_t)n_rows * (n_cols / D) * (D / 16);
  const dim3 grid((unsigned)((total + 255) / 256));
  if (dt == DT_F32)
    hipLaunchKernelGGL(rope_broadcast_kernel<float>, grid, dim3(256), 0, st, (const float*)src, src_rows, (float*)dst, ld,
                       n_rows, n_cols, rot_cols, q_cols, D, pos, cos_tab, sin_tab, (float*)q_alt, shift);
  else
    hipLaunchKernelGGL(rope_broadcast_kernel<bf16_t>, grid, dim3(256), 0, st, (const bf16_t*)src, src_rows, (bf16_t*)dst,
                       ld, n_rows, n_cols, rot_cols, q_cols, D, pos, cos_tab, sin_tab, (bf16_t*)q_alt, shift);
  return hipGetLastError();
}

// ---------------------------------------------------------------- cache writer (prefill)
// One workgroup per (16-row block of a document, kv head): rotate k of the block's rows
// at their positions, then store k and v into the document's region.  FP8 caches get one
// scale per block and per K/V: amax / 448 (1 for an all-zero block), codes = E4M3(x/scale).
template <typename T, typename TKV>
__global__ __launch_bounds__(256) void write_kv_kernel(const T* __restrict__ qkv, int64_t ld,
                                                       const KvBlock* __restrict__ blocks, int H, int Hkv, int D,
                                                       int layer, int n_layers, const float* __restrict__ cos_t,
                                                       const float* __restrict__ sin_t, uint8_t* __restrict__ pool) {
  __shared__ float kv_s[2][16][128 + 1];
  __shared__ float red[2][4];
  const KvBlock b = blocks[blockIdx.x];
  const int h = blockIdx.y, half = D / 2;
  const int nrow = min(16, b.L - b.p0);
  const int kcol = H * D + h * D, vcol = (H + Hkv) * D + h * D;
  float amax_k = 0.f, amax_v = 0.f;
  for (int e = threadIdx.x; e < 16 * half; e += 256) {
    int r = e / half, i = e % half;
    float k1 = 0.f, k2 = 0.f, v1 = 0.f, v2 = 0.f;
    if (r < nrow) {
      const T* row = qkv + (int64_t)(b.row0 + r) * ld;
      float x1 = to_f32(row[kcol + i]), x2 = to_f32(row[kcol + i + half]);
      int p = b.p0 + r;
      float c = cos_t[(int64_t)p * half + i], s = sin_t[(int64_t)p * half + i];
      rope_pair(x1, x2, c, s, k1, k2);
      v1 = to_f32(row[vcol + i]);
      v2 = to_f32(row[vcol + i + half]);
    }
    kv_s[0][r][i] = k1; kv_s[0][r][i + half] = k2;
    kv_s[1][r][i] = v1; kv_s[1][r][i + half] = v2;
    amax_k = fmaxf(amax_k, fmaxf(fabsf(k1), fabsf(k2)));
    amax_v = fmaxf(amax_v, fmaxf(fabsf(v1), fabsf(v2)));
  }
  float sc_k = 1.f, sc_v = 1.f;
  if constexpr (sizeof(TKV) == 1) {
    amax_k = wave_max(amax_k);
    amax_v = wave_max(amax_v);
    if ((threadIdx.x & 63) == 0) { red[0][threadIdx.x >> 6] = amax_k; red[1][threadIdx.x >> 6] = amax_v; }
  }
  __syncthreads();
  if constexpr (sizeof(TKV) == 1) {
    float ak = fmaxf(fmaxf(red[0][0], red[0][1]), fmaxf(red[0][2], red[0][3]));
    float av = fmaxf(fmaxf(red[1][0], red[1][1]), fmaxf(red[1][2], red[1][3]));
    sc_k = ak == 0.f ? 1.f : ak / 448.0f;
    sc_v = av == 0.f ? 1.f : av / 448.0f;
  }
  const int64_t kv_elems = (int64_t)b.L * D;
  uint8_t* base = pool + b.off;
  TKV* kdst = reinterpret_cast<TKV*>(base) + ((int64_t)(layer * Hkv + h) * 2) * kv_elems;
  TKV* vdst = kdst + kv_elems;
  for (int e = threadIdx.x; e < nrow * D; e += 256) {
    int r = e / D, c = e % D;
    float kx = kv_s[0][r][c], vx = kv_s[1][r][c];
    int64_t o = (int64_t)(b.p0 + r) * D + c;
    if constexpr (sizeof(TKV) == 1) {
      kdst[o] = (fp8_t)f32_to_e4m3(kx / sc_k);
      vdst[o] = (fp8_t)f32_to_e4m3(vx / sc_v);
    } else {
      kdst[o] = from_f32<TKV>(kx);
      vdst[o] = from_f32<TKV>(vx);
    }
  }
  if constexpr (sizeof(TKV) == 1) {
    if (threadIdx.x == 0) {
      int nblk = (b.L + 15) >> 4;
      float* sb = reinterpret_cast<float*>(base + (int64_t)2 * n_layers * Hkv * kv_elems);
      float* ks = sb + ((int64_t)(layer * Hkv + h) * 2) * nblk;
      ks[b.p0 >> 4] = sc_k;
      ks[nblk + (b.p0 >> 4)] = sc_v;
    }
  }
}

hipError_t rope_write_kv(int dt, int kvdt, void* qkv, int64_t ld, const KvBlock* blocks, int n_blocks, int H,
                         int Hkv, int D, int layer, int n_layers, const float* cos_tab, const float* sin_tab,
                         uint8_t* pool, hipStream_t st) {
  if (n_blocks <= 0) return hipSuccess;
  if (D > 128) return hipErrorInvalidValue;
  dim3 grid(n_blocks, Hkv);
  if (dt == DT_F32) {
    if (kvdt != DT_F32) return hipErrorInvalidValue;
    hipLaunchKernelGGL((write_kv_kernel<float, float>), grid, dim3(256), 0, st, (const float*)qkv, ld, blocks, H, Hkv, D,
                       layer, n_layers, cos_tab, sin_tab, pool);
  } else if (kvdt == DT_BF16) {
    hipLaunchKernelGGL((write_kv_kernel<bf16_t, bf16_t>), grid, dim3(256), 0, st, (const bf16_t*)qkv, ld, blocks, H,
                       Hkv, D, layer, n_layers, cos_tab, sin_tab, pool);
  } else if (kvdt == DT_FP8) {
    hipLaunchKernelGGL((write_kv_kernel<bf16_t, fp8_t>), grid, dim3(256), 0, st, (const bf16_t*)qkv, ld, blocks, H, Hkv,
                       D, layer, n_layers, cos_tab, sin_tab, pool);
  } else {
    return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------- row copy (decode bookkeeping)
template <typename T>
__global__ void copy_rows_kernel(const T* __restrict__ src, int64_t ld, int col0, int n_cols,
                                 const int32_t* __restrict__ srow, const int32_t* __restrict__ drow, int n,
                                 T* __restrict__ dst, int64_t ldd) {
  int i = blockIdx.x;
  if (i >= n) return;
  const T* s = src + (int64_t)srow[i] * ld + col0;
  T* d = dst + (int64_t)drow[i] * ldd;
  for (int c = threadIdx.x; c < n_cols; c += blockDim.x) d[c] = s[c];
}

hipError_t copy_kv_rows(int dt, const void* qkv, int64_t ld, int kcol, int n_cols, const int32_t* src_rows,
                        const int32_t* dst_rows, int n, void* dst, int64_t ldd, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  if (dt == DT_F32)
    hipLaunchKernelGGL(copy_rows_kernel<float>, dim3(n), dim3(256), 0, st, (const float*)qkv, ld, kcol, n_cols, src_rows,
                       dst_rows, n, (float*)dst, ldd);
  else
    hipLaunchKernelGGL(copy_rows_kernel<bf16_t>, dim3(n), dim3(256), 0, st, (const bf16_t*)qkv, ld, kcol, n_cols,
                       src_rows, dst_rows, n, (bf16_t*)dst, ldd);
  return hipGetLastError();
}

// ---------------------------------------------------------------- pooled features
// Mean over a document's rows of x * inv_rms(x) * g.  Bound by reading x once (8 KiB a row): a
// workgroup takes up to 64 rows of one document, a wavefront a row at a time, whose 2048 values
// stay in registers between the sum of squares and the column sums; the four wavefronts' sums
// meet in LDS.  Documents of one chunk are finished there, the others' partial sums by a second
// launch, in chunk order.  (One thread per document and column walking all rows, with the inverse
// RMS from a pass of its own, took 1606 us for 63 000 rows in 81 documents, the longest document's
// chain of loads; now 118 us, 4.4 TB/s.)  More than 2048 columns: one workgroup per 2048, each
// summing the whole row's squares.
constexpr int kPoolCols = 2048;
__global__ __launch_bounds__(256) void pooled_chunk_kernel(const float* __restrict__ x, int d,
                                                           const PoolChunk* __restrict__ chunks, float eps,
                                                           const float* __restrict__ g, float* __restrict__ part,
                                                           float* __restrict__ pooled) {
  __shared__ __attribute__((aligned(16))) float sum[4][kPoolCols];
  constexpr int KEEP = kPoolCols / 256;
  const PoolChunk ch = chunks[blockIdx.x];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c0 = blockIdx.y * kPoolCols;
  f32x4 acc[KEEP];
#pragma unroll
  for (int it = 0; it < KEEP; it++) acc[it] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto load = [&](int r, f32x4 (&v)[KEEP]) {
    const float* xr = x + (int64_t)(ch.row0 + r) * d + c0;
#pragma unroll
    for (int it = 0; it < KEEP; it++) {
      const int c = lane * 4 + 256 * it;
      v[it] = c0 + c < d ? *reinterpret_cast<const f32x4*>(xr + c) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  };
  f32x4 next[KEEP];
  if (wave < ch.n) load(wave, next);
  for (int r = wave; r < ch.n; r += 4) {
    f32x4 v[KEEP];
    float ss = 0.f;
#pragma unroll
    for (int it = 0; it < KEEP; it++) {
      v[it] = next[it];
      ss += v[it][0] * v[it][0] + v[it][1] * v[it][1] + v[it][2] * v[it][2] + v[it][3] * v[it][3];
    }
    if (r + 4 < ch.n) load(r + 4, next);
    if (d > kPoolCols) {
      const float* xr = x + (int64_t)(ch.row0 + r) * d;
      for (int c = lane * 4; c < d; c += 256) {
        if (c >= c0 && c < c0 + kPoolCols) continue;
        const f32x4 o = *reinterpret_cast<const f32x4*>(xr + c);
        ss += o[0] * o[0] + o[1] * o[1] + o[2] * o[2] + o[3] * o[3];
      }
    }
    const float inv = 1.0f / sqrtf(wave_sum(ss) / (float)d + eps);
#pragma unroll
    for (int it = 0; it < KEEP; it++)
#pragma unroll
      for (int q = 0; q < 4; q++) acc[it][q] = fmaf(v[it][q], inv, acc[it][q]);
  }
#pragma unroll
  for (int it = 0; it < KEEP; it++) *reinterpret_cast<f32x4*>(&sum[wave][lane * 4 + 256 * it]) = acc[it];
  __syncthreads();
  for (int c = threadIdx.x; c < kPoolCols && c0 + c < d; c += 256) {
    const float s = (sum[0][c] + sum[1][c]) + (sum[2][c] + sum[3][c]);
    if (ch.slot < 0) pooled[(int64_t)ch.doc * d + c0 + c] = s * g[c0 + c] / (float)ch.n;
    else part[(int64_t)ch.slot * d + c0 + c] = s;
  }
}

// documents of several chunks: slots slot .. slot + n - 1, L rows
__global__ __launch_bounds__(256) void pooled_finish_kernel(const float* __restrict__ part, int d,
                                                            const PoolDoc* __restrict__ docs,
                                                            const float* __restrict__ g, float* __restrict__ pooled) {
  const PoolDoc w = docs[blockIdx.x];
  const int c = blockIdx.y * 256 + threadIdx.x;
  if (c >= d) return;
  float s = 0.f;
#pragma unroll 8
  for (int q = 0; q < w.n; q++) s += part[(int64_t)(w.slot + q) * d + c];
  pooled[(int64_t)w.doc * d + c] = s * g[c] / (float)w.L;
}

hipError_t pooled_mean(const float* x, int d, const PoolChunk* chunks, int n_chunks, const PoolDoc* docs, int n_docs,
                       const float* g, float eps, float* part, float* pooled, hipStream_t st) {
  if (n_chunks <= 0) return hipSuccess;
  if (d % 4) return hipErrorInvalidValue;
  hipLaunchKernelGGL(pooled_chunk_kernel, dim3(n_chunks, (d + kPoolCols - 1) / kPoolCols), dim3(256), 0, st, x, d,
                     chunks, eps, g, part, pooled);
  if (n_docs > 0)
    hipLaunchKernelGGL(pooled_finish_kernel, dim3(n_docs, (d + 255) / 256), dim3(256), 0, st, (const float*)part, d,
                       docs, g, pooled);
  return hipGetLastError();
}

// ---------------------------------------------------------------- logit heads
// one workgroup per item: y = rmsnorm(x_row) * g kept in LDS (FP32), then dot products with
// the requested head rows, reduced in FP32
template <typename T>
__global__ __launch_bounds__(256) void head_filter_kernel(const float* __restrict__ x, int64_t ldx, int d,
                                                          const float* __restrict__ g, float eps,
                                                          const T* __restrict__ W, int yes_id, int no_id, float thp,
                                                          float thn, const int32_t* __restrict__ in_rows,
                                                          const int32_t* __restrict__ out_rows,
                                                          float* __restrict__ logits, int8_t* __restrict__ decision) {
  __shared__ float red[3][4];
  int item = blockIdx.x;
  const float* xr = x + (int64_t)(in_rows ? in_rows[item] : item) * ldx;
  int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  float ss = 0.f;
  for (int c = threadIdx.x; c < d; c += 256) ss += xr[c] * xr[c];
  ss = wave_sum(ss);
  if (lane == 0) red[0][wv] = ss;
  __syncthreads();
  float tot = red[0][0] + red[0][1] + red[0][2] + red[0][3];
  float inv = 1.0f / sqrtf(tot / (float)d + eps);
  const T* wy = W + (int64_t)yes_id * d;
  const T* wn = W + (int64_t)no_id * d;
  float ay = 0.f, an = 0.f;
  for (int c = threadIdx.x; c < d; c += 256) {
    float y = xr[c] * inv * g[c];
    ay += y * to_f32(wy[c]);
    an += y * to_f32(wn[c]);
  }
  ay = wave_sum(ay);
  an = wave_sum(an);
  if (lane == 0) { red[1][wv] = ay; red[2][wv] = an; }
  __syncthreads();
  if (threadIdx.x == 0) {
    float ly = red[1][0] + red[1][1] + red[1][2] + red[1][3];
    float ln = red[2][0] + red[2][1] + red[2][2] + red[2][3];
    const int64_t o = out_rows[item];
    logits[2 * o] = ly;
    logits[2 * o + 1] = ln;
    float lo = ly - ln;
    if (decision) decision[o] = lo > thp ? 1 : (lo < thn ? 0 : -1);
  }
}

hipError_t head_filter(int dt, const float* x, int64_t ldx, int n_items, int d, const float* g, float eps,
                       const void* head, int yes_id, int no_id, float th_pos, float th_neg, const int32_t* in_rows,
                       const int32_t* out_rows, float* logits, int8_t* decision, hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
  if (dt == DT_F32)
    hipLaunchKernelGGL(head_filter_kernel<float>, dim3(n_items), dim3(256), 0, st, x, ldx, d, g, eps,
                       (const float*)head, yes_id, no_id, th_pos, th_neg, in_rows, out_rows, logits, decision);
  else
    hipLaunchKernelGGL(head_filter_kernel<bf16_t>, dim3(n_items), dim3(256), 0, st, x, ldx, d, g, eps,
                       (const bf16_t*)head, yes_id, no_id, th_pos, th_neg, in_rows, out_rows, logits, decision);
  return hipGetLastError();
}

// Label logits of IT items x 32 labels per workgroup, then each item's argmax in a second launch.  A
// (item, label) product is summed as before, eight values per lane and 512-value step and then
// across the wavefront, but a head row is read from L2 once for IT items instead of once per
// item, and the labels spread over eight workgroups: one workgroup per item walked all 256 rows
// (1 MiB from L2 an item; 109 us for 192 items, now 16 + 4).
template <typename T, int IT>
__global__ __launch_bounds__(256) void head_map_kernel(const float* __restrict__ x, int64_t ldx, int n_items, int d,
                                                       const float* __restrict__ g, float eps, const T* __restrict__ W,
                                                       int lo, int n, const int32_t* __restrict__ in_rows,
                                                       const int32_t* __restrict__ out_rows,
                                                       float* __restrict__ logits, int64_t ldl) {
  extern __shared__ __attribute__((aligned(16))) float ysm[];   // IT x d
  __shared__ float red[IT][4];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int i0 = blockIdx.x * IT;
  const float* xr[IT];
  float ss[IT];
#pragma unroll
  for (int i = 0; i < IT; i++) {
    const int item = min(i0 + i, n_items - 1);
    xr[i] = x + (int64_t)(in_rows ? in_rows[item] : item) * ldx;
    ss[i] = 0.f;
  }
  for (int c = threadIdx.x; c < d; c += 256)
#pragma unroll
    for (int i = 0; i < IT; i++) {
      const float v = xr[i][c];
      ysm[i * d + c] = v;
      ss[i] += v * v;
    }
#pragma unroll
  for (int i = 0; i < IT; i++) {
    ss[i] = wave_sum(ss[i]);
    if (lane == 0) red[i][wv] = ss[i];
  }
  __syncthreads();
  float inv[IT];
#pragma unroll
  for (int i = 0; i < IT; i++)
    inv[i] = 1.0f / sqrtf((red[i][0] + red[i][1] + red[i][2] + red[i][3]) / (float)d + eps);
  for (int c = threadIdx.x; c < d; c += 256) {
    const float gc = g[c];
#pragma unroll
    for (int i = 0; i < IT; i++) ysm[i * d + c] = ysm[i * d + c] * inv[i] * gc;
  }
  __syncthreads();
#pragma unroll 1
  for (int hf = 0; hf < 2; hf++) {
    const int j0 = blockIdx.y * 32 + 16 * hf + 4 * wv;
    if (j0 >= n) break;
    float a[IT][4];
#pragma unroll
    for (int i = 0; i < IT; i++)
#pragma unroll
      for (int q = 0; q < 4; q++) a[i][q] = 0.f;
    for (int c = 8 * lane; c < d; c += 512) {
      float wvv[4][8];
#pragma unroll
      for (int q = 0; q < 4; q++) Vec8<T>::load(W + (int64_t)(lo + min(j0 + q, n - 1)) * d + c, wvv[q]);
#pragma unroll
      for (int i = 0; i < IT; i++) {
        const f32x4 y0 = *reinterpret_cast<const f32x4*>(ysm + i * d + c);
        const f32x4 y1 = *reinterpret_cast<const f32x4*>(ysm + i * d + c + 4);
#pragma unroll
        for (int q = 0; q < 4; q++) {
#pragma unroll
          for (int t = 0; t < 4; t++) a[i][q] = fmaf(y0[t], wvv[q][t], a[i][q]);
#pragma unroll
          for (int t = 0; t < 4; t++) a[i][q] = fmaf(y1[t], wvv[q][4 + t], a[i][q]);
        }
      }
    }
    float mine = 0.f;                                  // lane 4 i + q keeps the sum of (item i, label j0 + q)
#pragma unroll
    for (int i = 0; i < IT; i++)
#pragma unroll
      for (int q = 0; q < 4; q++) {
        const float v = wave_sum(a[i][q]);
        if (lane == 4 * i + q) mine = v;
      }
    const int item = i0 + lane / 4, j = j0 + lane % 4;
    if (lane < 4 * IT && item < n_items && j < n) logits[(int64_t)out_rows[item] * ldl + j] = mine;
  }
}

// argmax over an item's n logits, lowest index on ties: one wavefront per item
__global__ __launch_bounds__(256) void head_argmax_kernel(const float* __restrict__ logits, int64_t ldl, int n_items,
                                                          int lo, int n, const int32_t* __restrict__ out_rows,
                                                          int32_t* __restrict__ tok_out, int64_t ldt,
                                                          int32_t* __restrict__ next_tok, bool next_by_out) {
  const int item = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (item >= n_items) return;
  const int64_t orow = out_rows[item];
  float best = -INFINITY;
  int bi = 0x7fffffff;
#pragma unroll 4
  for (int j = lane; j < n; j += 64) {
    const float v = logits[orow * ldl + j];
    if (v > best || (v == best && j < bi)) { best = v; bi = j; }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ob = __shfl_xor(best, o, 64);
    const int oi = __shfl_xor(bi, o, 64);
    if (ob > best || (ob == best && oi < bi)) { best = ob; bi = oi; }
  }
  if (lane == 0) {
    tok_out[orow * ldt] = lo + bi;
    if (next_tok) next_tok[next_by_out ? orow : item] = lo + bi;
  }
}

template <typename T, int IT>
static hipError_t launch_head_map(const float* x, int64_t ldx, int n_items, int d, const float* g, float eps,
                                  const T* head, int lo, int n, const int32_t* in_rows, const int32_t* out_rows,
                                  float* logits, int64_t ldl, hipStream_t st) {
  static const hipError_t attr = hipFuncSetAttribute((const void*)head_map_kernel<T, IT>,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, 150 << 10);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((head_map_kernel<T, IT>), dim3((n_items + IT - 1) / IT, (n + 31) / 32), dim3(256),
                     (size_t)IT * d * sizeof(float), st, x, ldx, n_items, d, g, eps, head, lo, n, in_rows, out_rows,
                     logits, ldl);
  return hipGetLastError();
}

template <typename T>
static hipError_t head_map_t(const float* x, int64_t ldx, int n_items, int d, const float* g, float eps, const T* head,
                             int lo, int n, const int32_t* in_rows, const int32_t* out_rows, float* logits, int64_t ldl,
                             hipStream_t st) {
  // two items while their rows fit 64 KiB of LDS, else one.  More items a workgroup read the head
  // less often from L2 but leave CUs idle and make each one's chain longer: 192 items of 2048
  // columns 16 us with two, 20 with four, 27 with eight; two is also the fastest at 1 and at 2048.
  if (d <= 8192) return launch_head_map<T, 2>(x, ldx, n_items, d, g, eps, head, lo, n, in_rows, out_rows, logits, ldl, st);
  return launch_head_map<T, 1>(x, ldx, n_items, d, g, eps, head, lo, n, in_rows, out_rows, logits, ldl, st);
}

hipError_t head_map(int dt, const float* x, int64_t ldx, int n_items, int d, const float* g, float eps,
                    const void* head, int lo, int n, const int32_t* in_rows, const int32_t* out_rows, float* logits,
                    int64_t ld_logits, int32_t* tok_out, int64_t ld_tok, int32_t* next_tok, bool next_by_out,
                    hipStream_t st) {
  if (n_items <= 0) return hipSuccess;
  if (d % 8) return hipErrorInvalidValue;     // eight-value row pieces
  const hipError_t e =
      dt == DT_F32 ? head_map_t<float>(x, ldx, n_items, d, g, eps, (const float*)head, lo, n, in_rows, out_rows, logits,
                                       ld_logits, st)
                   : head_map_t<bf16_t>(x, ldx, n_items, d, g, eps, (const bf16_t*)head, lo, n, in_rows, out_rows,
                                        logits, ld_logits, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(head_argmax_kernel, dim3((n_items + 3) / 4), dim3(256), 0, st, (const float*)logits, ld_logits,
                     n_items, lo, n, out_rows, tok_out, ld_tok, next_tok, next_by_out);
  return hipGetLastError();
}

// ---------------------------------------------------------------- validation
// A workgroup or (WAVES = 1) a wavefront per list, four pairs of neighbours per lane in flight: with
// one pair at a time a wavefront waited for memory 64 times for a list of 4096 rows (25 us for 1024
// lists of up to that).  A workgroup per list ends a long one sooner, a wavefront per list starts
// many short ones sooner (1.2 M workgroups/ms): us with workgroups and wavefronts 4.8 and 8.9 for
// 1024 lists of up to 4096 rows, 7.8 and 11.1 for 4096, 13 and 14 for 8000, 23 and 20 for 16 000;
// 5.0 and 4.9 for 2000 of 1024; 3.1 and 2.6 for 1000 of 256, 12.8 and 4.9 for 12 000; 25.6 and 8.5
// for 30 000 of 4.
template <int WAVES>
__global__ __launch_bounds__(256) void validate_kernel(const int32_t* __restrict__ idx,
                                                       const ListCheck* __restrict__ lists, int n_lists,
                                                       int* __restrict__ bad) {
  constexpr int T = 64 * WAVES;
  const int li = blockIdx.x * (4 / WAVES) + (int)threadIdx.x / T, t = threadIdx.x % T;
  if (li >= n_lists) return;   // whole wavefronts, and for WAVES = 4 no workgroup
  const ListCheck l = lists[li];
  int wrong = 0;
  for (int i0 = t; i0 < l.n; i0 += 4 * T) {
    int v[4], before[4];
#pragma unroll
    for (int u = 0; u < 4; u++) {
      const int i = min(i0 + T * u, l.n - 1);
      v[u] = idx[l.off + i];
      before[u] = i > 0 ? idx[l.off + i - 1] : -1;
    }
#pragma unroll
    for (int u = 0; u < 4; u++)
      if (v[u] < 0 || v[u] >= l.L || before[u] >= v[u]) wrong = 1;
  }
  if constexpr (WAVES == 4) wrong = __syncthreads_or(wrong);
  else wrong = __any(wrong);
  if (t == 0 && wrong) atomicAdd(bad, 1);
}

hipError_t validate_lists(const int32_t* idx, const ListCheck* lists, int n_lists, int longest, int* bad,
                          hipStream_t st) {
  if (n_lists <= 0) return hipSuccess;
  if (n_lists > 2 * longest)
    hipLaunchKernelGGL(validate_kernel<1>, dim3((n_lists + 3) / 4), dim3(256), 0, st, idx, lists, n_lists, bad);
  else
    hipLaunchKernelGGL(validate_kernel<4>, dim3(n_lists), dim3(256), 0, st, idx, lists, n_lists, bad);
  return hipGetLastError();
}

// Token ids outside [0, vocab): one count per wavefront that saw any.
__global__ __launch_bounds__(256) void validate_tokens_kernel(const int32_t* __restrict__ tok, int64_t n, int vocab,
                                                              int* __restrict__ bad) {
  int ok = 1;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    int t = tok[i];
    if (t < 0 || t >= vocab) ok = 0;
  }
  ok = __all(ok);
  if ((threadIdx.x & 63) == 0 && !ok) atomicAdd(bad, 1);
}

hipError_t validate_tokens(const int32_t* tok, int64_t n, int vocab, int* bad, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = std::min<int64_t>((n + 255) / 256, 4096);
  hipLaunchKernelGGL(validate_tokens_kernel, dim3((unsigned)blocks), dim3(256), 0, st, tok, n, vocab, bad);
  return hipGetLastError();
}

// ---------------------------------------------------------------- weights
template <typename T>
__global__ void convert_kernel(const float* __restrict__ src, const float* __restrict__ src2, int64_t rows,
                               int64_t cols, T* __restrict__ dst, int inter) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t out_rows = inter ? 2 * rows : rows;
  if (i >= out_rows * cols) return;
  int64_t r = i / cols, c = i % cols;
  float v;
  if (inter) {
    int64_t blk = r / 32, e = r % 32;
    v = e < 16 ? src[(blk * 16 + e) * cols + c] : src2[(blk * 16 + e - 16) * cols + c];
  } else {
    v = src[i];
  }
  dst[i] = from_f32<T>(v);
}

hipError_t convert_weights(int dt, const float* src, const float* src2, int64_t rows, int64_t cols, void* dst,
                           int interleave16, hipStream_t st) {
  int64_t total = (interleave16 ? 2 * rows : rows) * cols;
  if (total <= 0) return hipSuccess;
  if (interleave16 && rows % 16) return hipErrorInvalidValue;
  dim3 grid((unsigned)((total + 255) / 256));
  if (dt == DT_F32)
    hipLaunchKernelGGL(convert_kernel<float>, grid, dim3(256), 0, st, src, src2, rows, cols, (float*)dst, interleave16);
  else
    hipLaunchKernelGGL(convert_kernel<bf16_t>, grid, dim3(256), 0, st, src, src2, rows, cols, (bf16_t*)dst, interleave16);
  return hipGetLastError();
}

template <typename TKV>
__global__ void read_cache_kernel(const uint8_t* __restrict__ region, int L, int D, int layer, int n_layers, int Hkv,
                                  int h, int kv, float* __restrict__ out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)L * D) return;
  const int64_t kv_elems = (int64_t)L * D;
  const TKV* src = reinterpret_cast<const TKV*>(region) + ((int64_t)(layer * Hkv + h) * 2 + kv) * kv_elems;
  if constexpr (sizeof(TKV) == 1) {
    int nblk = (L + 15) >> 4;
    const float* sb = reinterpret_cast<const float*>(region + (int64_t)2 * n_layers * Hkv * kv_elems);
    float sc = sb[((int64_t)(layer * Hkv + h) * 2 + kv) * nblk + (i / D) / 16];
    out[i] = e4m3_to_f32(src[i]) * sc;
  } else {
    out[i] = to_f32(src[i]);
  }
}

hipError_t read_cache(int kvdt, const uint8_t* region, int L, int D, int layer, int n_layers, int Hkv, int h, int kv,
                      float* out, hipStream_t st) {
  int64_t n = (int64_t)L * D;
  dim3 grid((unsigned)((n + 255) / 256));
  if (kvdt == DT_F32)
    hipLaunchKernelGGL(read_cache_kernel<float>, grid, dim3(256), 0, st, region, L, D, layer, n_layers, Hkv, h, kv, out);
  else if (kvdt == DT_BF16)
    hipLaunchKernelGGL(read_cache_kernel<bf16_t>, grid, dim3(256), 0, st, region, L, D, layer, n_layers, Hkv, h, kv, out);
  else
    hipLaunchKernelGGL(read_cache_kernel<fp8_t>, grid, dim3(256), 0, st, region, L, D, layer, n_layers, Hkv, h, kv, out);
  return hipGetLastError();
}

__global__ void fill_kernel(int32_t* p, int32_t v, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
hipError_t fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, v, n);
  return hipGetLastError();
}

}  // namespace kvop
