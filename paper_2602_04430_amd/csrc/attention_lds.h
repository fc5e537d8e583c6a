// What the attention kernels with direct global -> LDS loads share: explicit waits on the tiles in
// flight, loads that keep to the vector-memory counter, and a lane-group maximum.
#pragma once
#include "common.h"

namespace kvop {

typedef __attribute__((address_space(3))) void lds_void_t;

// BYTES from each lane's address to consecutive slots from l on (l: the same for the wavefront)
template <int BYTES, typename T> __device__ inline void load_to_lds(const T* g, void* l) {
#if defined(__HIP_DEVICE_COMPILE__)   // the host pass knows no 16-byte form
  __builtin_amdgcn_global_load_lds(g, (lds_void_t*)l, BYTES, 0, 0);
#endif
}

// Offsets within a key source are 32 bits.  A cached document has fewer than 65 536 rows of at most
// 512 bytes; an own row is as long as the projection's, and a suffix of such rows may pass 4 GiB, so
// its base moves on every kOwnRows rows.
constexpr int kOwnRows = 1024;

template <int N> __device__ inline void vm_wait() {
  static_assert(N >= 0 && N <= 63, "vmcnt range");
  // gfx9 s_waitcnt: vmcnt in bits 3:0 and 15:14, expcnt 6:4 (7: no wait), lgkmcnt 11:8 (15: no wait)
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// waits until only `behind` (0 .. MAXB, uniform) tiles of OPS operations and ROWS row-number loads
// are outstanding
template <int MAXB, int OPS, int ROWS> __device__ inline void vm_wait_behind(int behind) {
  if constexpr (MAXB < 0) {
    vm_wait<0>();
  } else {
    if (behind >= MAXB) vm_wait<MAXB * OPS + ROWS>();
    else vm_wait_behind<MAXB - 1, OPS, ROWS>(behind);
  }
}

// maximum over the four lanes l % 16 + {0, 16, 32, 48}: two register-to-register lane swaps (a
// shuffle through LDS would add its latency twice to every softmax step)
__device__ inline float max_over_groups(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const float m = fmaxf(__builtin_bit_cast(float, (uint32_t)a[0]), __builtin_bit_cast(float, (uint32_t)a[1]));
  const uint32_t v = __builtin_bit_cast(uint32_t, m);
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return fmaxf(__builtin_bit_cast(float, (uint32_t)b[0]), __builtin_bit_cast(float, (uint32_t)b[1]));
}

// m c - mc with the product rounded first
__device__ inline float scaled_minus(float m, float c, float mc) {
#pragma clang fp contract(off)
  return m * c - mc;
}

// plain global load (global_load, not flat: a flat load also counts in lgkmcnt)
template <typename T> __device__ inline T gload(const T* p) {
  return *reinterpret_cast<const __attribute__((address_space(1))) T*>(reinterpret_cast<uintptr_t>(p));
}

}  // namespace kvop
