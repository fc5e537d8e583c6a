// What the kernels with direct global -> LDS loads share: explicit waits on the loads in flight, loads
// that keep to the vector-memory counter, transposed LDS reads, and for attention the rounding of a
// scaled maximum, a lane-group maximum and the own rows' step.
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

// Transposed LDS reads as inline assembly, each block with its own wait.  (The builtin form makes
// the compiler wait for every direct-to-LDS load in flight (vmcnt(0)) before it, since it
// cannot tell which LDS bytes the read touches.)  The caller reads only stages whose
// loads have completed (by its own wait).
__device__ inline uint32_t lds_addr(const uint8_t* p) { return (uint32_t)reinterpret_cast<uintptr_t>(p); }
// y[2 i] from address ad[i], y[2 i + 1] from ad[i] + STEP
template <int STEP> __device__ inline void ds_read_tr16_x8(const uint32_t (&ad)[4], u32x2 (&y)[8]) {
  asm volatile(
      "ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %8 offset:%c12\n\t"
      "ds_read_b64_tr_b16 %2, %9\n\tds_read_b64_tr_b16 %3, %9 offset:%c12\n\t"
      "ds_read_b64_tr_b16 %4, %10\n\tds_read_b64_tr_b16 %5, %10 offset:%c12\n\t"
      "ds_read_b64_tr_b16 %6, %11\n\tds_read_b64_tr_b16 %7, %11 offset:%c12\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(y[0]), "=&v"(y[1]), "=&v"(y[2]), "=&v"(y[3]), "=&v"(y[4]), "=&v"(y[5]), "=&v"(y[6]), "=&v"(y[7])
      : "v"(ad[0]), "v"(ad[1]), "v"(ad[2]), "v"(ad[3]), "i"(STEP)
      : "memory");
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
