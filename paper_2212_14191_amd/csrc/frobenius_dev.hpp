// FrobeniusMap of one polynomial by one workgroup, shared by the element-wise
// and the ciphertext kernels.
//
// out_j = in_{pi(j)}, pi(j) = ((2j+1) g mod 2N - 1) / 2, reads with a stride of
// g words mod N: straight from memory every 4-byte element costs a line of its
// own, and the L2's line rate bounds the map.  Here the polynomial goes through
// LDS: whole-line loads, gathers whose odd stride hits 64 different banks,
// whole-line stores.  At N = 2^16 the halves take turns in LDS and a thread
// keeps its 64 results in registers between.  Bound by HBM for many
// polynomials (512 at N = 2^16, g = 5 / 5^37: 112 / 190 -> 49 us, 5.5 TB/s).
// Few polynomials leave most CUs idle: frob_by_poly (internal.hpp).
#pragma once
#include <type_traits>

#include "internal.hpp"

namespace tfhe {
namespace {

template <int kLogN>
struct FrobShape {
  static constexpr int threads = kLogN <= 13 ? 256 : kLogN == 14 ? 512 : 1024;
  static constexpr int words = kLogN == 16 ? 1 << 15 : 1 << kLogN;  // LDS
};

// f(log_n as a constant), log_n = 12..16
template <typename F>
void frob_switch(uint32_t log_n, F f) {
  switch (log_n) {
    case 12: f(std::integral_constant<int, 12>{}); break;
    case 13: f(std::integral_constant<int, 13>{}); break;
    case 14: f(std::integral_constant<int, 14>{}); break;
    case 15: f(std::integral_constant<int, 15>{}); break;
    default: f(std::integral_constant<int, 16>{}); break;
  }
}

// `lds` holds FrobShape<kLogN>::words; every thread of the workgroup calls this once.
template <int kLogN>
__device__ __forceinline__ void frob_poly(const uint32_t* in, uint32_t* out, uint32_t galois, uint32_t* lds) {
  using S = FrobShape<kLogN>;
  constexpr uint32_t N = 1u << kLogN, T = S::threads, H = S::words, R = N / T, kPhases = N / H;
  typedef __attribute__((address_space(3))) void lds_t;
  const uint32_t tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t src0 = (((2 * tid + 1) * galois) & (2 * N - 1)) >> 1;
  uint32_t v[kPhases > 1 ? R : 1];
#pragma unroll
  for (uint32_t ph = 0; ph < kPhases; ++ph) {
    if (ph) __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < H / 4 / T; ++k) {  // 1 KiB per wave and load
      const uint32_t c = (wave + k * (T / 64)) * 256;
      const uint32_t lds_addr = (uint32_t)(uintptr_t)(lds_t*)(lds + c);
      asm volatile(
          "s_mov_b32 m0, %0\n\t"
          "global_load_lds_dwordx4 %1, off"
          :
          : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(in + ph * H + c + 4 * lane)
          : "memory", "m0");
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    uint32_t src = src0;
#pragma unroll
    for (uint32_t r = 0; r < R; ++r, src = (src + T * galois) & (N - 1)) {  // pi(j + T) = pi(j) + T g mod N
      if (kPhases == 1) {
        out[r * T + tid] = lds[src];
      } else {
        asm volatile("" : "+v"(src));  // (not 64 addresses kept for both phases)
        const bool here = src / H == ph;
        const uint32_t w = lds[src & (H - 1)];
        v[r] = ph == 0 || here ? w : v[r];
      }
    }
  }
  if (kPhases > 1) {
#pragma unroll
    for (uint32_t r = 0; r < R; ++r) out[r * T + tid] = v[r];
  }
}

}  // namespace
}  // namespace tfhe
