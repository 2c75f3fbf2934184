// Element-wise kernels of the hierarchical reconstruction (Sec. IV-A,
// Table 2): Hada-Mult, Ele-Add, Ele-Sub and FrobeniusMap, over the
// (limb, batch, N) layout.  All are HBM-bound: 16-byte accesses, one pass.
#include "frobenius_dev.hpp"

namespace tfhe {
namespace {

constexpr int kThreads = 256;

template <int kOp>
__device__ __forceinline__ uint4 ew(uint4 x, uint4 y, const ModConst& m) {
  if (kOp == EW_ADD || kOp == EW_CT_ADD)
    return make_uint4(add_mod(x.x, y.x, m.q), add_mod(x.y, y.y, m.q), add_mod(x.z, y.z, m.q), add_mod(x.w, y.w, m.q));
  if (kOp == EW_SUB)
    return make_uint4(sub_mod(x.x, y.x, m.q), sub_mod(x.y, y.y, m.q), sub_mod(x.z, y.z, m.q), sub_mod(x.w, y.w, m.q));
  return make_uint4(mul_mod(x.x, y.x, m), mul_mod(x.y, y.y, m), mul_mod(x.z, y.z, m), mul_mod(x.w, y.w, m));
}

// blockIdx.y is the limb, so that its constants are scalar (an index over all
// limbs took a 64-bit division per 16 bytes).  A ciphertext op does both
// components of a position: one launch, and CMULT reads its plaintext once.
// Bound by HBM; CMULT then HADD of 32 ciphertexts, N = 2^15, level 12: 103 ->
// 97 us for the pair of calls (554 MB; 5.7 TB/s, part of it the last-level
// cache's).  Streaming hints on the loads or stores are 1-4 % slower.
template <int kOp>
__global__ void __launch_bounds__(kThreads)
ew_kernel(const ModConst* __restrict__ mods, const uint4* __restrict__ a, const uint4* __restrict__ b,
          uint4* __restrict__ c, uint64_t plane4, uint64_t per_limb4, uint32_t n4) {
  constexpr bool kPair = kOp == EW_CT_MUL || kOp == EW_CT_ADD;
  const uint32_t limb = blockIdx.y;
  const ModConst m = mods[limb];
  const uint64_t base = limb * per_limb4, step = (uint64_t)gridDim.x * kThreads;
  for (uint64_t k = blockIdx.x * (uint64_t)kThreads + threadIdx.x; k < per_limb4; k += step) {
    const uint64_t i = base + k;
    const uint4 y = b[kOp == EW_MUL_BCAST ? (uint64_t)limb * n4 + (k & (n4 - 1)) : i], x = a[i];
    if (kPair) {
      const uint4 x1 = a[plane4 + i], y1 = kOp == EW_CT_ADD ? b[plane4 + i] : y;
      c[i] = ew<kOp>(x, y, m);
      c[plane4 + i] = ew<kOp>(x1, y1, m);
    } else {
      c[i] = ew<kOp>(x, y, m);
    }
  }
}

// out_j = in_{pi(j)}, pi(j) = ((2j+1) k mod 2N - 1) / 2 (FrobeniusMap).
__global__ void __launch_bounds__(kThreads)
frobenius_kernel(const uint32_t* __restrict__ in, uint32_t* __restrict__ out, uint32_t galois,
                 uint64_t total, uint32_t log_n) {
  const uint32_t n = 1u << log_n, mask2n = 2 * n - 1;
  for (uint64_t i = blockIdx.x * (uint64_t)kThreads + threadIdx.x; i < total;
       i += (uint64_t)gridDim.x * kThreads) {
    const uint32_t j = (uint32_t)(i & (n - 1));
    const uint32_t src = (((2 * j + 1) * galois) & mask2n) >> 1;
    out[i] = in[(i - j) + src];
  }
}

// The same with a workgroup per polynomial.
template <int kLogN>
__global__ void __launch_bounds__(FrobShape<kLogN>::threads)
frobenius_poly(const uint32_t* in, uint32_t* out, uint32_t galois) {
  __shared__ __attribute__((aligned(16))) uint32_t lds[FrobShape<kLogN>::words];
  const uint64_t at = (uint64_t)blockIdx.x << kLogN;
  frob_poly<kLogN>(in + at, out + at, galois, lds);
}

// out[l][b][i] = in[b][i] mod q_l for small signed integers in (-2^31, 2^31).
__global__ void __launch_bounds__(kThreads)
load_small_kernel(const ModConst* __restrict__ mods, const int32_t* __restrict__ in,
                  uint32_t* __restrict__ out, uint64_t total, uint64_t per_limb) {
  for (uint64_t i = blockIdx.x * (uint64_t)kThreads + threadIdx.x; i < total;
       i += (uint64_t)gridDim.x * kThreads) {
    const uint32_t l = (uint32_t)(i / per_limb);
    const uint32_t q = mods[l].q;
    const int32_t x = in[i % per_limb];
    uint32_t r = (uint32_t)(x < 0 ? -(int64_t)x : x) % q;
    out[i] = (x < 0 && r) ? q - r : r;
  }
}

uint32_t grid_for(uint64_t items) {
  uint64_t blocks = (items + kThreads - 1) / kThreads;
  return (uint32_t)(blocks < 8192 ? (blocks ? blocks : 1) : 8192);
}

}  // namespace

hipError_t ew_launch(EwOp op, const ModConst* mods, const uint32_t* a, const uint32_t* b,
                     uint32_t* c, uint32_t limb_count, uint32_t batch, uint32_t n, hipStream_t s) {
  if (op == EW_CT_ADD) limb_count /= 2;
  const uint64_t per_limb4 = (uint64_t)batch * n / 4;
  if (limb_count == 0 || per_limb4 == 0) return hipSuccess;
  if (limb_count > 65535) return hipErrorInvalidValue;
  const dim3 grid(grid_for(per_limb4), limb_count);
  const uint64_t plane4 = limb_count * per_limb4;
  const uint4 *A = (const uint4*)a, *B = (const uint4*)b;
  uint4* C = (uint4*)c;
  auto run = [&](auto kernel) {
    TFHE_TIMED(K_EW, s, hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, s, mods, A, B, C, plane4, per_limb4, n / 4));
  };
  switch (op) {
    case EW_MUL: run(ew_kernel<EW_MUL>); break;
    case EW_ADD: run(ew_kernel<EW_ADD>); break;
    case EW_SUB: run(ew_kernel<EW_SUB>); break;
    case EW_MUL_BCAST: run(ew_kernel<EW_MUL_BCAST>); break;
    case EW_CT_MUL: run(ew_kernel<EW_CT_MUL>); break;
    case EW_CT_ADD: run(ew_kernel<EW_CT_ADD>); break;
  }
  return hipGetLastError();
}

hipError_t load_small_launch(const ModConst* mods, const int32_t* in, uint32_t* out,
                             uint32_t limb_count, uint32_t batch, uint32_t n, hipStream_t s) {
  const uint64_t per_limb = (uint64_t)batch * n, total = per_limb * limb_count;
  TFHE_TIMED(K_EW, s, hipLaunchKernelGGL(load_small_kernel, dim3(grid_for(total)), dim3(kThreads), 0, s,
                                         mods, in, out, total, per_limb));
  return hipGetLastError();
}

hipError_t frobenius_launch(const uint32_t* in, uint32_t* out, uint32_t galois, uint32_t rows,
                            uint32_t log_n, hipStream_t s) {
  if (frob_by_poly(log_n, rows, frob_lines(galois, log_n))) {
    frob_switch(log_n, [&](auto ln) {
      constexpr int kLogN = decltype(ln)::value;
      TFHE_TIMED(K_FROB, s, hipLaunchKernelGGL(frobenius_poly<kLogN>, dim3(rows), dim3(FrobShape<kLogN>::threads), 0,
                                               s, in, out, galois));
    });
    return hipGetLastError();
  }
  const uint64_t total = (uint64_t)rows << log_n;
  TFHE_TIMED(K_FROB, s, hipLaunchKernelGGL(frobenius_kernel, dim3(grid_for(total)), dim3(kThreads), 0, s, in, out,
                     galois, total, log_n));
  return hipGetLastError();
}

}  // namespace tfhe
