// Device building blocks shared by the four-step transform kernels (the
// two-pass kernels and the one-pass kernel): the descriptor table of a fused
// launch, the INT8 matrix-core contraction with its digit-plane fusion and
// Montgomery step, the twist-and-re-slice, the radix-r level B, work-item
// location and the LDS / memory-counter waits.  See ntt_fourstep.hip for the
// arithmetic (balanced byte digits, exactness bounds).
#pragma once
#include <type_traits>

#include "internal.hpp"

namespace tfhe {

// Descriptor table of a fused launch (passed by value as a kernel argument):
// unit k covers global polynomials [begin[k], begin[k+1]).  Every
// unit of a launch has the same N and direction.
constexpr int kMaxUnits = 40;
struct FsUnit {
  const uint32_t* in;
  uint32_t* out;
  const FourStepLimb* limbs;  // the unit's first limb, and its tables (limb l's at
  const unsigned char* tables;  // tables + l * tab_stride: an address, not a load)
  uint32_t batch, batch_inv;
  // inverse second pass: its twist per limb ([limb][64][4]), null for the plan's
  const uint2* twist;
  // second-pass epilogue (forward transforms): out = (acc - y) m_l, or
  // out += (acc - y) m_l, with m_l the Shoup pair of the unit's limb l
  const uint32_t* acc;
  const uint2* mult;
  uint32_t accumulate;
  uint32_t out_tiled;     // inverse second pass: quad-tiled results
};
struct FsTable {
  uint32_t count, total;  // units, polynomials
  uint32_t log_n;
  uint32_t cols;          // S = N / P: columns of this pass (row stride in natural order)
  uint32_t ipp_log;       // log2 of the items per polynomial (N / item words)
  uint32_t share, extra;  // polynomials of walker a: share, one more for a < extra
  uint64_t tab_stride;    // of the limbs' tables, in bytes: pass 1's PassTables,
  uint64_t tab_op;        // pass 2's, pass 1's post-twist; OnePassTables at tab_op
  uint32_t begin[kMaxUnits];  // a unit's first polynomial
  FsUnit u[kMaxUnits];
};
static_assert(sizeof(FsTable) <= 4096, "an FsTable is passed as a kernel argument");
// One-pass kernel (ntt_onepass.hip): N = 2^12..2^15, no epilogue; one
// launch over every unit of `t` (same N and direction).
bool op_supported(uint32_t log_n);
hipError_t op_run(const tfhe_ntt_plan_s* p, bool inverse, const FsTable& t, hipStream_t s);
// First passes with a broadcast or converted input (ntt_convpass.hip): one
// plan's forward units with in_bcast; unit k's tiled output goes to mids[k].
hipError_t cv_run(const tfhe_ntt_plan_s* p, const NttUnit* const* units, uint32_t* const* mids, uint32_t count,
                  hipStream_t s);

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));

__device__ __forceinline__ v4i mfma(v4i a, v4i b, v4i c) {
  return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0);
}

// Constants that no kernel writes, read through the scalar cache.
#define const_as const __attribute__((address_space(4)))

// A modulus as the passes use it: q, -q^{-1} mod 2^32, -q and the twist's
// digit offset 0x80808080 - q (mod 2^32).  k16 is 2^16, opaque to the
// compiler, which otherwise splits a 64-bit multiply-add by it into shifts
// and carries (see fuse_redc).
struct Red {
  uint32_t q, qneg, nq, cq, k16;
  int qs;  // q, its sign unknown to the compiler (else no signed multiply-add)
};
__device__ __forceinline__ Red make_red(uint32_t q, uint32_t qneg) {
  uint32_t k16 = 0x10000u;
  int qs = (int)q;
  asm("" : "+s"(k16), "+s"(qs));
  return Red{q, qneg, 0u - q, 0x80808080u - q, k16, qs};
}

// The modulus for a block of code that multiplies by qs: its sign extension,
// kept from another block, would make a 64 x 64 bit product of every one.
__device__ __forceinline__ Red local(const Red& R) {
  Red r = R;
  asm volatile("" : "+s"(r.qs));
  return r;
}

// a b 2^{-32} mod q as (V + m q) / 2^32, V = a b, m = -V q^{-1} mod 2^32:
// below 2^32 for any a, b < 2^32, and below 2q for a, b < q (not reduced).
__device__ __forceinline__ uint32_t mont_mul_lazy(uint32_t a, uint32_t b, const Red& R) {
  const uint64_t V = (uint64_t)a * b;
  const uint32_t m = (uint32_t)V * R.qneg;
  return (uint32_t)(((uint64_t)m * R.q + V) >> 32);
}

// Fusion and one Montgomery step: V 2^{-32} mod q, in [0, q + 2^17).
// (V + m q) is a multiple of 2^32 below 2^64, so its high word is exact
// (one v_mad_u64_u32).
__device__ __forceinline__ uint32_t fuse_redc(int c0, int c1, int c2, int c3, const Red& R) {
  const uint32_t lo = (uint32_t)c0 + ((uint32_t)c1 << 8);
  const uint32_t hi = (uint32_t)c2 + ((uint32_t)c3 << 8);
  const uint64_t V = (uint64_t)hi * R.k16 + lo;
  const uint32_t m = (uint32_t)V * R.qneg;
  return (uint32_t)(((uint64_t)m * R.q + V) >> 32);
}

// The same fusion, signed, with the twist in one Montgomery step: V w 2^{-32}
// mod q for V = (c0 + 2^8 c1) + 2^16 (c2 + 2^8 c3) and t = {w, 2^16 w mod q},
// below 0.63 q in magnitude.  The halves are below 2^28 + 2^20, so both products
// with w, w16 < q < 2^31 are below 2^59.1; with m = -T q^{-1} mod 2^32 as a
// signed number, (T + m q) / 2^32 lies within q (1/8 + 2^-11 + 1/2): inside the
// digit window as it is (six instructions; fusing, reducing and multiplying one
// after the other take nine).
__device__ __forceinline__ int fuse_twist(int c0, int c1, int c2, int c3, uint2 t, const Red& R) {
  const int lo = (int)((uint32_t)c0 + ((uint32_t)c1 << 8)), hi = (int)((uint32_t)c2 + ((uint32_t)c3 << 8));
  const int64_t T = (int64_t)hi * (int)t.y + (int64_t)lo * (int)t.x;
  const int m = (int)((uint32_t)T * R.qneg);
  return (int)(((int64_t)m * R.qs + T) >> 32);
}
// a b 2^{-32} mod q, signed: below |a| |b| 2^{-32} + q / 2 in magnitude.
__device__ __forceinline__ int mont_signed(int a, int b, const Red& R) {
  const int64_t T = (int64_t)a * b;
  const int m = (int)((uint32_t)T * R.qneg);
  return (int)(((int64_t)m * R.qs + T) >> 32);
}
// The residue of v in (-q, q).
__device__ __forceinline__ uint32_t wrap_signed(int v, uint32_t q) { return min((uint32_t)v, (uint32_t)v + q); }

// Twist (Shoup, t = {w, companion}) and re-slice into digits.  With
// h = floor(r w' / 2^32) the product z = r w - h q lies in
// [0, q (1 + r / 2^32)), so z - q is in [-q, q r / 2^32): inside the digit
// window [-0x80808080, 0x7F7F7F7F] for every q < 2^31 as long as
// r <= 0.996 2^32 (callers: r < q + 2^17, or below 1.94 q after a lazy
// Montgomery product).  Its digits are (z + (0x80808080 - q)) ^ 0x80808080.
__device__ __forceinline__ uint32_t twist_digits(uint32_t r, uint2 t, const Red& R) {
  const uint32_t h = __umulhi(r, t.y);
  return (r * t.x + h * R.nq + R.cq) ^ 0x80808080u;
}

// Digits of a canonical residue w < q.  Above 0x7F7F7F7F it enters as w - q:
// d = w + 0x80808080 then wraps to a small number and d - q to a large one,
// while below the larger of the two is d.
__device__ __forceinline__ uint32_t residue_digits(uint32_t w) { return (w + 0x80808080u) ^ 0x80808080u; }
__device__ __forceinline__ uint32_t residue_digits_big(uint32_t w, uint32_t q) {
  const uint32_t d = w + 0x80808080u;
  return max(d, d - q) ^ 0x80808080u;
}

// After level A, lane (s, g) register j holds MFMA row i = 4g + j, i.e.
// vector m = i / kR, element v = i % kR.  After level B register j holds
// output t of vector m (the output index is s + 16 t).
template <int kR>
__device__ __forceinline__ void lane_out(int g, int j, int& m, int& t) {
  if (kR == 16) { m = 0; t = 4 * g + j; }
  else if (kR == 8) { m = g >> 1; t = 2 * j + (g & 1); }
  else if (kR == 4) { m = g; t = j; }
  else if (kR == 2) { m = 2 * g + (j >> 1); t = j & 1; }
  else { m = 4 * g + j; t = 0; }
}

// Radix-4 DFT y_t = sum_v x_v w4^{vt} (w4 of order 4) on residues in [0, q).
__device__ __forceinline__ void dft4(uint32_t* x, uint2 w4, uint32_t q) {
  const uint32_t a0 = add_mod(x[0], x[2], q), a1 = sub_mod(x[0], x[2], q);
  const uint32_t b0 = add_mod(x[1], x[3], q);
  const uint32_t b1 = mul_shoup(sub_mod(x[1], x[3], q), w4.x, w4.y, q);
  x[0] = add_mod(a0, b0, q);
  x[1] = add_mod(a1, b1, q);
  x[2] = sub_mod(a0, b0, q);
  x[3] = sub_mod(a1, b1, q);
}

// Level B for kR < 16: the kR-point cyclic DFT over v of y (residues in
// [0, q)), with lb[x] = rho^x for the root rho of order kR.  For kR = 8 the
// eight inputs of a vector sit in lanes g and g ^ 1 (four each): lane
// parity h computes the outputs t = 2 j + h from e_j = z_j + z_{j+4} (h = 0)
// or o_j = (z_j - z_{j+4}) rho^j (h = 1) with a radix-4 DFT by rho^2.
template <int kR>
__device__ __forceinline__ void level_b(uint32_t* y, const uint2* lb, const uint2* rj, int g,
                                        uint32_t q) {
  if (kR == 2) {
#pragma unroll
    for (int j = 0; j < 4; j += 2) {
      const uint32_t a = y[j], b = y[j + 1];
      y[j] = add_mod(a, b, q);
      y[j + 1] = sub_mod(a, b, q);
    }
  } else if (kR == 4) {
    dft4(y, lb[1], q);
  } else if (kR == 8) {
    const bool h = g & 1;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      // swapping the odd rows of 16 lanes of one copy with the even rows of
      // another leaves z_j in the first and z_{j+4} in the second, in both lanes
      const auto z = __builtin_amdgcn_permlane16_swap(y[j], y[j], false, false);
      const uint32_t hi = z[1];
      y[j] = mul_shoup(add_mod(z[0], h ? q - hi : hi, q), rj[j].x, rj[j].y, q);
    }
    dft4(y, lb[2], q);
  }
}
// Geometry of a pass with P = 16 kR points.  A work item is P rows x W
// vectors (columns) of one polynomial, 1024 words per wave; each wave
// transforms four sets of vectors per item.  Its LDS tile is a sequence of
// 1 KiB slabs; slab k holds rows Rs k .. Rs k + Rs - 1 of every column of the
// item, slot L (16 bytes) row Rs k + L % Rs, columns 4 (L / Rs) .. + 3 (a
// "quad"), so one direct-to-LDS load covers Rs rows x W columns.  Narrow
// items (W = 16 for kR = 16) use 4 waves and Rs = 16: 64-byte row segments.
// Wide items (kR = 16 with at least 32 columns) use 8 waves and Rs = 8, so
// every load and store moves whole 128-byte lines.  For kR < 16, Rs = kR and
// W = 256 / kR >= 32.  Slabs are padded where 16 lanes of an LDS access
// would otherwise hit the same banks in several slabs.
template <bool kFirst, int kR, bool kWide>
struct Geo {
  static constexpr int waves = kWide ? 8 : 4;
  static constexpr int threads = 64 * waves;
  static constexpr int item = 1024 * waves;      // words per work item
  static constexpr int slabs = item / 256;
  static constexpr int P = 16 * kR;
  static constexpr int W = item / P;             // vectors per item
  static constexpr int Mt = 16 / kR;             // vectors per MFMA tile (quads per wave)
  static constexpr int Rs = kWide ? 8 : kR;      // rows per slab
  static constexpr int pitch = kWide ? 256 + 32 : (kFirst || kR == 16) ? 256 : 256 + 4 * kR;
  static constexpr int tile = slabs * pitch;
  static_assert(!kWide || kR == 16, "wide items are for the 256-point stage");
};

typedef __attribute__((address_space(3))) void lds_void_t;

// Each wave loads slabs 4 wave .. 4 wave + 3 of an item: one 16-byte
// direct-to-LDS load per lane per slab (streaming hint: every byte is read
// once); lane L's bytes land at the slab base +
// 16 L.  Issued as inline assembly so that the compiler does not serialise
// later LDS reads on these loads: the pipeline waits for them explicitly
// (wait_item) before a barrier.
template <int kPitch>
__device__ __forceinline__ void issue_tile(const uint32_t* src, const uint32_t* off, uint32_t* stage, int wave) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t* g = src + off[j];
    const uint32_t lds_addr = (uint32_t)(uintptr_t)(lds_void_t*)(stage + (4 * wave + j) * kPitch);
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "global_load_lds_dwordx4 %1, off nt"
        :
        : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(g)
        : "memory", "m0");
  }
}

// Loads the values (a kernel's arguments) here, together: each line of the
// arguments is a miss of some 200 ns in the scalar cache, one after the other
// where the code happens to use them.
template <typename A, typename B, typename C, typename D, typename E, typename F>
__device__ __forceinline__ void touch(A a, B b, C c, D d, E e, F f) {
  asm volatile("" ::"s"(a), "s"(b), "s"(c), "s"(d), "s"(e), "s"(f));
}

struct Item {
  uint32_t unit, limb;
  size_t poly_base;  // word offset of the polynomial within the unit's arrays
};
// n / d for n < 2^31, with inv = ceil(2^32 / d) from div_inv (the plain
// quotient is some 35 dependent vector instructions, at every kernel's start).
inline uint32_t div_inv(uint32_t d) { return d > 1 ? 0xFFFFFFFFu / d + 1 : 0; }
__device__ __forceinline__ uint32_t div_by(uint32_t n, uint32_t d, uint32_t inv) {
  if (d == 1) return n;
  const uint32_t k = __umulhi(n, inv);  // the quotient or one more
  return k * d > n ? k - 1 : k;
}
// The unit of global polynomial p (a walk's start; later polynomials advance
// the running index in locate): one scalar load for a few units, else the lanes
// compare one entry each.
__device__ __forceinline__ uint32_t find_unit(const uint32_t* begin, uint32_t count, uint32_t p) {
  if (count == 1) return 0;
  if (count <= 8) {
    uint32_t k = 0;
#pragma unroll
    for (uint32_t i = 1; i < 8; ++i) k += (uint32_t)(i < count) & (uint32_t)(begin[i] <= p);
    return k;
  }
  const uint32_t lane = threadIdx.x & 63;
  const bool past = lane < count && begin[lane < count ? lane : 0] <= p;
  return (uint32_t)__popcll(__ballot(past)) - 1;
}
// Global polynomial p -> (unit, limb, offset); `k` is a running unit index
// (p only increases along a walk).
__device__ __forceinline__ Item locate(const FsTable& t, uint32_t p, uint32_t& k) {
  while (k + 1 < t.count && p >= t.begin[k + 1]) ++k;
  const uint32_t local = p - t.begin[k];
  Item it;
  it.unit = k;
  it.limb = div_by(local, t.u[k].batch, t.u[k].batch_inv);
  it.poly_base = (size_t)local << t.log_n;
  return it;
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// Workgroup barrier without the memory fence of __syncthreads (which would
// wait for every outstanding load): LDS accesses of this wave are completed
// first; the direct-to-LDS loads are covered by wait_item.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
}

}  // namespace
}  // namespace tfhe
