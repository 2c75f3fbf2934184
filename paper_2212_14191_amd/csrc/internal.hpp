// Internal types of the library: plan and context state, error plumbing,
// kernel launchers.  Not part of the ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <string>
#include <vector>

#include "../../include/tfhe.h"
#include "modarith.hpp"

namespace tfhe {

void set_error(const std::string& msg);
tfhe_status fail(tfhe_status s, const std::string& msg);
tfhe_status hip_check(hipError_t e, const char* what);

// Tables of one pass of the four-step algorithm (per limb and direction).
// A pass transforms vectors of P = 16 r points (r in {1, 2, 4, 8, 16}),
// decomposed as 16 x r: a radix-16 level on the matrix cores (level A), a
// twist, and a radix-r level (level B: matrix cores when r = 16, VALU
// butterflies otherwise).  Laid out exactly as the kernels load them.
//   opA[j][lane][4]   level-A twiddle operand, digit plane j (4 dwords/lane)
//   opB[j][lane][4]   level-B twiddle operand (r = 16 only)
//   twist[lane][j]    twist after level A, {w, 2^16 w mod q} for w = T 2^32 mod q
//   lb[16]            level-B constants (r < 16): lb[0..3] = rho^0..rho^3 of
//                     the radix-r root rho; lb[8 + t] = factor of output t
struct PassTables {
  uint32_t opA[4][64][4];
  uint32_t opB[4][64][4];
  uint2 twist[64][4];
  uint2 lb[16];
};

// Plain matrices of one 256-point pass (16 x 16 split) for the vector-ALU
// GEMM variant, as Shoup pairs {w, companion}: level A WA[u][s], twist
// T[s][v], level B WB[t][v].
// Vector-ALU variant: the two 16-point matrices in Montgomery form with
// R = 2^64 (W 2^64 mod q), stored output-major (WA[s][u], WB[t][v]), and the
// twist as Shoup pairs T[s][v].
struct CoPass {
  uint32_t WA[16][16], WB[16][16];
  uint2 T[16][16];
};

// Tables of the one-pass four-step kernel (N = 2^12..2^15) for one limb and
// direction; its first pass uses the two-pass kernel's pass-1 tables.  The
// post-twist factors also serve the conversion-fused first pass (forward,
// N = 2^12..2^16), whose waves each take one step's columns.
//   p2       second pass.  Forward (256-point): level B's twiddles unscaled
//            and the twist carrying 2^64, so opB equals opA (the 16-point DFT
//            matrix is symmetric).  Inverse (N1-point): opA with the level-A
//            index u = g + 4c for lane (i, g), dword c, instead of 4g + c.
//   post_b   [set][j / 2][lane][j % 2] first-pass post-twist, the factor fixed
//            per lane: P(4m + set, out), Shoup; after a matrix-core level B
//            {w, 2^16 w mod q} for w = 2^32 P; a lane's 16 bytes lie next to the next lane's, so that
//            LDS copies are read without bank conflicts
//   post_a   [step][lane][j] the factor of a step whose first column quad is
//            Q0 = step * 16 / r: P(4 Q0 + 4m, out) / P(4m, out), times 2^32
//            (Montgomery form); (m, out) as lane / register j hold them.
struct OnePassTables {
  PassTables p2;
  uint2 post_b[4][2][64][2];
  uint32_t post_a[64][64][4];
};

// Device-side description of one limb for the four-step kernels (the matrix-core
// kernels' tables lie at computed places: tfhe_plan_impl::d_fs_blob).
struct FourStepLimb {
  const CoPass* co1;        // vector-ALU variant (N = 2^16 only): pass matrices
  const CoPass* co2;
  const uint2* co_post;     // [256 columns][256 outputs]: post-twist of pass 1
  uint32_t q, qneg;         // modulus and -q^{-1} mod 2^32
};

struct tfhe_plan_impl {
  uint32_t log_n = 0, n = 0, n_limbs = 0;
  tfhe_ntt_algo algo = TFHE_NTT_BUTTERFLY;  // what AUTO resolves to
  bool has_mfma = false;
  bool has_co = false;            // vector-ALU four-step variant (N = 2^16)
  int device = 0;
  uint32_t num_cus = 256;         // compute units of the device
  uint32_t fs_wg_per_cu = 0;      // persistent four-step workgroups per CU (0: occupancy)
  uint32_t fs_wide = 0;           // 256-point stage items: 0 auto, 1 narrow, 2 wide when possible
  uint32_t fs_passes = 0;         // four-step HBM passes: 0 auto (by size and launch: use_onepass), 1 one, 2 two
  uint32_t fs_ring = 0;           // LDS ring stages of the wide-item passes: 0 auto (2), 2, 3
  uint32_t ks_inner = 0;          // key switching: 0 default (fused), 1 fused second pass + inner product, 2 separate
  std::vector<uint32_t> q, psi;
  // device arrays
  ModConst* d_mod = nullptr;      // [n_limbs]
  uint2* d_bf_fwd = nullptr;      // [n_limbs][N] {psi^{brv(i)}, companion}
  uint2* d_bf_inv = nullptr;      // [n_limbs][N] {psi^{-brv(i)}, companion}
  uint2* d_ninv = nullptr;        // [n_limbs] {N^{-1}, companion}
  FourStepLimb* d_fs_fwd = nullptr;  // [n_limbs]
  FourStepLimb* d_fs_inv = nullptr;  // [n_limbs]
  void* d_fs_blob = nullptr;          // owns all four-step tables: limb l, direction d at (2 l + d) fs_limb_bytes
  size_t fs_limb_bytes = 0;           // (PassTables of pass 1 and 2, pass 1's post-twist, OnePassTables at fs_op_off)
  size_t fs_op_off = 0;
  std::vector<void*> owned;
};

}  // namespace tfhe

struct tfhe_ntt_plan_s : tfhe::tfhe_plan_impl {};

namespace tfhe {

// Constants of one target modulus m of a basis conversion fused with a
// transform (ntt_convpass.hip): c[r] the representative of C[r] 2^32 mod m in
// [-m/2, m/2), init = m 2^32 + (2^30 sum_r c[r] mod m).
struct CvTarget {
  int32_t c[8];
  uint64_t init;
  uint32_t q, qneg;
};
// The basis conversion whose results a forward transform takes as its input
// (NttUnit::conv): x_t = sum_r y_r C[t][r] mod m_t from nin <= 8 planes of
// residues y_r (already times the inputs' constants: NttUnit::twist).  Target
// u is extended-basis position pos = u, or u + nd from the digit's first limb
// d0 on (its own nd limbs are skipped); position pos is plan limb pos below
// `level`, L + pos - level above.
struct ConvSource {
  const CvTarget* tgt;  // [plan limb]
  uint32_t nin, d0, nd, level, L;
  bool tiled;           // the inputs are quad-tiled (NttUnit::out_tiled)
};

// ---- operation-level batching: one fused launch over many transforms
// A transform unit: `batch` polynomials of limbs [limb_begin, +limb_count) of
// a plan, forward or inverse, in -> out (in == out allowed), with its own
// slice of the workspace.
struct NttUnit {
  const tfhe_ntt_plan_s* plan;
  bool inverse;
  const uint32_t* in;
  uint32_t* out;
  uint32_t limb_begin, limb_count, batch;
  // Forward four-step transforms only: instead of the transform y, write
  // out = (acc - y) mult_l (epi_add: out += ...), mult_l the Shoup pair of
  // limb limb_begin + l; acc has the layout of out.
  const uint32_t* acc = nullptr;
  const uint2* epi_mult = nullptr;
  bool epi_add = false;
  // Forward four-step transforms only: run the first pass alone, writing its
  // tiled intermediate to `out` (the second pass is left to a fused
  // consumer, ip_run)
  bool pass1_only = false;
  // Forward four-step transforms only: every limb of the unit reads the same
  // input plane `in` ([batch][N], values below 2^31, not reduced by the
  // limb's modulus), i.e. the transform of that integer polynomial modulo
  // each of the unit's limbs
  bool in_bcast = false;
  // With in_bcast: the limbs' inputs are the results of this conversion of
  // the nin planes at `in` ([nin][batch][N]); limb_count counts its targets
  // (limb_begin 0), and with pass1_only target u's tiled intermediate goes
  // to position pos of `out` ([level + K][batch][N]).
  const ConvSource* conv = nullptr;
  // With in_bcast and no conversion: the input plane is quad-tiled
  bool in_tiled = false;
  // Inverse four-step transforms of N >= 2^15 only (two passes): the results
  // are written quad by quad, coefficient n = 256 n1 + n2 of a polynomial at
  // ((n2 / 4) N1 + n1) 4 + n2 % 4 (N1 = N / 256), as a conversion or broadcast
  // input reads them
  bool out_tiled = false;
  // Inverse four-step transforms only: the second pass's twist of each limb
  // ([limb_count][64][4]), the plan's times a constant of the limb: the
  // results come out times that constant.
  const uint2* twist = nullptr;
};
// Runs every unit with the four-step algorithm (all units need has_mfma) or
// the butterfly; ws must hold the sum of the units' workspaces.
hipError_t fs_run_units(const NttUnit* u, uint32_t count, void* ws, hipStream_t s);
hipError_t bf_run_units(const NttUnit* u, uint32_t count, void* ws, hipStream_t s);
size_t unit_ws_bytes(const NttUnit& u, bool mfma);

// ---- butterfly launchers (ntt_butterfly.hip)
size_t bf_workspace_bytes(const tfhe_ntt_plan_s* p, uint32_t limb_count, uint32_t batch);
hipError_t bf_forward(const tfhe_ntt_plan_s* p, const uint32_t* in, uint32_t* out, void* ws,
                      uint32_t limb_begin, uint32_t limb_count, uint32_t batch, hipStream_t s);
hipError_t bf_inverse(const tfhe_ntt_plan_s* p, const uint32_t* in, uint32_t* out, void* ws,
                      uint32_t limb_begin, uint32_t limb_count, uint32_t batch, hipStream_t s);

// ---- four-step MFMA launchers (ntt_fourstep.hip)
bool fs_supported(uint32_t log_n);
size_t fs_workspace_bytes(const tfhe_ntt_plan_s* p, uint32_t limb_count, uint32_t batch);
hipError_t fs_forward(const tfhe_ntt_plan_s* p, const uint32_t* in, uint32_t* out, void* ws,
                      uint32_t limb_begin, uint32_t limb_count, uint32_t batch, hipStream_t s);
hipError_t fs_inverse(const tfhe_ntt_plan_s* p, const uint32_t* in, uint32_t* out, void* ws,
                      uint32_t limb_begin, uint32_t limb_count, uint32_t batch, hipStream_t s);
// Workgroups per CU in the grid of a two-pass kernel with 8-wave items, of
// which one is resident: the others start as the first ones end.  Each of them
// fills its ring and loads its limb's tables (first pass: 64 KiB of post-twist
// among them) anew, and with one item each it prefetches nothing, so a launch of
// few items takes one workgroup per CU; with many, several balance the tail.
// Every 16 workgroups walk a range of polynomials of their own; where these
// ranges start a multiple of 16 polynomials apart, all walk the same addresses
// modulo some MiB, and five (other ranges) are faster than four.
// us with 1 : 2 : 4 (: 5) per CU, by items per CU:
//   N = 2^16, one direction
//      3  27.4 : 35.1 : 34.2;   4  35.9 : 37.9 : 45.3;   6  47.2 : 52.0 : 66.7;
//     10  70.9 : 75.0 : 90.7;  20  132.9 : 134.0 : 139.7;  24  162.3 : 159.5 : 163.0
//   N = 2^16, forward and inverse
//     28  371 : 383 : 383 : 392;   38  509 : 505 : 509 : 529;  40 (8 limbs)  542 : 530 : 516 : 561;
//     48  662 : 653 : 623 : 631;   60  807 : 789 : 777 : 781;  104  1394 : 1359 : 1337 : 1349;
//    176  2305 : 2274 : 2247 : 2262;  16 n polynomials apart (with four):  64  834 : 882 : 886 : 835;
//     96  1257 : 1241 : 1258 : 1236;  128  1688 : 1719 : 1816 : 1651
//   N = 2^15, forward and inverse
//     16  234 : 242 : 246 : 259;   48  647 : 645 : 646 : 653;  88  1164 : 1156 : 1154 : 1164
//   RESCALE, N = 2^16, level 24, 2..32 elements (1 : 2 : 4): 41.4 : 47.1 : 43.2, 62.5 : 63.1 : 74.3,
//     102 : 103 : 106, 180 : 185 : 189, 371 : 377 : 380
//   HMULT, N = 2^16, level 12, 4 pairs: 139.8 : 153.1 : 149.6, 8: 239 : 250 : 273, 64: 1656 : 1640 : 1646
inline uint32_t wide_wg_per_cu(uint32_t polys, uint32_t items_per_poly, uint32_t num_cus) {
  const uint64_t items = (uint64_t)polys * items_per_poly;
  if (items <= 24ull * num_cus) return 1;
  if (items < 48ull * num_cus) return 2;
  const uint32_t groups = num_cus >= 4 ? num_cus / 4 : 1, apart = (polys + groups / 2) / groups;
  return apart % 16 == 0 ? 5 : 4;
}
// Vector-ALU GEMM variant of the same passes (plan->has_co); same workspace.
hipError_t co_transform(const tfhe_ntt_plan_s* p, bool inverse, const uint32_t* in, uint32_t* out,
                        void* ws, uint32_t limb_begin, uint32_t limb_count, uint32_t batch,
                        hipStream_t s);

// ---- element-wise launchers (elementwise.hip)
// The ciphertext ops take both components of a and c, one after the other:
// EW_CT_MUL by one plaintext b [limb_count][batch][N]; EW_CT_ADD with a second
// ciphertext b, limb_count counting the limbs of both components.
enum EwOp { EW_MUL = 0, EW_ADD = 1, EW_SUB = 2, EW_MUL_BCAST = 3, EW_CT_MUL = 4, EW_CT_ADD = 5 };
hipError_t ew_launch(EwOp op, const ModConst* mods, const uint32_t* a, const uint32_t* b,
                     uint32_t* c, uint32_t limb_count, uint32_t batch, uint32_t n, hipStream_t s);
hipError_t frobenius_launch(const uint32_t* in, uint32_t* out, uint32_t galois, uint32_t rows,
                            uint32_t log_n, hipStream_t s);
// Per-batch-element Galois elements of a multi-rotation: row r of the
// [rows][N] array (rows = limbs x batch, batch fastest) uses g[r % batch].
constexpr uint32_t kMaxRotBatch = TFHE_ROTATE_MULTI_MAX;
struct GaloisSet {
  uint32_t batch;
  uint32_t g[kMaxRotBatch];
};
// How many lines (of 128 bytes) 64 lanes touch that map a polynomial element by
// element: 2-3 for the identity and the conjugation, 2 |g| for small g, 64 at
// most.  g = +-1 mod N / k (rotations by N / 4k slots and their multiples) is k
// streams; what a lane leaves of a line is read N / k elements on, for k <= 16
// and N >= 2^15 by a workgroup of the same XCD, so they count less (times below).
inline uint32_t frob_lines(uint32_t galois, uint32_t log_n) {
  uint64_t seen[32] = {};  // N <= 2^16
  uint32_t src = galois / 2, lines = 0;
  for (uint32_t j = 0; j < 64; ++j, src += galois) {
    const uint32_t line = (src & ((1u << log_n) - 1)) / 32;
    const uint64_t bit = 1ull << (line % 64);
    lines += (seen[line / 64] & bit) == 0;
    seen[line / 64] |= bit;
  }
  const uint32_t part = (1u << log_n) / 16 - 1;
  const bool streams = (galois & part) == 1 || (galois & part) == part;
  return log_n < 15 || !streams ? lines : log_n == 15 ? lines / 2 : lines / 4;
}
// Whether FrobeniusMap goes by whole polynomials through LDS (frobenius_dev.hpp,
// N = 2^12..2^16) or element by element: the former once there are enough
// polynomials to fill the CUs, the earlier the more lines the latter touches.
// With g = +-1 that reads whole lines itself, and at N >= 2^15, where a workgroup
// fills a CU's LDS, stays ahead until input and output outgrow the last-level
// cache.  us, by element : by polynomial, `polys` at galois -1, 3, 5, 25 / 5^37:
//   2^12  96    2.8:2.8   2.8:2.8   2.8:2.9   3.1:2.9 /  3.0:2.9;  192  3.2:3.0   3.2:3.0   3.2:3.0    4.0:3.0
//   2^13  64    2.9:3.1   2.9:3.1   2.9:3.1   3.9:3.1 /  3.4:3.1;  128  3.5:3.4   3.5:3.4   3.5:3.4    6.5:3.4
//   2^14  64    3.5:3.7   3.5:3.7   3.5:3.6   6.5:3.7 /  7.0:3.7;  96   4.1:4.0   4.0:4.0   5.9:4.0    9.7:4.0
//         256   6.0:5.6-7.1 11.6:5.6 15.6:5.6 21.5:5.6;           384  10.0:8.3 16.1:8.7  21.5:8.7   31.4:8.7
//   2^15  32    3.5:4.4   3.5:4.4   3.6:4.4   6.5:4.4 /  7.7:4.4;  48   4.1:4.7   4.0:4.7   5.9:4.7    9.7:4.8
//         96    5.3:6.2   9.6:6.2  12.4:6.2  16.7:6.2;             1024 40:43     73:43     112:43     175:43
//   2^16  32    4.8:10.2  4.9:10.2  9.6:10.3 12.0:10.2 / 13.7:10.2; 48  5.3:11.0  9.5:11.0 12.4:11.0  16.8:11.0
//         64    6.0:11.9 11.4:11.9 15.6:11.9 21.6:11.8;            96  10.3:14.3 16.1:14.2 21.5:14.2  31.4:14.2
//         512   40:49     73:49     112:49    176:49;             1024 122:111   144:111   232:111    497:110
// and at galois 1 + N / 4, 1 + N / 8, 1 + N / 16:
//   2^15  48    4.1:4.7   4.6:4.7    6.0:4.7;  96  5.6:6.1   6.8:6.1   9.6:6.1;   512  21.7:22.7  26:23  41:23
//   2^16  48    5.5:11    6.6:11.0   9.2:11.0; 96  10.3:14   12.5:14   17.5:14.1; 512  39:49      50:49  81:49
inline bool frob_by_poly(uint32_t log_n, uint64_t polys, uint32_t lines) {
  if (log_n < 12 || log_n > 16) return false;
  if (lines <= 4) return log_n >= 15 ? polys << log_n > 1ull << 25 : polys >= (log_n == 14 ? 384 : 192);
  if (lines <= 8) return polys >= 96;
  if (lines <= 32) return polys >= (log_n >= 15 ? 48 : 96);
  return polys >= (log_n >= 15 ? 32 : 64);
}
// The same for a set: the mean over the first eight.
inline uint32_t frob_lines(const GaloisSet& gs, uint32_t log_n) {
  const uint32_t n = gs.batch < 8 ? gs.batch : 8;
  uint32_t sum = 0;
  for (uint32_t b = 0; b < n; ++b) sum += frob_lines(gs.g[b], log_n);
  return sum / n;
}

// ---- per-kernel event timing (timing.cpp)
enum KernelId {
  K_FS_PASS1 = 0, K_FS_PASS2, K_BF_SINGLE, K_BF_COLS, K_BF_ROWS, K_EW, K_TENSOR, K_MODUP,
  K_INNER, K_MD_CONV, K_MD_FINAL, K_FROB, K_RS_BCAST, K_RS_FINAL, K_CO_PASS1, K_CO_PASS2, K_OP, K_IP,
  K_CONV_PASS1
};
// Resident workgroups per CU of a kernel, queried once per process: the
// dispatcher's workers may race to fill the cache; they store one value.
template <typename K>
int occupancy_cached(std::atomic<int>& cache, K kernel, int threads) {
  int v = cache.load(std::memory_order_relaxed);
  if (v == 0) {
    int n = 0;
    v = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, threads, 0) == hipSuccess && n > 0 ? n : 1;
    cache.store(v, std::memory_order_relaxed);
  }
  return v;
}

bool timing_on();
void* timing_begin(int id, hipStream_t s);
void timing_end(void* token, hipStream_t s);
// Launch with optional event bracketing.
#define TFHE_TIMED(id, stream, ...)                  \
  do {                                               \
    void* tfhe_tok_ = ::tfhe::timing_begin(id, stream); \
    __VA_ARGS__;                                     \
    ::tfhe::timing_end(tfhe_tok_, stream);           \
  } while (0)

hipError_t load_small_launch(const ModConst* mods, const int32_t* in, uint32_t* out,
                             uint32_t limb_count, uint32_t batch, uint32_t n, hipStream_t s);

// ---- host-side number theory (plan.cpp)
bool is_prime_u32(uint32_t q);
ModConst make_modconst(uint32_t q);
uint32_t pow_mod(uint32_t b, uint64_t e, uint32_t q);
uint32_t inv_mod(uint32_t x, uint32_t q);
uint32_t default_psi(uint32_t q, uint32_t log_n);  // 0 if none

}  // namespace tfhe
