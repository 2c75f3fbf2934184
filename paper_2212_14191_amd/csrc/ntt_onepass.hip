// One-pass four-step NTT (Sec. IV-B/IV-C, Eq. 9 and Eq. 10) for N = N1 x 256,
// N = 2^12..2^15: the same two matrix-core stages as the two-pass kernels
// (ntt_fourstep.hip: the map n = 256 n1 + n2, k = k1 + N1 k2, byte-digit
// contractions, Montgomery fusion, twists), but a workgroup keeps whole
// polynomials in LDS, so each polynomial crosses HBM once in each direction
// instead of twice (the paper's Stages 1-5 as one pipeline per transform).
//
// Per polynomial: direct-to-LDS loads of the natural-order input; pass 1
// (the first stage over the columns of the P1 x S view) in place; pass 2
// (the second stage over its rows), whose results are held in registers
// until every wave has read its rows, then written into LDS in natural output
// order (position = pass-1 index + P1 x pass-2 index); 16-byte streaming
// stores.  For N <= 2^14 a workgroup has 4 waves and one polynomial buffer,
// so that two or three workgroups share a CU: one's loads and stores overlap
// the others' arithmetic (measured faster than one 8-wave workgroup that
// double-buffers: 1.2-1.25 x at 2^13 and 2^14).  A launch of no more
// polynomials than CUs has nothing to overlap and takes 8 waves at 2^13 and
// 2^14 (256 polynomials: 9.7 -> 8.7 and 17.4 -> 15.8 us when introduced, 7.7
// and 13.7 now; 16 waves at 2^14 had too few registers: 24.8).  At 2^15 the polynomial takes 128 KiB and one
// workgroup of 8 waves owns the CU.
//
// LDS layout: 1 KiB chunks of the polynomial in order; inside a chunk the
// 16-byte quads are XOR-swizzled (quad Q at Q ^ X, X a function of the chunk
// and of Q's bits 4-5, below 16), which the direct-to-LDS loads realise by
// choosing each lane's global address.  The constants make every access of
// both passes free of bank conflicts (64 banks; 16 lanes per 16-byte access,
// 64 per 4-byte access), verified by enumeration of the access patterns.
// The output order uses its own swizzle.
//
// The first pass's post-twist P(column, output) is split into a factor fixed
// per lane (Shoup form, or in the fusion after a matrix-core level B; staged in LDS, or read through the caches at 2^14
// where two workgroups' polynomials fill the LDS) and a factor per step
// (Montgomery form, in registers).
#include "fourstep_dev.hpp"

namespace tfhe {
namespace {

// Per (log N, direction): waves per workgroup of a large launch and the
// swizzle constants: input X = (a c + b (Q >> 4)) & 15; output
// X = (a c + b (Q >> sh)) & (2^sh - 1), with c the chunk and Q the quad.
template <int kLogN, bool kInv>
struct OpCfg;
#define TFHE_OPCFG(LN, INV, W, IA, IB, OA, OB, OS, PB)                      \
  template <>                                                              \
  struct OpCfg<LN, INV> {                                                  \
    static constexpr int waves = W;                                        \
    static constexpr uint32_t in_a = IA, in_b = IB, out_a = OA, out_b = OB; \
    static constexpr uint32_t out_sh = OS;                                 \
    static constexpr bool pb_lds = PB;                                     \
  };
TFHE_OPCFG(12, false, 4, 1, 4, 0, 1, 4, true)
TFHE_OPCFG(13, false, 4, 9, 4, 1, 1, 3, true)
TFHE_OPCFG(14, false, 4, 5, 4, 1, 4, 4, false)
TFHE_OPCFG(15, false, 8, 9, 4, 1, 4, 4, true)
TFHE_OPCFG(12, true, 4, 4, 1, 1, 0, 4, true)
TFHE_OPCFG(13, true, 4, 4, 1, 1, 0, 4, true)
TFHE_OPCFG(14, true, 4, 4, 1, 1, 0, 4, false)
TFHE_OPCFG(15, true, 8, 5, 4, 1, 0, 4, true)
#undef TFHE_OPCFG

template <uint32_t kA, uint32_t kB>
__device__ __forceinline__ uint32_t sw_in(uint32_t w) {
  const uint32_t c = w >> 8, Q = (w >> 2) & 63u;
  const uint32_t X = (kA * c + kB * (Q >> 4)) & 15u;
  return (c << 8) | ((Q ^ X) << 2) | (w & 3u);
}

template <uint32_t kA, uint32_t kB, uint32_t kSh>
__device__ __forceinline__ uint32_t sw_out(uint32_t w) {
  const uint32_t c = w >> 8, Q = (w >> 2) & 63u;
  const uint32_t X = (kA * c + kB * (Q >> kSh)) & ((1u << kSh) - 1u);
  return (c << 8) | ((Q ^ X) << 2) | (w & 3u);
}

// The value, opaque to the optimiser: address arithmetic derived from it is
// recomputed where it is used instead of being hoisted out of the
// polynomial loop, where dozens of precomputed LDS addresses would occupy
// registers for the whole kernel.
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

template <int kLogN, bool kInv, int W>
__global__ void __launch_bounds__((64 * W), (W <= 4 ? 2 : W / 4))
op_kernel(const FsTable tab) {
  using C = OpCfg<kLogN, kInv>;
  constexpr int N = 1 << kLogN, N1 = N >> 8;
  constexpr int kR1 = kInv ? 16 : N1 / 16, kR2 = kInv ? N1 / 16 : 16;
  constexpr int P1 = 16 * kR1, S = N / P1;   // pass 1: S columns of P1 points
  constexpr int Mt1 = 16 / kR1, Mt2 = 16 / kR2;
  constexpr int St1 = S / (4 * Mt1) / W, St2 = P1 / (4 * Mt2) / W;  // steps per wave
  constexpr int CH = N / 256 / W;  // 1 KiB chunks per wave and polynomial
  constexpr bool kUA = kInv;       // second-pass level-A index u = g + 4c
  static_assert(St1 >= 1 && St2 >= 1 && CH >= 1, "shape");
  // the step factor's lazy products stay below (2 - 2^{1 - St1}) q, so the
  // post-twist's input stays below 1.94 q (twist_digits)
  static_assert(St1 <= 4, "post-twist range");
  // the polynomial, then the limb's matrix-core operands and twists
  // (both passes) and the per-lane post-twist factors, staged once per limb
  // (the post-twist factors stay in global memory, read per polynomial
  // through the caches, where LDS must hold two workgroups' polynomials)
  constexpr bool kPbLds = C::pb_lds;
  constexpr int kTabOpA1 = N, kTabTw1 = kTabOpA1 + 1024, kTabOpA2 = kTabTw1 + 512;
  constexpr int kTabTw2 = kTabOpA2 + 1024, kTabPb = kTabTw2 + 512, kLdsWords = kTabPb + (kPbLds ? 2048 : 0);
  __shared__ __attribute__((aligned(16))) uint32_t buf[kLdsWords];

  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i16 = lane & 15, g = lane >> 4;
  touch(tab.count, tab.tab_op, tab.begin[7], tab.u[0].in, tab.u[0].batch_inv, tab.u[0].twist);
  const uint32_t p_begin = blockIdx.x * tab.share + min(blockIdx.x, tab.extra);
  const uint32_t p_end = (blockIdx.x + 1) * tab.share + min(blockIdx.x + 1, tab.extra);
  if (p_begin >= p_end) return;

  // running unit indices of the load and compute walks
  uint32_t kf = find_unit(tab.begin, tab.count, p_begin), kc = kf;
  // direct-to-LDS loads of polynomial p: chunk c = wave + k W;
  // LDS slot L of the chunk receives natural quad L ^ X(c, L >> 4)
  auto issue_load = [&](uint32_t p) {
    const Item it = locate(tab, p, kf);
    const uint32_t* src = tab.u[it.unit].in + it.poly_base;
    const uint32_t al = (uint32_t)opaque(lane);
#pragma unroll
    for (int k = 0; k < CH; ++k) {
      const uint32_t c = wave + k * W;
      const uint32_t X = (C::in_a * c + C::in_b * (al >> 4)) & 15u;
      const uint32_t* gp = src + c * 256 + 4 * (al ^ X);
      const uint32_t lds_addr = (uint32_t)(uintptr_t)(lds_void_t*)(buf + c * 256);
      asm volatile(
          "s_mov_b32 m0, %0\n\t"
          "global_load_lds_dwordx4 %1, off nt"
          :
          : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(gp)
          : "memory", "m0");
    }
  };
  issue_load(p_begin);
  // direct-to-LDS loads of a limb's tables, 1 KiB each: level-A operands and
  // twist of both passes, post-twist (copies through registers, table after
  // table, took 1 us each on a launch's first polynomial)
  constexpr int kNt = kPbLds ? 20 : 12;
  const uint32_t lane16 = 16 * lane;
  auto issue_tables = [&](const unsigned char* base, const uint2* twist) {
#pragma unroll
    for (int k = 0; k < (kNt + W - 1) / W; ++k) {
      const int ch = wave + k * W;
      if (ch < kNt) {
        const uint64_t at = ch < 4    ? ch * 1024
                            : ch < 6  ? offsetof(PassTables, twist) + (ch - 4) * 1024
                            : ch < 10 ? tab.tab_op + (ch - 6) * 1024
                            : ch < 12 ? tab.tab_op + offsetof(PassTables, twist) + (ch - 10) * 1024
                                      : tab.tab_op + offsetof(OnePassTables, post_b) + (ch - 12) * 1024;
        const unsigned char* src =
            twist && ch >= 10 && ch < 12 ? (const unsigned char*)twist + (ch - 10) * 1024 : base + at;
        const uint32_t lds_addr = (uint32_t)(uintptr_t)(lds_void_t*)(buf + kTabOpA1 + ch * 256);
        asm volatile(
            "s_mov_b32 m0, %0\n\t"
            "global_load_lds_dwordx4 %1, %2"
            :
            : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(lane16), "s"(src)
            : "memory", "m0");
      }
    }
  };

  // per-limb values in registers (the rest of the limb's tables is in LDS)
  const void* cur = nullptr;  // whose tables are staged: the limb's, with the unit's twist if it has one
  const uint2* pb_src = nullptr;  // the limb's post-twist factors (global)
  Red R{};
  uint2 lb1[4], lb2[16];  // level-B constants (uniform: scalar registers)
  // post-twist step factors: the wave's first step's, and the ratio between
  // consecutive steps of a wave (the factor is geometric in the step index)
  uint32_t pa0[4], pad[4];

  for (uint32_t p = p_begin; p < p_end; ++p) {
    const Item it = locate(tab, p, kc);
    const FourStepLimb* limb = tab.u[it.unit].limbs + it.limb;
    const uint2* const twist = kInv ? tab.u[it.unit].twist : nullptr;
    const void* const key = twist ? (const void*)(twist + it.limb * 256) : limb;
    if (key != cur) {
      // rare (a few times per workgroup), and every wave is past the
      // previous polynomial's last barrier, so the staged tables are free
      const auto* L = (const_as FourStepLimb*)limb;
      const unsigned char* const base = tab.u[it.unit].tables + it.limb * tab.tab_stride;
      const OnePassTables* O = (const OnePassTables*)(base + tab.tab_op);
      issue_tables(base, twist ? twist + it.limb * 256 : nullptr);
      R = make_red(L->q, L->qneg);
      pb_src = &O->post_b[0][0][0][0];
      const v4u a0 = *(const v4u*)&O->post_a[wave][lane][0], ad = *(const v4u*)&O->post_a[St1 > 1 ? W : wave][lane][0];
      const auto* b1 = (const_as uint32_t*)(base + offsetof(PassTables, lb));
      const auto* b2 = (const_as uint32_t*)((const unsigned char*)O + offsetof(PassTables, lb));
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (kR1 < 16) lb1[j] = make_uint2(b1[2 * j], b1[2 * j + 1]);
        pa0[j] = a0[j];
        pad[j] = ad[j];
      }
      if (kR2 < 16) {
#pragma unroll
        for (int i = 0; i < 16; ++i) lb2[i] = make_uint2(b2[2 * i], b2[2 * i + 1]);
      }
      cur = key;
    }
    // this wave's loads of the polynomial and of the tables (the builtin tells
    // the compiler as well)
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    lds_barrier();  // the polynomial is in LDS (every wave's loads landed)

    const uint32_t q = R.q;
    const v4i bias = {(int)q, (int)q, (int)q, (int)q};
    const v4i zero = {0, 0, 0, 0};

    // ---- pass 1: columns, in place.  Lane (i, g) reads row
    // kR1 (4g + c) + i % kR1 of quad Q0 + i / kR1 (the four sets are the
    // quad's four columns) and writes output s + 16 t of column quad Q0 + m.
    {
      v4i opA1[4];
      uint2 tw1[4], pb[4][4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        opA1[j] = *(const v4i*)(buf + kTabOpA1 + (j * 64 + lane) * 4);
        tw1[j] = *(const uint2*)(buf + kTabTw1 + (lane * 4 + j) * 2);
#pragma unroll
        for (int sg = 0; sg < 4; ++sg)
          pb[j][sg] = kPbLds ? *(const uint2*)(buf + kTabPb + (((sg * 2 + j / 2) * 64 + lane) * 2 + j % 2) * 2)
                             : pb_src[((sg * 2 + j / 2) * 64 + lane) * 2 + j % 2];
      }
      uint32_t pa[4] = {pa0[0], pa0[1], pa0[2], pa0[3]};
#pragma unroll
      for (int st = 0; st < St1; ++st) {
        const int Q0 = (wave + st * W) * Mt1;
        const int ai = opaque(i16), ag = opaque(g);  // for addresses
        if (st > 0) {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            pa[j] = kR1 == 16 ? (uint32_t)mont_signed((int)pa[j], (int)pad[j], R) : mont_mul_lazy(pa[j], pad[j], R);
        }
        uint4 rows[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int row = kR1 * (4 * ag + c) + ai % kR1, quad = Q0 + ai / kR1;
          rows[c] = *(const uint4*)(buf + sw_in<C::in_a, C::in_b>(row * S + 4 * quad));
        }
        // only moduli above 0x7F7F7F7F (uniform) need the window's correction
        if (q > 0x7F7F7F7Fu) {
#pragma unroll
          for (int c = 0; c < 4; ++c)
            rows[c] = make_uint4(residue_digits_big(rows[c].x, q), residue_digits_big(rows[c].y, q),
                                 residue_digits_big(rows[c].z, q), residue_digits_big(rows[c].w, q));
        } else {
#pragma unroll
          for (int c = 0; c < 4; ++c)
            rows[c] = make_uint4(residue_digits(rows[c].x), residue_digits(rows[c].y), residue_digits(rows[c].z),
                                 residue_digits(rows[c].w));
        }
        const Red M = local(R);
        // (nor the twists' sign extensions from another step)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          asm volatile("" : "+v"(tw1[j].x), "+v"(tw1[j].y));
          if (kR1 == 16) {
#pragma unroll
            for (int sg = 0; sg < 4; ++sg) asm volatile("" : "+v"(pb[j][sg].x), "+v"(pb[j][sg].y));
          }
        }
        uint32_t o[4][4];  // [register j][set]
        uint2 rj[4];
        if (kR1 == 8) {
#pragma unroll
          for (int j = 0; j < 4; ++j) rj[j] = (g & 1) ? lb1[j] : lb1[0];
        }
#pragma unroll
        for (int sg = 0; sg < 4; ++sg) {
          v4i x;
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            x[c] = (int)(sg == 0 ? rows[c].x : sg == 1 ? rows[c].y : sg == 2 ? rows[c].z : rows[c].w);
          }
          const v4i a0 = mfma(x, opA1[0], zero);
          const v4i a1 = mfma(x, opA1[1], zero);
          const v4i a2 = mfma(x, opA1[2], zero);
          const v4i a3 = mfma(x, opA1[3], zero);
          uint32_t y[4];
          if (kR1 == 16) {
            v4i z;
#pragma unroll
            for (int j = 0; j < 4; ++j)
              z[j] = (int)residue_digits(fuse_twist(a0[j], a1[j], a2[j], a3[j], tw1[j], M));
            // level B (only the inverse's 256-point stage here): the same
            // symmetric matrix, unscaled, so opB equals opA
            const v4i b0 = mfma(opA1[0], z, zero);
            const v4i b1 = mfma(opA1[1], z, zero);
            const v4i b2 = mfma(opA1[2], z, zero);
            const v4i b3 = mfma(opA1[3], z, zero);
#pragma unroll
            for (int j = 0; j < 4; ++j)
              y[j] = (uint32_t)mont_signed(fuse_twist(b0[j], b1[j], b2[j], b3[j], pb[j][sg], M), (int)pa[j], M);
          } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
              y[j] = wrap_signed(fuse_twist(a0[j], a1[j], a2[j], a3[j], tw1[j], M), q);
            level_b<kR1>(y, lb1, rj, g, q);
          }
#pragma unroll
          for (int j = 0; j < 4; ++j)
            o[j][sg] = kR1 == 16 ? residue_digits(y[j]) : twist_digits(mont_mul_lazy(y[j], pa[j], M), pb[j][sg], M);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          int m, t;
          lane_out<kR1>(ag, j, m, t);
          const int row = ai + 16 * t;
          *(uint4*)(buf + sw_in<C::in_a, C::in_b>(row * S + 4 * (Q0 + m))) =
              make_uint4(o[j][0], o[j][1], o[j][2], o[j][3]);
        }
      }
    }
    lds_barrier();

    // ---- pass 2: rows.  Step rows R0 .. R0 + 4 Mt2 - 1; set sg and tile
    // vector m take row R0 + 4m + sg; lane (i, g), dword c reads element
    // kR2 u + i % kR2 (u = 4g + c, or g + 4c for the inverse).
    uint4 res[St2][4];
    {
      const Red M = local(R);
      v4i opA2[4];
      uint2 tw2[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        opA2[j] = *(const v4i*)(buf + kTabOpA2 + (j * 64 + lane) * 4);
        tw2[j] = *(const uint2*)(buf + kTabTw2 + (lane * 4 + j) * 2);
      }
      uint2 rj[4], pf[4];  // level-B multipliers; factor of output t (lb2[8 + t])
      if (kR2 < 16) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          int m, t;
          lane_out<kR2>(g, j, m, t);
          pf[j] = lb2[8 + t];
          rj[j] = (g & 1) ? lb2[j] : lb2[0];
        }
      }
      // the first step's 16 word addresses; a step further lies kStep words on,
      // whole chunks that leave the swizzle as it is (computed per step, the
      // addresses took a quarter of this pass's instructions)
      constexpr int kStep = W * 4 * Mt2 * S;
      static_assert(kStep % 256 == 0 && C::in_a * (kStep / 256) % 16 == 0, "step against swizzle");
      int at[4][4];
      const int ai = opaque(i16), ag = opaque(g);
#pragma unroll
      for (int sg = 0; sg < 4; ++sg)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int u = kUA ? ag + 4 * c : 4 * ag + c;
          const int row = wave * 4 * Mt2 + 4 * (ai / kR2) + sg, e = kR2 * u + ai % kR2;
          at[sg][c] = sw_in<C::in_a, C::in_b>(row * S + e);
        }
#pragma unroll
      for (int st = 0; st < St2; ++st) {
#pragma unroll
        for (int sg = 0; sg < 4; ++sg) {
          v4i x;
#pragma unroll
          for (int c = 0; c < 4; ++c) x[c] = (int)buf[at[sg][c] + st * kStep];
          const v4i a0 = mfma(x, opA2[0], zero);
          const v4i a1 = mfma(x, opA2[1], zero);
          const v4i a2 = mfma(x, opA2[2], zero);
          const v4i a3 = mfma(x, opA2[3], zero);
          uint32_t y[4];
          if (kR2 == 16) {
            v4i z;
#pragma unroll
            for (int j = 0; j < 4; ++j)
              z[j] = (int)residue_digits(fuse_twist(a0[j], a1[j], a2[j], a3[j], tw2[j], M));
            const v4i b0 = mfma(opA2[0], z, bias);  // level B: the same symmetric matrix
            const v4i b1 = mfma(opA2[1], z, zero);
            const v4i b2 = mfma(opA2[2], z, bias);
            const v4i b3 = mfma(opA2[3], z, zero);
#pragma unroll
            for (int j = 0; j < 4; ++j) y[j] = reduce_once(fuse_redc(b0[j], b1[j], b2[j], b3[j], M), q);
          } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
              y[j] = wrap_signed(fuse_twist(a0[j], a1[j], a2[j], a3[j], tw2[j], M), q);
            level_b<kR2>(y, lb2, rj, g, q);
#pragma unroll
            for (int j = 0; j < 4; ++j) y[j] = mul_shoup(y[j], pf[j].x, pf[j].y, q);
          }
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            if (sg == 0) res[st][j].x = y[j];
            else if (sg == 1) res[st][j].y = y[j];
            else if (sg == 2) res[st][j].z = y[j];
            else res[st][j].w = y[j];
          }
        }
      }
    }
    lds_barrier();  // every wave has read its rows
#pragma unroll
    for (int st = 0; st < St2; ++st) {
      const int R0 = (wave + st * W) * 4 * Mt2;
      const int ai = opaque(i16), ag = opaque(g);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        int m, t;
        lane_out<kR2>(ag, j, m, t);
        const uint32_t pos = R0 + 4 * m + P1 * (ai + 16 * t);
        *(uint4*)(buf + sw_out<C::out_a, C::out_b, C::out_sh>(pos)) = res[st][j];
      }
    }
    lds_barrier();

    // ---- store: natural order, whole 1 KiB chunks per instruction; the next
    // polynomial is loaded once every wave has read its chunks
    const int al = opaque(lane);
    uint32_t* const dst = tab.u[it.unit].out + it.poly_base;
#pragma unroll
    for (int k = 0; k < CH; ++k) {
      const uint32_t c = wave + k * W;
      const uint4 v = *(const uint4*)(buf + sw_out<C::out_a, C::out_b, C::out_sh>(c * 256 + 4 * al));
      __builtin_nontemporal_store(*(const v4u*)&v, (v4u*)(dst + c * 256 + 4 * al));
    }
    lds_barrier();
    if (p + 1 < p_end) issue_load(p + 1);
  }
}

template <int kLogN, bool kInv, int W>
void op_launch_w(const tfhe_ntt_plan_s* p, FsTable t, hipStream_t s) {
  static std::atomic<int> occ{0};
  const uint32_t w =
      p->fs_wg_per_cu ? p->fs_wg_per_cu : (uint32_t)occupancy_cached(occ, op_kernel<kLogN, kInv, W>, 64 * W);
  const uint32_t grid = std::min(std::max(1u, p->num_cus * w), t.total);
  t.share = t.total / grid;
  t.extra = t.total % grid;
  TFHE_TIMED(K_OP, s, hipLaunchKernelGGL((op_kernel<kLogN, kInv, W>), dim3(grid), dim3(64 * W), 0, s, t));
}

template <int kLogN, bool kInv>
void op_launch(const tfhe_ntt_plan_s* p, const FsTable& t, hipStream_t s) {
  // no more polynomials than CUs: nothing else runs beside a workgroup
  if constexpr (kLogN == 13 || kLogN == 14) {
    if (t.total <= p->num_cus) return op_launch_w<kLogN, kInv, 8>(p, t, s);
  }
  op_launch_w<kLogN, kInv, OpCfg<kLogN, kInv>::waves>(p, t, s);
}

}  // namespace

bool op_supported(uint32_t log_n) { return log_n >= 12 && log_n <= 15; }

// One launch over every unit of the table (same N and direction).
hipError_t op_run(const tfhe_ntt_plan_s* p, bool inverse, const FsTable& t, hipStream_t s) {
  if (t.total == 0) return hipSuccess;
  switch (p->log_n * 2 + (inverse ? 1 : 0)) {
    case 24: op_launch<12, false>(p, t, s); break;
    case 25: op_launch<12, true>(p, t, s); break;
    case 26: op_launch<13, false>(p, t, s); break;
    case 27: op_launch<13, true>(p, t, s); break;
    case 28: op_launch<14, false>(p, t, s); break;
    case 29: op_launch<14, true>(p, t, s); break;
    case 30: op_launch<15, false>(p, t, s); break;
    case 31: op_launch<15, true>(p, t, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace tfhe
