// Basis conversion (ModUp / ModDown Conv, Sec. II-B) fused with the first
// pass of the forward four-step transform of its results (ntt_fourstep.hip):
//   x_t = sum_r y_r C[t][r] mod m_t
// (y_r in [0, q_r) the limb r of the input, already times the conversion's
// constant of r: the inverse transform that wrote it has folded that in),
// then the N1-point stage over the columns of x_t and its post-twist, for
// every target limb t.  The converted planes (three times the inputs' bytes
// in ModUp and ModDown at the benchmark's shape) are never written or read.
// RESCALE's broadcast transform is the same kernel without the conversion:
// the one input plane enters every limb's transform as it is.
//
// A wave takes 1024 coefficients: the N1 rows of a few columns.  It loads them
// from every input plane straight into registers, in the lane layout of the
// first pass's level A (16 coefficients of each input: 128 registers for
// eight inputs), and computes every target from there with no data exchanged
// between waves: one multiply-add per input and coefficient, then the matrix
// cores.  What changes per target is the limb's tables (operands, twist,
// post-twist: 14 or 18 KiB), which the waves of a workgroup read from an LDS
// copy that is loaded one target ahead.  Bound by the vector ALUs (32-37
// instructions per coefficient and target, two waves per SIMD).
//
// Measured for 64 pairs at N = 2^16, level 24, as a kernel of its own that
// wrote the converted planes and a plain first pass -> here: ModUp 0.31 + 0.49
// -> 0.51 ms, ModDown 0.20 + 0.34 -> 0.34 ms, RESCALE's first pass 0.34 ->
// 0.21 ms.  The same conversion on the matrix cores (byte digits of y against
// byte digits of the constants) takes fewer vector instructions but 0.60 ms
// for ModUp (0.53 here then): its operands go through LDS and the matrix cores' cycles are
// taken from the same SIMD.
//
// Exactness: the inputs enter as y_r - 2^30 in [-2^30, 2^30) and the
// constants as the representatives of C 2^32 in [-m/2, m/2), so
// |sum| <= 8 2^30 m/2 = m 2^32; an initial value of m 2^32 plus the offsets'
// share (2^30 sum_r C 2^32 mod m) makes it a non-negative number below
// (2m + 1) 2^32 < 2^64 (m < 2^31).  One conditional subtraction of m 2^32
// and one Montgomery step leave x_t in [0, 2m], which enters the balanced
// digits as x_t - m.
#include <algorithm>

#include "fourstep_dev.hpp"

namespace tfhe {
namespace {

// Inputs of one launch, by value (a kernel argument).  Item = one workgroup:
// `chunk` consecutive targets of one batch element and column block; the
// items of unit k are item_begin[k] .. item_begin[k + 1] - 1.
constexpr int kMaxCvUnits = 40;
struct CvUnit {
  const uint32_t* in;      // input r, element b at in + (r batch + b) N, quad-tiled or not
  uint32_t* out;           // position pos, element b at out + (pos batch + b) N (tiled)
  const CvTarget* tgt;     // [plan limb]
  uint32_t batch, nin, targets, d0, nd, level, tiled, chunks;
  uint32_t chunks_inv, batch_inv;  // div_inv of 8 chunks and of batch
};
struct CvTable {
  uint32_t count, L, chunk;
  const unsigned char* blob;     // forward four-step tables of limb l at blob + l per
  uint64_t per, op_off;          // op_off: the limb's OnePassTables
  const ModConst* mods;          // [plan limb]
  uint32_t item_begin[kMaxCvUnits + 1];
  CvUnit u[kMaxCvUnits];
};
static_assert(sizeof(CvTable) <= 4096, "a CvTable is passed as a kernel argument");

// Workgroups of W = 4 waves of 1024 coefficients.  With eight inputs two of them
// share a CU (256 registers per lane): one's input loads, table copies and
// barriers run under the other's arithmetic (one 8-wave workgroup per CU took
// 0.57 instead of 0.54 ms for ModUp of 64 pairs at N = 2^16, level 24).  The
// plain input leaves room for 16 waves per CU, as two workgroups of 8 (but see
// cv_launch_w for small launches).
template <int kR, int kIn, int W>
struct CvShape {
  static constexpr int waves = W, threads = 64 * waves;
  static constexpr int blocks = 4 * kR / waves;  // items per polynomial: N / (1024 waves)
  static constexpr int per_cu = kIn == 8 ? 2 : kIn == 4 ? 3 : 16 / waves;  // workgroups
  // tables of one target in LDS: opA, opB (kR = 16), twist, post_b
  static constexpr int tw = kR == 16 ? 2048 : 1024, pb = tw + 512, tab = pb + 2048;
};

// Which lane group holds output t of tile vector m (the inverse of lane_out).
template <int kR>
__device__ __forceinline__ int group_of(int m, int t) {
  return kR == 16 ? t >> 2 : kR == 8 ? 2 * m + (t & 1) : kR == 4 ? m : kR == 2 ? m >> 1 : m >> 2;
}

// kIn: inputs held in registers (0: one plane, no conversion).
template <int kR, int kIn, int W>
__global__ void __launch_bounds__((CvShape<kR, kIn, W>::threads), (kIn == 0 && kR > 1 ? 4 : 2))
cv_pass(const CvTable tab) {
  using S = CvShape<kR, kIn, W>;
  constexpr int kPlanes = kIn == 0 ? 1 : kIn, Mt = 16 / kR;
  __shared__ __attribute__((aligned(16))) uint32_t lds[1024 * S::waves + 2 * S::tab];
  uint32_t* const tabs = lds + 1024 * S::waves;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i16 = lane & 15, g = lane >> 4;

  touch(tab.count, tab.mods, tab.item_begin[7], tab.u[0].in, tab.u[0].batch, tab.u[0].batch_inv);
  // item -> (unit, chunk, column block, element)
  const uint32_t k = find_unit(tab.item_begin, tab.count, blockIdx.x);
  const CvUnit& U = tab.u[k];
  const uint32_t batch = U.batch, d0 = U.d0, nd = U.nd, level = U.level, L = tab.L;
  // (the chunks of one block and element are 8 workgroups apart: on one XCD,
  // whose L2 then serves the inputs to all of them)
  const uint32_t per = S::blocks * batch, full = per & ~7u, chunks = U.chunks;
  uint32_t local = blockIdx.x - tab.item_begin[k], ch = 0, at = local;
  if (chunks > 1) {
    if (local < full * chunks) {
      const uint32_t grp = div_by(local, 8 * chunks, U.chunks_inv), r = local - grp * 8 * chunks;
      ch = r / 8;
      at = 8 * grp + r % 8;
    } else {
      local -= full * chunks;
      while (local >= per - full) local -= per - full, ++ch;
      at = full + local;
    }
  }
  const uint32_t blk = div_by(at, batch, U.batch_inv), b = at - blk * batch, u0 = ch * tab.chunk;
  const uint32_t u1 = min(u0 + tab.chunk, U.targets);
  const uint32_t step = blk * S::waves + wave, c0w = step * 4 * Mt;  // this wave's columns c0w .. + 4 Mt - 1
  constexpr uint32_t log_n = 12 + (kR == 16 ? 4 : kR == 8 ? 3 : kR == 4 ? 2 : kR == 2 ? 1 : 0);
  const uint64_t plane = (uint64_t)batch << log_n;
  auto pos_of = [&](uint32_t u) { return u < d0 ? u : u + nd; };
  auto limb_of = [&](uint32_t pos) { return pos < level ? pos : L + pos - level; };

  // a limb's tables into LDS buffer `buf`, 1 KiB per load: opA (opB), twist,
  // then post_b; this wave's loads' offsets in the limb's tables
  constexpr int n1 = kR == 16 ? 10 : 6, nt = n1 + 8, rounds = (nt + S::waves - 1) / S::waves;
  uint32_t tab_off[rounds];
#pragma unroll
  for (int c = 0; c < rounds; ++c) {
    const int ch = c * S::waves + wave;
    tab_off[c] = ch < n1 ? (kR == 16 || ch < 4 ? ch : ch + 4) * 1024
                         : (uint32_t)tab.op_off + offsetof(OnePassTables, post_b) + (ch - n1) * 1024;
  }
  const uint32_t lane16 = 16 * lane;
  auto issue_tables = [&](uint32_t limb, int buf) {
    const unsigned char* base = tab.blob + limb * tab.per;
#pragma unroll
    for (int c = 0; c < rounds; ++c) {
      const int ch = c * S::waves + wave;
      if (ch < nt) {
        const uint32_t lds_addr = (uint32_t)(uintptr_t)(lds_void_t*)(tabs + buf * S::tab + ch * 256);
        asm volatile(
            "s_mov_b32 m0, %0\n\t"
            "global_load_lds_dwordx4 %1, %2"
            :
            : "s"(__builtin_amdgcn_readfirstlane(lds_addr)), "v"(lane16), "s"(base + tab_off[c])
            : "memory", "m0");
      }
    }
  };
  auto post_a = [&](uint32_t limb) {
    const unsigned char* op = tab.blob + limb * tab.per + tab.op_off + offsetof(OnePassTables, post_a);
    return *(const v4u*)(op + step * 1024 + lane16);
  };

  uint32_t limb = limb_of(pos_of(u0));
  v4u pa = post_a(limb);
  issue_tables(limb, 0);
  // a target's constants (scalar loads; fetched one target ahead)
  auto target = [&](uint32_t limb) {
    CvTarget t{};
    if (kIn) {
      const auto* p = (const_as CvTarget*)U.tgt + limb;
#pragma unroll
      for (int r = 0; r < kIn; ++r) t.c[r] = p->c[r];
      t.init = p->init;
      t.q = p->q;
      t.qneg = p->qneg;
    } else {
      const auto* p = (const_as ModConst*)tab.mods + limb;
      t.q = p->q;
      t.qneg = p->qneg;
    }
    return t;
  };
  CvTarget now = target(limb);

  // ---- the inputs: y[r][4c + i] is column i of quad c0w / 4 + i16 / kR in row
  // kR (4g + c) + i16 % kR.  In natural order a load covers, per row, 4 Mt
  // columns (128 bytes at kR = 2); with kR >= 8, where that would be 32 or 16
  // bytes, the producer writes quad by quad ([quad][row][4]): 256-byte runs.
  uint32_t y[kPlanes][16];
  {
    const uint32_t row = kR * 4 * g + i16 % kR, quad = c0w / 4 + i16 / kR;
    const uint32_t rs = U.tiled ? 4 : 256, qs = U.tiled ? 64 * kR : 4;
    const uint32_t* src = U.in + ((uint64_t)b << log_n) + row * rs + quad * qs;
#pragma unroll
    for (int r = 0; r < kPlanes; ++r) {
      // (an input that is not there has zero constants: the last one again,
      // since a branch around its loads would wait for them before the next)
      const uint64_t at = min((uint32_t)r, U.nin - 1) * plane;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const v4u w = *(const v4u*)(src + at + c * kR * rs);
#pragma unroll
        for (int i = 0; i < 4; ++i) y[r][4 * c + i] = w[i];
      }
    }
    if (kIn) {
#pragma unroll
      for (int r = 0; r < kPlanes; ++r)
#pragma unroll
        for (int e = 0; e < 16; ++e) y[r][e] -= 1u << 30;
    }
  }

  // the first tables too; the builtin tells the compiler so, which otherwise
  // waits in the target loop (for the stores as well) before using pa
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  uint32_t* const gather = lds + wave * 1024;
  uint32_t* const out = U.out + ((uint64_t)b << log_n) + c0w * 16;
  int buf = 0;
  for (uint32_t u = u0; u < u1; ++u, buf ^= 1) {
    const uint32_t pos = pos_of(u);
    // the tables were issued before the last target's 4 stores (the first
    // target's have been awaited)
    if (u != u0) wait_vmcnt<4>();
    lds_barrier();  // tables complete; every wave is done with the other buffer
    v4u pa_next = pa;
    uint32_t limb_next = limb;
    CvTarget next = now;
    if (u + 1 < u1) {
      limb_next = limb_of(pos_of(u + 1));
      next = target(limb_next);
      pa_next = post_a(limb_next);
      issue_tables(limb_next, buf ^ 1);
    }
    const uint32_t* const T = tabs + buf * S::tab;
    const Red R = make_red(now.q, now.qneg);
    const uint32_t q = R.q;
    const uint64_t init = now.init;
    uint2 lb[4], rj[4];  // kR < 16: rho^0..rho^3; register j's multiplier (kR = 8)
    if (kR < 16) {
      const auto* p = (const_as uint32_t*)(tab.blob + limb * tab.per + offsetof(PassTables, lb));
#pragma unroll
      for (int j = 0; j < 4; ++j) lb[j] = make_uint2(p[2 * j], p[2 * j + 1]);
#pragma unroll
      for (int j = 0; j < 4; ++j) rj[j] = (g & 1) ? lb[j] : lb[0];
    }
    // The inputs are kept opaque to the compiler from target to target: it
    // would otherwise keep their sign extensions in registers as well.
    if (kIn) {
#pragma unroll
      for (int r = 0; r < kPlanes; ++r)
#pragma unroll
        for (int e = 0; e < 16; ++e) asm volatile("" : "+v"(y[r][e]));
    }

    auto body = [&](auto big_q) {
      constexpr bool kBigQ = decltype(big_q)::value;
      v4i opA[4], opB[4];
      uint2 tw[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        opA[j] = *(const v4i*)(T + (j * 64 + lane) * 4);
        if (kR == 16) opB[j] = *(const v4i*)(T + 1024 + (j * 64 + lane) * 4);
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const v4u w = *(const v4u*)(T + S::tw + (lane * 2 + h) * 4);
        tw[2 * h] = make_uint2(w[0], w[1]);
        tw[2 * h + 1] = make_uint2(w[2], w[3]);
      }
      const v4i zero = {0, 0, 0, 0};
#pragma unroll
      for (int sg = 0; sg < 4; ++sg) {
        v4i x;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          if (kIn) {
            uint64_t acc = init;
#pragma unroll
            for (int r = 0; r < kPlanes; ++r) acc += (uint64_t)((int64_t)(int32_t)y[r][4 * c + sg] * now.c[r]);
            const uint32_t hi = (uint32_t)(acc >> 32);
            acc = ((uint64_t)min(hi, hi - q) << 32) | (uint32_t)acc;
            const uint32_t m = (uint32_t)acc * R.qneg;
            const uint32_t v = (uint32_t)(((uint64_t)m * q + acc) >> 32);  // [0, 2q]
            x[c] = (int)(kBigQ ? residue_digits_big(reduce_once(v, q), q) : (v + R.cq) ^ 0x80808080u);
          } else {
            x[c] = (int)residue_digits_big(y[0][4 * c + sg], q);
          }
        }
        const v4i a0 = mfma(x, opA[0], zero);
        const v4i a1 = mfma(x, opA[1], zero);
        const v4i a2 = mfma(x, opA[2], zero);
        const v4i a3 = mfma(x, opA[3], zero);
        // post-twist: the lane's factor (after a matrix-core level B in its
        // fusion, else Shoup) and the step's (Montgomery)
        const v4u pbv[2] = {*(const v4u*)(T + S::pb + ((sg * 2) * 64 + lane) * 4),
                            *(const v4u*)(T + S::pb + ((sg * 2 + 1) * 64 + lane) * 4)};
        auto pb = [&](int j) { return make_uint2(pbv[j / 2][2 * (j % 2)], pbv[j / 2][2 * (j % 2) + 1]); };
        uint32_t d[4];
        if (kR == 16) {
          v4i zd;
#pragma unroll
          for (int j = 0; j < 4; ++j) zd[j] = (int)residue_digits(fuse_twist(a0[j], a1[j], a2[j], a3[j], tw[j], R));
          const v4i b0 = mfma(opB[0], zd, zero);
          const v4i b1 = mfma(opB[1], zd, zero);
          const v4i b2 = mfma(opB[2], zd, zero);
          const v4i b3 = mfma(opB[3], zd, zero);
#pragma unroll
          for (int j = 0; j < 4; ++j)
            d[j] = residue_digits(mont_signed(fuse_twist(b0[j], b1[j], b2[j], b3[j], pb(j), R), (int)pa[j], R));
        } else {
          uint32_t z[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) z[j] = wrap_signed(fuse_twist(a0[j], a1[j], a2[j], a3[j], tw[j], R), q);
          level_b<kR>(z, lb, rj, g, q);
#pragma unroll
          for (int j = 0; j < 4; ++j) d[j] = twist_digits(mont_mul_lazy(z[j], pa[j], R), pb(j), R);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          int m, t;
          lane_out<kR>(g, j, m, t);
          gather[t * (1024 / kR) + m * 64 + 16 * (sg ^ g) + i16] = d[j];
        }
      }
    };
    if (kIn && q > 0x7F7F7F7Fu) body(std::true_type{});
    else body(std::false_type{});

    // this wave's runs (a wave's LDS accesses complete in order; the
    // compiler fence keeps the 16-byte reads after the 4-byte writes): word f
    // of the wave's 1024 is word f % (1024 / kR) of output block t = f / (1024 / kR)
    asm volatile("" ::: "memory");
    uint32_t* const dst = out + pos * plane;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int f = 256 * j + 4 * lane, t = f / (1024 / kR), w = f % (1024 / kR);
      const int m = w / 64, cw = (w % 64) / 16;
      const v4u v = *(const v4u*)(gather + t * (1024 / kR) + m * 64 + 16 * (cw ^ group_of<kR>(m, t)) + w % 16);
      __builtin_nontemporal_store(v, (v4u*)(dst + t * 4096 + w));
    }
    asm volatile("" ::: "memory");
    pa = pa_next;
    limb = limb_next;
    now = next;
  }
}

template <int kR, int kIn, int W>
hipError_t cv_launch_w(const tfhe_ntt_plan_s* p, CvTable& t, hipStream_t s) {
  using S = CvShape<kR, kIn, W>;
  // Targets per workgroup: more of them share one load of the inputs, fewer
  // fill the CUs.  Loading the inputs takes about as long as two targets; the
  // workgroups run in rounds of per_cu per CU.
  uint32_t most = 1;
  for (uint32_t k = 0; k < t.count; ++k) most = std::max(most, t.u[k].targets);
  auto items_of = [&](const CvUnit& u, uint32_t c) { return (uint64_t)((u.targets + c - 1) / c) * S::blocks * u.batch; };
  const uint64_t resident = (uint64_t)p->num_cus * S::per_cu;
  uint64_t best = ~0ull;
  for (uint32_t c = 1; c <= most; ++c) {
    uint64_t items = 0;
    for (uint32_t k = 0; k < t.count; ++k) items += items_of(t.u[k], c);
    const uint64_t cost = (items + resident - 1) / resident * (2 + c);
    if (cost <= best) best = cost, t.chunk = c;
  }
  uint64_t items = 0;
  for (uint32_t k = 0; k < t.count; ++k) {
    t.item_begin[k] = (uint32_t)items;
    t.u[k].chunks = (t.u[k].targets + t.chunk - 1) / t.chunk;
    t.u[k].chunks_inv = div_inv(8 * t.u[k].chunks);
    t.u[k].batch_inv = div_inv(t.u[k].batch);
    items += items_of(t.u[k], t.chunk);
  }
  if (items >= (1ull << 31)) return hipErrorInvalidValue;
  t.item_begin[t.count] = (uint32_t)items;
  TFHE_TIMED(K_CONV_PASS1, s,
             hipLaunchKernelGGL((cv_pass<kR, kIn, W>), dim3((uint32_t)items), dim3(S::threads), 0, s, t));
  return hipGetLastError();
}

// Without a conversion, workgroups of 8 waves share one copy of the tables among
// more of them; but at N = 2^13 and 2^14 they took longer to start than the
// plain first pass that this kernel replaced, and a launch of no more than two
// 4-wave workgroups per CU is over after one of each (whole RESCALE calls, us, 8
// waves : 4, N = 2^14: 2 polynomials 22.8 : 21.9, 32 24.3 : 23.1, 128 27.8 :
// 28.1 / 27.8 : 27.6, 224 32.8 : 34.3, 1472 98 : 101; the pass itself 6.3 : 5.2
// for 2, plain 5.1; N = 2^13: 32 19.1 : 18.4, 480 46.1 : 48.7; N = 2^15 not
// clearly either way, 2^16 slower).
template <int kR, int kIn>
hipError_t cv_launch(const tfhe_ntt_plan_s* p, CvTable& t, hipStream_t s) {
  if constexpr (kIn == 0 && (kR == 2 || kR == 4)) {
    uint64_t items = 0;
    for (uint32_t k = 0; k < t.count; ++k)
      items += (uint64_t)t.u[k].targets * t.u[k].batch * CvShape<kR, kIn, 4>::blocks;
    if (items <= 2ull * p->num_cus) return cv_launch_w<kR, kIn, 4>(p, t, s);
  }
  return cv_launch_w<kR, kIn, (kIn == 0 && kR > 1 ? 8 : 4)>(p, t, s);
}

template <int kIn>
hipError_t cv_launch_r(const tfhe_ntt_plan_s* p, CvTable& t, hipStream_t s) {
  switch (p->log_n) {
    case 12: return cv_launch<1, kIn>(p, t, s);
    case 13: return cv_launch<2, kIn>(p, t, s);
    case 14: return cv_launch<4, kIn>(p, t, s);
    case 15: return cv_launch<8, kIn>(p, t, s);
    default: return cv_launch<16, kIn>(p, t, s);
  }
}

}  // namespace

// First passes of the broadcast and conversion units of one plan (mids[k]:
// unit k's tiled output), kMaxCvUnits units per launch.  Units of one launch
// agree in kind (conversion or not).
hipError_t cv_run(const tfhe_ntt_plan_s* p, const NttUnit* const* units, uint32_t* const* mids, uint32_t count,
                  hipStream_t s) {
  for (uint32_t i = 0; i < count;) {
    CvTable t{};
    t.chunk = 1;
    t.blob = (const unsigned char*)p->d_fs_blob;
    t.per = 2 * p->fs_limb_bytes;  // forward and inverse tables of a limb follow each other
    t.op_off = p->fs_op_off;
    t.mods = p->d_mod;
    uint32_t nin = 0;
    for (; i < count && t.count < (uint32_t)kMaxCvUnits; ++i) {
      const NttUnit& u = *units[i];
      if (u.limb_count * u.batch == 0) continue;
      CvUnit& v = t.u[t.count++];
      if (u.conv) {
        const ConvSource& c = *u.conv;
        v = CvUnit{u.in, mids[i], c.tgt, u.batch, c.nin, u.limb_count, c.d0, c.nd, c.level, c.tiled ? 1u : 0u, 1, 0, 0};
        t.L = c.L;
        nin = std::max(nin, c.nin);
      } else {
        v = CvUnit{u.in, mids[i], nullptr, u.batch, 1, u.limb_count, u.limb_count, 0, u.limb_count, u.in_tiled ? 1u : 0u, 1, 0, 0};
      }
    }
    if (t.count == 0) break;
    const hipError_t e = nin == 0 ? cv_launch_r<0>(p, t, s) : nin <= 4 ? cv_launch_r<4>(p, t, s) : cv_launch_r<8>(p, t, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace tfhe
