// kernel_stubs.cpp with the stand-ins of the transform units and of the
// element-wise launcher replaced by ones that also touch what the fused
// conversions, the folded constants and the ciphertext operations touch: every
// input plane of a conversion and its constants, every target plane at its
// extended-basis position, a unit's own twist and its epilogue's multipliers,
// and both components of a ciphertext.  Linked in kernel_stubs.cpp's place.
#include "../../paper_2212_14191_amd/csrc/ckks_internal.hpp"

#define fs_run_units plain_run_units
#define ew_launch plain_ew_launch
#include "kernel_stubs.cpp"
#undef fs_run_units
#undef ew_launch

namespace tfhe {

static volatile uint64_t g_pairs;
static void rd_pairs(const uint2* p, uint64_t count) {
  if (count) g_pairs = g_pairs + p[0].x + p[count - 1].y;
}

static void conv_io(const NttUnit& u, uint32_t* mid) {
  const ConvSource& c = *u.conv;
  const uint64_t plane = (uint64_t)u.batch * u.plan->n;
  for (uint32_t r = 0; r < c.nin; ++r) rd(u.in + r * plane, plane);
  for (uint32_t t = 0; t < u.limb_count; ++t) {
    const uint32_t pos = t < c.d0 ? t : t + c.nd, limb = pos < c.level ? pos : c.L + pos - c.level;
    g_pairs = g_pairs + c.tgt[limb].init + (uint32_t)c.tgt[limb].c[0] + c.tgt[limb].q;
    wr(mid + pos * plane, plane);
  }
}

hipError_t fs_run_units(const NttUnit* units, uint32_t count, void* ws, hipStream_t) {
  unsigned char* w = (unsigned char*)ws;
  for (uint32_t k = 0; k < count; ++k) {
    const NttUnit& u = units[k];
    if (u.twist) rd_pairs(u.twist, (uint64_t)u.limb_count * 256);
    if (u.epi_mult) rd_pairs(u.epi_mult, u.limb_count);
    const size_t b = u.pass1_only ? 0 : unit_ws_bytes(u, true);
    uint32_t* const mid = u.pass1_only ? u.out : (uint32_t*)w;
    w += round256(b);
    if (!u.conv) {
      unit_io(u, mid, b / 4);
      continue;
    }
    conv_io(u, mid);
    if (u.pass1_only) continue;
    if (u.acc) rd(u.acc, words_of(u));
    if (u.epi_add) rd(u.out, words_of(u));
    wr(u.out, words_of(u));
  }
  return hipSuccess;
}

hipError_t ew_launch(EwOp op, const ModConst* mods, const uint32_t* a, const uint32_t* b, uint32_t* out, uint32_t limbs,
                     uint32_t batch, uint32_t n, hipStream_t s) {
  if (op != EW_CT_MUL) return plain_ew_launch(op, mods, a, b, out, limbs, batch, n, s);
  const uint64_t w = (uint64_t)limbs * batch * n;
  rd(a, w);
  rd(a + w, w);
  rd(b, w);
  wr(out, w);
  wr(out + w, w);
  return hipSuccess;
}

}  // namespace tfhe
