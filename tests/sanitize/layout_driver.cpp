// Which inverse transforms write quad-tiled results (NttUnit::out_tiled), for
// every N and number of passes a plan asks for: where the second pass is the
// two-pass kernel's and N >= 2^15, natural order would reach the fused
// conversions' first pass in pieces of 16 or 32 bytes.  N = 2^16 has two
// passes whatever the plan asks for.
#include <cstdio>
#include <cstdlib>

#include "../../paper_2212_14191_amd/csrc/ckks_internal.hpp"

#define fs_run_units stub_run_units
#include "kernel_stubs.cpp"
#undef fs_run_units

static int tiled = 0, natural = 0, disagree = 0;

namespace tfhe {
hipError_t fs_run_units(const NttUnit* u, uint32_t count, void* ws, hipStream_t s) {
  for (uint32_t k = 0; k < count; ++k) {
    if (u[k].inverse) ++(u[k].out_tiled ? tiled : natural);
    const bool reads_tiled = u[k].conv ? u[k].conv->tiled : u[k].in_tiled;
    if (u[k].in_bcast && reads_tiled != (tiled != 0)) ++disagree;
  }
  return stub_run_units(u, count, ws, s);
}
}  // namespace tfhe

int main() {
  int failures = 0;
  for (uint32_t log_n = 14; log_n <= 16; ++log_n) {
    tfhe_ckks_ctx c = nullptr;
    tfhe_ntt_plan plan = nullptr;
    if (tfhe_ckks_ctx_create(&c, log_n, 2, 1, 1, nullptr, nullptr, TFHE_NTT_FOURSTEP_MFMA) != TFHE_OK ||
        tfhe_ckks_ctx_plan(c, &plan) != TFHE_OK)
      return 1;
    const size_t ct = (size_t)16 << log_n;  // level 2, one element
    uint32_t *a = (uint32_t*)std::aligned_alloc(256, ct), *out = (uint32_t*)std::aligned_alloc(256, ct);
    uint32_t* key = (uint32_t*)std::aligned_alloc(256, (size_t)24 << log_n);
    for (int passes = 0; passes <= 2; ++passes) {
      if (tfhe_ntt_plan_set_param(plan, TFHE_PARAM_FS_PASSES, passes) != TFHE_OK) return 1;
      const bool want = log_n == 16 || (log_n == 15 && passes != 1);
      for (int op = 0; op < 2; ++op) {
        size_t wsb = 0;
        if ((op ? tfhe_rescale_workspace_size(c, 2, 1, &wsb) : tfhe_hmult_workspace_size(c, 2, 1, &wsb)) != TFHE_OK)
          return 1;
        void* ws = std::aligned_alloc(256, wsb);
        tiled = natural = disagree = 0;
        const tfhe_status st = op ? tfhe_rescale(c, a, out, 2, 1, ws, wsb, nullptr)
                                  : tfhe_hmult(c, a, a, out, key, 2, 1, ws, wsb, nullptr);
        std::free(ws);
        if (st != TFHE_OK || (want ? natural : tiled) != 0 || (want ? tiled : natural) == 0 || disagree) {
          std::printf("N = 2^%u, passes %d, %s: %d tiled, %d natural, %d disagree\n", log_n, passes,
                      op ? "rescale" : "hmult", tiled, natural, disagree);
          ++failures;
        }
      }
    }
    std::free(a);
    std::free(out);
    std::free(key);
    tfhe_ckks_ctx_destroy(c);
  }
  std::printf("%d failures\n", failures);
  return failures != 0;
}
