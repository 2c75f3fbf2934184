// Audit of CMULT and HADD with buffers of exactly the documented sizes, under
// AddressSanitizer.  With an argument 0..5 that buffer (CMULT's ciphertext,
// plaintext, result; HADD's two ciphertexts, result) is one limb short, which
// has to be reported.
#include <cstdio>
#include <cstdlib>
#include <initializer_list>

#include "tfhe.h"

int main(int argc, char** argv) {
  const int shrunk = argc > 1 ? std::atoi(argv[1]) : -1;
  int failures = 0;
  for (uint32_t log_n : {10u, 12u}) {
    tfhe_ckks_ctx c = nullptr;
    if (tfhe_ckks_ctx_create(&c, log_n, 6, 2, 3, nullptr, nullptr, TFHE_NTT_AUTO) != TFHE_OK) return 2;
    for (uint32_t level : {1u, 6u})
      for (uint32_t batch : {1u, 3u}) {
        uint32_t* p[6];
        for (int k = 0; k < 6; ++k) {
          const uint32_t limbs = (k == 1 ? 1 : 2) * level - (k == shrunk);
          p[k] = (uint32_t*)std::aligned_alloc(256, limbs ? (size_t)limbs * batch * 4 << log_n : 256);
        }
        failures += tfhe_cmult(c, p[0], p[1], p[2], level, batch, nullptr) != TFHE_OK;
        failures += tfhe_hadd(c, p[3], p[4], p[5], level, batch, nullptr) != TFHE_OK;
        for (uint32_t* q : p) std::free(q);
      }
    tfhe_ckks_ctx_destroy(c);
  }
  std::printf("%d failures\n", failures);
  return failures != 0;
}
