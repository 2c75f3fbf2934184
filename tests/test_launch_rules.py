"""Launch-shape rules of the library's host code, on the CPU: compiled from the
library's header against the stand-in HIP runtime and tabulated."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SAN = os.path.join(ROOT, "tests", "sanitize")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")

DRIVER = """
#include <cstdio>
#include "../paper_2212_14191_amd/csrc/internal.hpp"
int main() {
  for (uint32_t cus : {1u, 32u, 256u, 304u})
    for (uint32_t ipp : {1u, 4u, 8u})
      for (uint32_t polys = 1; polys * ipp <= 200 * cus; polys += polys * ipp < 60 * cus ? 1 : 7)
        std::printf("%u %u %u\\n", cus, polys * ipp, tfhe::wide_wg_per_cu(polys, ipp, cus));
}
"""


def test_wide_pass_workgroups_keep_their_ring_busy(tmp_path):
    """A workgroup that is not resident from the start pays its tables and its
    ring's first loads again: more than one per CU only where each still gets
    nine items or more."""
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text(DRIVER.replace("../", ROOT + "/"))
    r = subprocess.run(["g++", "-std=c++17", "-I" + os.path.join(SAN, "fakehip"), "-I" + os.path.join(ROOT, "include"),
                        str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    seen = set()
    for line in subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.splitlines():
        cus, items, w = map(int, line.split())
        assert w == 1 or items >= 9 * w * cus, (cus, items, w)
        seen.add(w)
    assert seen == {1, 2, 4, 5}


FROB_DRIVER = """
#include <cstdio>
#include "../paper_2212_14191_amd/csrc/internal.hpp"
int main() {
  unsigned log_n, g;
  while (std::scanf("%u %u", &log_n, &g) == 2) {
    const uint32_t s = tfhe::frob_lines(g, log_n);
    std::printf("%u %u %u %u %u\\n", s, tfhe::frob_by_poly(log_n, 32, s), tfhe::frob_by_poly(log_n, 64, s),
                tfhe::frob_by_poly(log_n, 512, s), tfhe::frob_by_poly(log_n, 2048, s));
  }
}
"""


def test_frobenius_by_element_where_it_reads_whole_lines(tmp_path):
    """The number of 128-byte lines that 64 lanes of the element-wise kernel touch
    is counted as they are, and maps that read whole lines (identity,
    conjugation) stay element by element where polynomials are few or fill a
    CU's LDS each."""
    src, exe = tmp_path / "frob.cpp", tmp_path / "frob"
    src.write_text(FROB_DRIVER.replace("../", ROOT + "/"))
    r = subprocess.run(["g++", "-std=c++17", "-I" + os.path.join(SAN, "fakehip"), "-I" + os.path.join(ROOT, "include"),
                        str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    cases = []
    for log_n in range(10, 17):
        n = 1 << log_n
        gs = [1, 2 * n - 1, n + 1, n - 1, 3, 5, 25, 2 * n - 5, n // 2 + 1, n // 4 + 1, 3 * n // 8 + 1]
        cases += [(log_n, g) for g in gs + [pow(5, e, 2 * n) for e in range(2, 40)]]
    r = subprocess.run([str(exe)], input="\n".join(f"{a} {b}" for a, b in cases), capture_output=True, text=True, check=True)
    for (log_n, g), line in zip(cases, r.stdout.splitlines()):
        n = 1 << log_n
        s, by32, by64, by512, by2048 = map(int, line.split())
        lines = {((2 * j + 1) * g % (2 * n) - 1) // 2 // 32 for j in range(64)}
        streams = (g % (n // 16)) in (1, n // 16 - 1)
        assert s == len(lines) // ({15: 2, 16: 4}.get(log_n, 1) if streams else 1), (log_n, g, s, len(lines))
        if s <= 3:
            assert not by32 and not by64 and by512 == (12 <= log_n <= 14) and by2048 == (12 <= log_n), (log_n, g)
        elif s > 32:
            assert by64 == by512 == by2048 == (log_n >= 12) and by32 == (log_n >= 15), (log_n, g)


def test_inverse_outputs_of_two_pass_transforms_are_quad_tiled(tmp_path):
    exe = str(tmp_path / "layout")
    csrc = os.path.join(ROOT, "paper_2212_14191_amd", "csrc")
    srcs = [os.path.join(csrc, f) for f in ("plan.cpp", "capi.cpp", "ckks.cpp", "timing.cpp")]
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-I" + os.path.join(SAN, "fakehip"),
                        "-I" + os.path.join(ROOT, "include"), "-x", "c++"] + srcs
                       + [os.path.join(SAN, "layout_driver.cpp"), "-lpthread", "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
