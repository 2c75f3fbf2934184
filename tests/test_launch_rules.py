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
  for (uint32_t cus : {32u, 256u, 304u})
    for (uint64_t items = 1; items <= 200ull * cus; items += items < 9 * cus ? 1 : cus / 4)
      std::printf("%u %llu %u\\n", cus, (unsigned long long)items, tfhe::wide_wg_per_cu(items, cus));
}
"""


def test_wide_pass_workgroups_keep_their_ring_busy(tmp_path):
    """A workgroup that is not resident from the start pays its tables and its
    ring's first loads again: more than one per CU only where each still gets
    a dozen items."""
    src, exe = tmp_path / "rules.cpp", tmp_path / "rules"
    src.write_text(DRIVER.replace("../", ROOT + "/"))
    r = subprocess.run(["g++", "-std=c++17", "-I" + os.path.join(SAN, "fakehip"), "-I" + os.path.join(ROOT, "include"),
                        str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    seen = set()
    for line in subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.splitlines():
        cus, items, w = map(int, line.split())
        assert w == 1 or items >= 12 * w * cus, (cus, items, w)
        seen.add(w)
    assert seen == {1, 2, 4}


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
