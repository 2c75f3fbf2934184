"""The workspace audit (AddressSanitizer, on the CPU) with stand-ins that follow
the key switch's fused conversions plane by plane, and the element-wise
ciphertext operations in exactly sized buffers.  The audits are also run on
mistakes planted in copies of the host code, which they have to report."""
import concurrent.futures
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SAN = os.path.join(ROOT, "tests", "sanitize")
CSRC = os.path.join(ROOT, "paper_2212_14191_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")

# (text of ckks.cpp, planted mistake)
MISTAKES = {
    "modup_intermediates": ("align256(plane * (size_t)digits * ext) : 0;", "align256(plane * (size_t)digits * (ext - 1)) : 0;"),
    "digit_twist": ("u.twist = c->d_up_tw + (size_t)(d0 + nd - 1)", "u.twist = c->d_up_tw + (size_t)(d0 + nd)"),
    "special_twist": ("for (uint32_t k = 0; k < K; ++k) scaled_twist(c->plan, L + k",
                      "for (uint32_t k = 1; k < K; ++k) scaled_twist(c->plan, L + k"),
    "digit_constants": ("c->d_up_cv + (size_t)key_idx * (c->L + c->K)", "c->d_up_cv + (size_t)(key_idx + 1) * (c->L + c->K)"),
}


FLAGS = ["g++", "-std=c++17", "-O1", "-g", "-fno-omit-frame-pointer", "-I" + os.path.join(SAN, "fakehip"),
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-fsanitize=address,undefined",
         "-fno-sanitize-recover=undefined"]
SRCS = [os.path.join(CSRC, f) for f in ("plan.cpp", "capi.cpp", "timing.cpp", "ckks.cpp")] + [
    os.path.join(SAN, f) for f in ("unit_stubs.cpp", "ws_audit_driver.cpp", "ct_audit_driver.cpp")]


def cc(args):
    r = subprocess.run(FLAGS + args, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]


@pytest.fixture(scope="module")
def objects(tmp_path_factory):
    """Each source compiled once."""
    d = tmp_path_factory.mktemp("objects")
    objs = {os.path.basename(f): str(d / (os.path.basename(f) + ".o")) for f in SRCS}
    with concurrent.futures.ThreadPoolExecutor(max_workers=4) as ex:
        list(ex.map(lambda f: cc(["-c", f, "-o", objs[os.path.basename(f)]]), SRCS))
    return objs


def link(tmp_path, objects, driver, **replaced):
    objs = dict(objects, **replaced)
    drop = {"ws_audit_driver.cpp", "ct_audit_driver.cpp"} - {driver}
    exe = str(tmp_path / "audit")
    cc([o for name, o in objs.items() if name not in drop] + ["-lpthread", "-o", exe])
    return exe


def run(exe, *args):
    r = subprocess.run([exe, *args], capture_output=True, text=True, timeout=300,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=0"))
    return r.returncode, r.stdout + r.stderr


def test_workspace_audit_with_conversion_units(tmp_path, objects):
    rc, out = run(link(tmp_path, objects, "ws_audit_driver.cpp"))
    assert rc == 0 and " 0 failures" in out and "Sanitizer" not in out, out[-6000:]


@pytest.mark.parametrize("name", sorted(MISTAKES))
def test_audit_reports_planted_mistakes(tmp_path, objects, name):
    text, wrong = MISTAKES[name]
    src = open(os.path.join(CSRC, "ckks.cpp")).read()
    assert src.count(text) == 1
    (tmp_path / "ckks.cpp").write_text(src.replace(text, wrong))
    cc(["-c", str(tmp_path / "ckks.cpp"), "-o", str(tmp_path / "ckks.o")])
    rc, out = run(link(tmp_path, objects, "ws_audit_driver.cpp", **{"ckks.cpp": str(tmp_path / "ckks.o")}))
    assert rc != 0 and "AddressSanitizer" in out, out[-3000:]


def test_ciphertext_operations_in_exact_buffers(tmp_path, objects):
    exe = link(tmp_path, objects, "ct_audit_driver.cpp")
    rc, out = run(exe)
    assert rc == 0 and "Sanitizer" not in out, out[-3000:]
    for short in range(6):
        rc, out = run(exe, str(short))
        assert rc != 0 and "AddressSanitizer" in out, short
