"""What the host code launches for a call, and what it makes of a launch that fails, without a GPU: the
library runs on a stand-in for the HIP runtime (fake_hip_runtime.cpp) in a process of its own, on device
addresses that nothing reads."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MGRIT_E_LAUNCH = -7
CALL = """
import ctypes, sys
ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
from paper_2203_04738_amd.binding import MgritGruCfg, lib
from ctypes import byref
L, entry, cfg = lib(), sys.argv[2], MgritGruCfg(*(int(a) for a in sys.argv[3:]))
A, n = [ctypes.c_void_p((i + 1) << 32) for i in range(16)], ctypes.c_size_t(1 << 40)
if entry == "scan":
    rc = L.gru_serial_scan(byref(cfg), *A[:7], A[15], n, None)
elif entry == "scan_backward":
    rc = L.gru_serial_scan_backward(byref(cfg), *A[:12], A[15], n, None)
elif entry == "forward":
    rc = L.mgrit_gru_forward(byref(cfg), *A[:8], A[15], n, None)
print("returned", rc)
"""


@pytest.fixture(scope="module")
def runtime(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("hip") / "libfake_hip.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", out,
                           os.path.join(ROOT, "tests", "fake_hip_runtime.cpp")])
    return out


def call(runtime, entry, *cfg, **env):
    """(what the call returned, the kernels it launched, as [workgroups, name])"""
    r = subprocess.run([sys.executable, "-c", CALL, runtime, entry, *(str(int(v)) for v in cfg)], cwd=ROOT,
                       env=dict(os.environ, **env), capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    lines = [line.split(" ", 2) for line in r.stdout.splitlines()]
    (rc,) = (int(f[1]) for f in lines if f[0] == "returned")
    return rc, [(int(f[1]), f[2]) for f in lines if f[0] in ("launched", "failed")]


def cfg(T, B, D, H, cf=1, levels=1, iters=1, fine=1, dtype=0):
    return T, B, D, H, cf, levels, iters, fine, 0, dtype, 0


@pytest.mark.parametrize("dtype", [1, 3])
@pytest.mark.parametrize("B,H,xcd", [(8, 1024, False), (1, 512, True), (64, 512, True), (64, 1024, True),
                                     (64, 256, True)])
def test_coarsest_level_on_bf16_weights_keeps_the_fp32_contraction(runtime, B, H, xcd, dtype):
    # (up to 64 rows; the scan as one level contracts terms of the state)
    rc, got = call(runtime, "forward", *cfg(4096, B, 64, H, cf=8, levels=3, dtype=dtype))
    scans = [name for _, name in got if "scan_kernel<" in name]
    assert rc == 0 and len(scans) == 2
    assert all(name.split(">(")[0].endswith("false") for name in scans), scans
    assert ("xcd_scan_kernel" in scans[0]) == xcd
    rc, got = call(runtime, "scan", *cfg(512, B, 64, H, dtype=dtype))
    scans = [name for _, name in got if "scan_kernel<" in name]
    assert rc == 0 and len(scans) == 2
    assert "xcd_scan_kernel" in scans[0]
    assert all(name.split(">(")[0].endswith("true") for name in scans), scans


@pytest.mark.parametrize("entry,kernel", [("scan", "mg::xcd_scan_kernel<0"), ("scan", "scan_mark_kernel"),
                                          ("scan", "mg::scan_kernel<0"), ("scan_backward", "adj_xcd_scan_kernel<1"),
                                          ("scan_backward", "scan_mark_kernel"),
                                          ("scan_backward", "mg::scan_kernel<1")])
def test_a_solve_that_cannot_be_launched_is_reported(runtime, entry, kernel):
    # (a later launch that succeeds must not hide it: the rows would hold the marks of unwritten ones)
    c = cfg(64, 32, 64, 512)
    rc, got = call(runtime, entry, *c)
    assert rc == 0 and any(kernel in name for _, name in got), got
    rc, _ = call(runtime, entry, *c, FAKE_HIP_FAIL=kernel)
    assert rc == MGRIT_E_LAUNCH


@pytest.mark.parametrize("H,D,terms", [(16384, 64, True), (18912, 64, True), (18920, 64, False),
                                       (1024, 262144, True), (1024, 349600, False)])
def test_widths_up_to_which_packed_terms_are_addressed(runtime, H, D, terms):
    # (32-bit offsets into 12 H^2 and 12 H D bytes; the projection's terms have a bound of their own)
    rc, got = call(runtime, "forward", *cfg(64, 32, D, H, cf=4, levels=2, dtype=2))
    names = " ".join(name for _, name in got)
    assert rc == 0
    assert ("split2_kernel" in names) == terms
    assert ("phi_step_kernel_bf16" in names) == terms
    assert "split3" in names and "projection_kernel(" not in names
