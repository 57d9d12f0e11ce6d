"""The host side of the plan without a GPU: the library runs on a HIP runtime
that executes nothing and records every call (fake_hip.cpp), in a process of its
own.  Checked is what a result cannot show: which buffers are freed while the plan
lives, what an option launches or waits for, and what orders kernels that share a
buffer."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, sys
sys.path.insert(0, %r)
hip = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)  # before the library: its HIP calls go here
hip.fake_log.restype = ctypes.c_char_p
hip.fake_used.restype = ctypes.c_size_t
from paper_2011_07099_amd import pfmm
lib = pfmm.load()
GREEN, NEAR, PREC, M2L, ACCEL = pfmm.GREEN, pfmm.NEAR, pfmm.PREC, pfmm.M2L, pfmm.ACCEL

def log():
    return hip.fake_log().decode().splitlines()

def of(lines, *kinds):
    return [l for l in lines if l.split()[0] in kinds]

def create(N, L, p, green="S"):
    h = ctypes.c_void_p()
    assert lib.pfmm_plan_create(N, L, p, GREEN[green], ctypes.byref(h)) == 0
    return h

def put(h, option, value):
    v = (ctypes.c_double if isinstance(value, float) else ctypes.c_int32)(value)
    return lib.pfmm_plan_set(h, option, ctypes.byref(v), ctypes.sizeof(v))

def stream(h, s):
    v = ctypes.c_void_p(s)
    assert lib.pfmm_plan_set(h, pfmm.OPT_STREAM, ctypes.byref(v), 8) == 0

A, B, C = (ctypes.c_void_p(x << 20) for x in (1 << 22, 1 << 23, 3 << 22))  # device addresses of arrays
""" % ROOT


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("amdclang++") or "/opt/rocm/bin/amdclang++"
    out = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run([cxx, "-O1", "-shared", "-fPIC", "-o", out, os.path.join(HERE, "fake_hip.cpp")], check=True)
    return out


def run(fake, body):
    from paper_2011_07099_amd import pfmm
    if not os.path.exists(pfmm.LIB_PATH):
        pytest.skip("libpfmm.so not built")
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, fake], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr


@pytest.mark.parametrize("N,L,p", [(64, 3, 8), (64, 2, 4), (128, 7, 6)])
def test_options_free_nothing(fake, N, L, p):
    """A captured solve holds the plan's buffers: only the plan's end frees them
    (temporaries of a tabulation, made and freed in one call, aside)."""
    run(fake, """
h = create(%d, %d, %d)
assert lib.pfmm_solve(h, A, B, None) == 0
log()
before = hip.fake_used()
for option, value in ((pfmm.OPT_NEAR, 1), (pfmm.OPT_PRECISION, 2), (pfmm.OPT_PRECISION, 0), (pfmm.OPT_NEAR, 0),
                      (pfmm.OPT_M2L, M2L["spectral"]), (pfmm.OPT_ACCEL, 1), (pfmm.OPT_NEAR, 1),
                      (pfmm.OPT_M2L, M2L["gemm"]), (pfmm.OPT_PRECISION, 1), (pfmm.OPT_GS_A1, -0.1)):
    if option == pfmm.OPT_NEAR and value and %d >> %d < 4:
        continue                                    # rocFFT's plans need a device
    assert put(h, option, value) == 0, (option, value, lib.pfmm_last_error())
    lines = log()
    here = {l.split()[1] for l in of(lines, "malloc")}
    freed = {l.split()[1] for l in of(lines, "free")}
    assert freed <= here, (option, value, freed - here)
assert hip.fake_used() >= before
assert lib.pfmm_plan_destroy(h) == 0
assert hip.fake_used() == 0, hip.fake_used()
""" % (N, L, p, N, L))


def test_precision_and_near_zone_options_run_nothing(fake):
    run(fake, """
h = create(64, 3, 8)
assert lib.pfmm_solve(h, A, B, None) == 0
assert put(h, pfmm.OPT_NEAR, 1) == 0 and put(h, pfmm.OPT_NEAR, 0) == 0   # its buffers, on first use
log()
for option, value in ((pfmm.OPT_PRECISION, 1), (pfmm.OPT_NEAR, 1), (pfmm.OPT_PRECISION, 2),
                      (pfmm.OPT_PRECISION, 0), (pfmm.OPT_NEAR, 0)):
    assert put(h, option, value) == 0
    assert log() == [], (option, value)
assert put(h, pfmm.OPT_ACCEL, 1) == 0
kernels = [l.split()[1] for l in of(log(), "launch")]
assert sum("k_kz64" in k for k in kernels) == 3, kernels   # the accelerations', not G's own again
""")


def test_a_failed_spectral_option_leaves_no_spectra_without_kernels(fake):
    """64^3 with one-cell leaves, p = 6: the option needs spectra of its own."""
    run(fake, """
h = create(64, 6, 6)
used = hip.fake_used()
hip.fake_fail_launches(1)
assert put(h, pfmm.OPT_M2L, M2L["spectral"]) != 0
hip.fake_fail_launches(0)
assert hip.fake_used() == used
log()
assert lib.pfmm_solve(h, A, B, None) == 0            # the default zones, as before
assert put(h, pfmm.OPT_M2L, M2L["spectral"]) == 0
assert any("k_khat_z" in l for l in of(log(), "launch"))
""")


def test_what_writes_the_convolution_s_spectrum_waits_for_the_last_one(fake):
    """Every writer of the shared spectrum and of G's transform waits for the
    last convolution, also on a stream whose handle it has seen before."""
    run(fake, """
h = create(32, 3, 4)
stream(h, 0x100)
assert lib.pfmm_plan_direct(h, A, B) == 0
event = of(log(), "record")[-1].split()[1]
for act in (lambda: lib.pfmm_plan_direct(h, A, C),                       # the same handle
            lambda: (stream(h, 0x200), lib.pfmm_plan_direct(h, A, B))[1],
            lambda: (stream(h, 0x100), put(h, pfmm.OPT_GS_A1, -0.1))[1]):
    assert act() == 0
    lines = log()
    first = next(i for i, l in enumerate(lines) if "k_pm_" in l or "k_mesh" in l)
    st = lines[first].split()[-1]
    assert "wait %s %s" % (st, event) in lines[:first], lines
hip.fake_capture(ctypes.c_void_p(0x100))              # a captured call has the caller's order
assert lib.pfmm_plan_direct(h, A, B) == 0
assert of(log(), "wait", "record") == []
""")


def test_fp32_columns_option_runs_nothing(fake):
    run(fake, """
h = create(64, 4, 4)
assert put(h, pfmm.OPT_M2L, M2L["spectral"]) == 0
log()
for v in (1, 0, 1):
    assert put(h, pfmm.OPT_ZONES_FP32, v) == 0
    assert log() == []
assert put(h, pfmm.OPT_ZONES_FP32, 0) == 0 and put(h, pfmm.OPT_GS_A1, -0.1) == 0
assert any("k_khat_f32" in l for l in log())          # the FP32 kernels follow G, the option on or off
""")


def test_optional_buffers_leave_a_quarter_of_the_card(fake):
    """Plans on a small card: the first take the transforms' buffers, and later
    ones, made where these would leave less than a quarter free, use the products
    instead of failing; what such plans allocate by themselves still fits."""
    run(fake, """
total = 2 << 30
hip.fake_total(ctypes.c_size_t(total))
routes, plans = [], []
while hip.fake_used() < 0.9 * total and len(plans) < 40:
    h = create(64, 3, 8)
    plans.append(h)
    log()
    assert lib.pfmm_solve(h, A, B, None) == 0
    kernels = " ".join(of(log(), "launch"))
    routes.append(("k_fwd64" in kernels, "k_toep" in kernels))
    if "k_fwd64" in kernels:
        assert hip.fake_used() <= 0.75 * total
assert routes[0] == (True, False) and routes[-1] == (False, True), routes
assert put(plans[-1], pfmm.OPT_ACCEL, 1) == 0 and put(plans[-1], pfmm.OPT_PRECISION, 2) == 0
assert lib.pfmm_solve(plans[-1], A, B, C) == 0
for h in plans:
    assert lib.pfmm_plan_destroy(h) == 0
assert hip.fake_used() == 0
""")


def test_a_plan_set_to_another_near_zone_before_its_first_solve_gives_buffers_back(fake):
    """Plan(..., near="fft") does not hold the direct near zone's 140 bytes a cell;
    set back, it has them and their kernels again, and after a solve it keeps them."""
    run(fake, """
N = 128
h = create(N, 3, 8)
log()
for _ in range(2):
    before = hip.fake_used()
    assert put(h, pfmm.OPT_NEAR, 1) == 0
    assert before - hip.fake_used() > 30 * N ** 3      # 140 bytes a cell less the FFT near zone's on first use
    log()
    assert put(h, pfmm.OPT_NEAR, 0) == 0
    lines = log()
    assert sum("k_kz64" in l for l in lines) == 1 and lines[-1].startswith("sync"), lines
assert put(h, pfmm.OPT_NEAR, 1) == 0 and put(h, pfmm.OPT_PRECISION, 2) == 0    # FP64: direct, whatever the option
assert lib.pfmm_solve(h, A, B, None) == 0
assert "k_fwd64" in " ".join(log())
used = hip.fake_used()
assert put(h, pfmm.OPT_PRECISION, 0) == 0 and put(h, pfmm.OPT_NEAR, 0) == 0 and put(h, pfmm.OPT_NEAR, 1) == 0
assert hip.fake_used() == used and log() == []
""")
