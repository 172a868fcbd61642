"""A call whose n-th launch fails leaves the counter of the state that the caller's
buffer holds (host only: the library linked against launches that do nothing,
tests/launch_faults.c, with its own code unchanged)."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import ctypes as C, sys
import paper_1107_5463_amd as smc
lib = smc.load_library()
lib.faults_reset.argtypes = [C.c_long]
lib.faults_count.restype = C.c_long
ws = C.c_void_p(1 << 30)

def handle(d, n, L, flags=0, J_kind=0, **kw):
    p = smc.make_params(d, n, L, 3, init="keep", J_kind=J_kind, delta=1.2, flags=flags | smc.FLAG_COUPLINGS_KEEP, **kw)
    h = C.c_void_p()
    lib.faults_reset(0)
    J = C.c_void_p(1 << 21) if J_kind else None
    assert lib.smc_init_lattice(C.byref(h), C.byref(p), C.c_void_p(1 << 20), J, ws, 1 << 40, None) == 0, lib.smc_last_error()
    assert lib.faults_count() == 0
    return h

def t_of(h):
    t = C.c_uint64()
    assert lib.smc_get_sweep_index(h, C.byref(t)) == 0
    return t.value

def run(expect, name, sweeps, measured, *args, **kw):
    # expect: the counter after a failure of launch 1, 2, ..; it is `sweeps` without one
    h = handle(*args, **kw)
    assert lib.smc_sweeps_kernel(h, sweeps, int(measured), None).decode() == name
    def call():
        return lib.smc_sweep_measure(h, 0.5, sweeps, C.c_void_p(1 << 22)) if measured else lib.smc_sweep(h, 0.5, sweeps)
    assert call() == 0 and t_of(h) == sweeps
    total = lib.faults_count()
    want = expect(total)
    assert len(want) == total, (name, total, want)
    for k in range(1, total + 1):
        lib.smc_set_sweep_index(h, 0)
        lib.faults_reset(k)
        assert call() == smc.SMC_EDEVICE and lib.faults_count() == k, (name, k)
        assert t_of(h) == want[k - 1], (name, args, k, t_of(h), want)
        assert lib.smc_destroy(h) == 0
        h = handle(*args, **kw)
    lib.smc_destroy(h)

# several launches through the workspace: nothing is in the caller's buffer before the last
run(lambda n: [0] * n, "ising_resident", 20, False, 2, 1, 1000)
run(lambda n: [0] * (n - 1) + [20], "ising_resident", 20, True, 2, 1, 1000)
run(lambda n: [0] * n, "ising_resident", 130, False, 2, 1, 1000)
run(lambda n: [0] * n, "ising_resident", 10, False, 3, 1, 64, J_kind=1)
run(lambda n: [0] * (n - 1) + [10], "ising_packed", 10, True, 2, 1, 8192)
run(lambda n: [0] * n, "ising_bricks", 20, False, 3, 1, 40, J_kind=2)
run(lambda n: [0] * (n - 1) + [20], "ising_bricks", 20, True, 3, 1, 40, J_kind=2)
# one workgroup: in place, launch by launch
run(lambda n: [0, 64, 128, 192], "ising_resident", 200, False, 2, 1, 32)
run(lambda n: [0], "ising_bricks", 20, True, 2, 1, 16, J_kind=2)
# sweeps and renormalisations in turn
run(lambda n: [0, 7, 7, 14, 14], "xy_bricks", 20, False, 2, 2, 16, renorm_every=7)
# from one buffer to the other and back: 2 sweeps, 1, 1, 1
run(lambda n: [0, 0, 3, 3, 5], "xy_march", 5, True, 2, 2, 3000, renorm_every=0)
# half-sweeps in place, as ever
run(lambda n: [0, 0, 1, 1, 2, 2], "heisenberg_stream", 3, False, 3, 3, 128, renorm_every=0)
print("ok")
"""


def test_counter_after_a_failed_launch(tmp_path):
    from paper_1107_5463_amd import build as pkg_build
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("hipcc is not installed")
    objdir = os.path.join(ROOT, "paper_1107_5463_amd", "_build")
    objs = [os.path.join(objdir, os.path.splitext(s)[0] + ".o") for s in pkg_build.SOURCES]
    if not all(os.path.exists(o) for o in objs):
        pkg_build.build()
    shim, lib = str(tmp_path / "launch_faults.o"), str(tmp_path / "libsmc_faults.so")
    subprocess.run(["gcc", "-O1", "-fPIC", "-c", os.path.join(ROOT, "tests", "launch_faults.c"), "-o", shim], check=True)
    subprocess.run([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-Wl,-Bsymbolic", "-o", lib] + objs + [shim],
                   check=True, capture_output=True)
    env = {k: v for k, v in os.environ.items() if not k.startswith("SMC_")}
    env["SMC_LIBRARY"] = lib
    p = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT, env=env, capture_output=True, text=True, timeout=120)
    assert p.returncode == 0 and p.stdout.strip().endswith("ok"), p.stdout[-2000:] + p.stderr[-3000:]
