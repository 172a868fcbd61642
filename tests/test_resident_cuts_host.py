"""The splits of the resident tests are those that run: each forced split that fits
takes the resident way, and one that does not is refused (host only)."""
import ctypes as C

import pytest

from test_gpu_resident import CASES


@pytest.mark.parametrize("d,L,kind,hb,packed,J0,beta,n,split", CASES)
def test_forced_splits_run(monkeypatch, d, L, kind, hb, packed, J0, beta, n, split):
    import paper_1107_5463_amd as smc
    monkeypatch.setenv("SMC_RESIDENT", split)
    lib = smc.load_library()
    flags = smc.FLAG_COUPLINGS_KEEP | (smc.FLAG_HEATBATH if hb else 0) | (smc.FLAG_PACKED if packed else 0)
    p = smc.make_params(d, 1, L, L + n, init="keep", J_kind=kind, J0=J0, flags=flags)
    h = C.c_void_p()
    # (addresses that nothing reads: a handle that keeps its spins launches nothing)
    assert lib.smc_init_lattice(C.byref(h), C.byref(p), C.c_void_p(1 << 20), C.c_void_p(1 << 21) if kind else None,
                                C.c_void_p(1 << 30), 1 << 40, None) == 0, lib.smc_last_error()
    launches = C.c_uint64()
    name = lib.smc_sweeps_kernel(h, n, 1, C.byref(launches)).decode()
    lib.smc_destroy(h)
    fits = (d, L, split) != (3, 64, "2,2048")
    assert (name == "ising_resident") == fits, (name, split)
    if fits:
        S, own = (int(x) for x in split.split(",")[:2])
        Wp = (L ** d // 2 + 31) // 32
        # bands: at most S half-sweeps a launch; one workgroup goes on in its own
        assert launches.value >= (2 * n + S - 1) // S if own < Wp else launches.value == (n + 63) // 64
