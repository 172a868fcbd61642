"""Stored tuning choices that were made for another kernel are not taken: band
heights for another number of sites a lane, and batch paths from before the
lattice had two."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,n,L", [(3, 3, 64), (2, 2, 256)])
def test_heights_go_with_their_sites_a_lane(smc_gpu, monkeypatch, tmp_path, d, n, L):
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("SMC_AUTOTUNE_CACHE", str(cache))
    monkeypatch.setenv("SMC_CONT_SPL", "2" if n == 3 else "4")
    smc_gpu.Lattice(d, n, L, 5, delta=1.0).autotune(0.7)
    (key, _), = [line.split(" ") for line in cache.read_text().strip().split("\n")]
    stale = f"{key} 64\n"
    cache.write_text(stale)
    # with the sites a lane it was made for, the choice is taken as it stands
    assert smc_gpu.Lattice(d, n, L, 5, delta=1.0).autotune(0.7) == 64
    monkeypatch.delenv("SMC_CONT_SPL")
    lat = smc_gpu.Lattice(d, n, L, 5, delta=1.0)  # 1 and 2 a lane by itself
    default = lat.kernel()[1]
    rows = C.c_uint32()
    lib = smc_gpu.load_library()
    assert lib.smc_autotune(lat._h, 0.7, None, 0, C.byref(rows)) == 0  # accepted without scratch, as before
    assert rows.value == default and cache.read_text() == stale
    H = lat.autotune(0.7)
    lines = dict(line.split(" ") for line in cache.read_text().strip().split("\n"))
    assert len(lines) == 2 and lines[key] == "64" and str(H) in lines.values()
    again = smc_gpu.Lattice(d, n, L, 5, delta=1.0)
    assert again.autotune(0.7) == H and len(cache.read_text().strip().split("\n")) == 2


@pytest.mark.parametrize("d,L,kept", [(3, [8, 16], True), (3, [8, 10], False), (2, [16, 32], False)])
def test_batch_paths(smc_gpu, monkeypatch, tmp_path, d, L, kept):
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("SMC_AUTOTUNE_CACHE", str(cache))
    smc_gpu.Batch(d, L * 8, [0.4] * 16, seed=3).autotune()
    key = cache.read_text().split(" ")[0]
    old = key[:-3] if key.endswith(":p2") else key
    cache.write_text(f"{old} 128,0,0\n")
    b = smc_gpu.Batch(d, L * 8, [0.4] * 16, seed=3)
    th, lf = b.autotune()
    lines = cache.read_text().strip().split("\n")
    assert len(lines) == (1 if kept else 2)
    if kept:
        assert (th, lf) == (128, False) and not b.packed(0)
