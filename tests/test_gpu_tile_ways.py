"""Which kernel a tiled call runs, by launch size, rule and hits, and that the
chain does not depend on it."""
import pytest
import torch

pytestmark = pytest.mark.gpu
AHEAD, PASSES = "ising_tiles_ahead", "ising_tiles_packed"


# either side of the lines between the kernels: launches of few hits and of a full
# chip form the masks in the passes (in 3D always from L = 448 on)
@pytest.mark.parametrize("d,L,T,hits,hb,way", [
    (2, 1024, 16, 1, False, AHEAD), (2, 4096, 16, 1, False, PASSES), (2, 4096, 16, 2, False, AHEAD),
    (2, 4096, 32, 3, False, PASSES), (2, 4096, 32, 4, False, AHEAD), (2, 4096, 64, 1, False, PASSES),
    (2, 4096, 64, 2, False, AHEAD), (2, 2880, 16, 1, True, PASSES), (2, 2880, 16, 2, True, AHEAD),
    (2, 4096, 64, 9, True, PASSES), (3, 224, 16, 5, True, PASSES), (3, 128, 16, 1, False, AHEAD), (3, 192, 16, 1, False, PASSES),
    (3, 192, 16, 2, True, AHEAD), (3, 256, 16, 11, False, PASSES), (3, 256, 16, 12, False, AHEAD),
    (3, 448, 16, 20, False, PASSES)])
def test_tile_ways(smc_gpu, monkeypatch, d, L, T, hits, hb, way):
    print(f"tile way d={d} L={L} T={T} hits={hits} hb={hb}", flush=True)
    out = []
    for kernel, name in ((None, way), ("byte", "ising_tiles")):
        if kernel:
            monkeypatch.setenv("SMC_TILE_KERNEL", kernel)
        else:
            monkeypatch.delenv("SMC_TILE_KERNEL", raising=False)
        lat = smc_gpu.Lattice(d, 1, L, seed=47, tile=T, hits=hits, heatbath=hb)
        assert lat.sweeps_kernel(3) == (name, 6)
        lat.sweep(0.4406868 if d == 2 else 0.2216546, 2)
        out.append(lat.spins.clone())
    assert torch.equal(*out)
