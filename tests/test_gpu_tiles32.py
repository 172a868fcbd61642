"""Tiles of edge 32 at one bit per site: the oracle's chain, with whole and
partly filled workgroups, every way of resolving ties, and the int8 kernel."""
import numpy as np
import pytest

import layout

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ties", ["group", "lane"])
@pytest.mark.parametrize("d,L,hb,J0,beta,group", [
    (2, 64, False, 1.0, 0.4406868, "wave"),    # 2 tiles a colour: half of a wave
    (2, 192, False, 1.0, 2.0, "group"),        # 18 tiles a colour: the last workgroup partly filled
    (2, 320, True, 1.0, 0.4406868, "wave"),
    (2, 128, True, 1.0, float("inf"), "group"),
    (2, 64, False, -1.0, 0.5, "group"),        # J0 < 0: the general decision
    (3, 64, False, 1.0, 0.2216546, "wave"),    # a tile is a workgroup of 512
    (3, 64, False, 1.0, 1.5, "group"),
    (3, 64, True, 1.0, 0.25, "group"),
    (3, 64, False, -1.0, 0.3, "group")])
def test_tiles_of_32_match_oracle(smc_gpu, oracle_mod, monkeypatch, d, L, hb, J0, beta, group, ties):
    print(f"tiles of 32 d={d} L={L} hb={hb} J0={J0} beta={beta} {group} {ties}", flush=True)
    monkeypatch.setenv("SMC_TILE_KERNEL", group)
    monkeypatch.setenv("SMC_PACKED_TIES", ties)
    lat = smc_gpu.Lattice(d, 1, L, seed=37, J0=J0, tile=32, hits=3, heatbath=hb)
    ref = oracle_mod.OracleLattice(d, 1, L, 37, J0=J0)
    lat.sweep(beta, 2)
    ref.sweep_rule(beta, 2, "heatbath" if hb else "metropolis", 32, 3)
    assert np.array_equal(layout.to_natural(lat.spins.cpu().numpy(), d, L), ref.s)


@pytest.mark.parametrize("d,L,hb", [(2, 1024, False), (2, 1024, True), (3, 128, False), (3, 128, True)])
def test_tiles_of_32_match_the_byte_kernel(smc_gpu, monkeypatch, d, L, hb):
    import torch
    states = []
    for kernel in ("byte", None):
        if kernel:
            monkeypatch.setenv("SMC_TILE_KERNEL", kernel)
        else:
            monkeypatch.delenv("SMC_TILE_KERNEL", raising=False)
        lat = smc_gpu.Lattice(d, 1, L, seed=41, tile=32, hits=5, heatbath=hb)
        lat.sweep(0.4406868 if d == 2 else 0.2216546, 3)
        states.append(lat.spins.clone())
    assert torch.equal(*states)
