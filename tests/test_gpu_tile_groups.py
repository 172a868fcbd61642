"""The bit-packed tiles in workgroups of 64 and of 256 lanes
(SMC_TILE_KERNEL=wave / group): the oracle's chain either way, with whole and
partly filled workgroups and every way of resolving ties."""
import numpy as np
import pytest

import layout

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ties", ["group", "lane"])
@pytest.mark.parametrize("group", ["wave", "group"])
@pytest.mark.parametrize("d,L,T,hb,J0", [
    (2, 160, 16, False, 1.0), (2, 32, 16, True, 1.0), (2, 64, 16, False, -1.0),
    (2, 384, 64, False, 1.0), (2, 128, 64, True, 1.0), (2, 256, 128, False, 1.0),
    (3, 32, 16, False, 1.0), (3, 64, 16, True, 1.0), (3, 32, 16, False, -1.0)])
def test_tile_groups_match_oracle(smc_gpu, oracle_mod, monkeypatch, d, L, T, hb, J0, group, ties):
    print(f"tile groups d={d} L={L} T={T} hb={hb} J0={J0} {group} {ties}", flush=True)
    monkeypatch.setenv("SMC_TILE_KERNEL", group)
    monkeypatch.setenv("SMC_PACKED_TIES", ties)
    lat = smc_gpu.Lattice(d, 1, L, seed=31, J0=J0, tile=T, hits=4, heatbath=hb)
    ref = oracle_mod.OracleLattice(d, 1, L, 31, J0=J0)
    lat.sweep(0.4406868 if d == 2 else 0.2216546, 2)
    ref.sweep_rule(0.4406868 if d == 2 else 0.2216546, 2, "heatbath" if hb else "metropolis", T, 4)
    assert np.array_equal(layout.to_natural(lat.spins.cpu().numpy(), d, L), ref.s)
