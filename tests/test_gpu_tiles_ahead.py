"""Tile passes with the masks of several hits formed ahead: the oracle's chain
for every number of waves (2: one forms, one runs the passes), chunks that the
hits do not fill, partly filled workgroups and the extreme thresholds."""
import numpy as np
import pytest

import layout

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("waves", [None, 2, 5, 12])
@pytest.mark.parametrize("d,L,T,hits,hb,J0,beta", [
    (2, 32, 16, 1, False, 1.0, 0.4406868),      # 2 tiles a colour of a workgroup's 16
    (2, 160, 16, 19, False, 1.0, 2.0),          # three chunks of masks, the last of 3 hits
    (2, 96, 16, 9, True, 1.0, 0.4406868),
    (2, 64, 16, 3, False, -1.0, 0.5),           # J0 < 0: classes of satisfied bonds
    (2, 192, 32, 8, False, 1.0, 0.4406868),
    (2, 64, 32, 5, True, 1.0, float("inf")),    # thresholds 0, 2^31 and 2^32
    (2, 128, 64, 10, False, 1.0, 0.0),          # every move accepted
    (2, 384, 64, 2, True, -1.0, 0.3),
    (3, 32, 16, 9, False, 1.0, 0.2216546),
    (3, 64, 16, 2, True, 1.0, 0.25),
    (3, 32, 16, 3, False, -1.0, 1.0)])
def test_masks_ahead_match_oracle(smc_gpu, oracle_mod, monkeypatch, d, L, T, hits, hb, J0, beta, waves):
    print(f"masks ahead d={d} L={L} T={T} hits={hits} hb={hb} J0={J0} beta={beta} waves={waves}", flush=True)
    monkeypatch.delenv("SMC_PACKED_TIES", raising=False)
    if waves is None:
        monkeypatch.delenv("SMC_TILE_KERNEL", raising=False)
    else:
        monkeypatch.setenv("SMC_TILE_KERNEL", f"ahead,{waves}")
    lat = smc_gpu.Lattice(d, 1, L, seed=43, J0=J0, tile=T, hits=hits, heatbath=hb)
    ref = oracle_mod.OracleLattice(d, 1, L, 43, J0=J0)
    lat.sweep(beta, 2)
    ref.sweep_rule(beta, 2, "heatbath" if hb else "metropolis", T, hits)
    assert np.array_equal(layout.to_natural(lat.spins.cpu().numpy(), d, L), ref.s)
