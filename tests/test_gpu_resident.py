"""Multi-sweep calls that run several half-sweeps a launch (the lattice's words
in LDS), or on a packed copy of an int8 lattice: bit for bit the oracle's
chain, and the half-sweep kernels' chain where the oracle is too slow.

SMC_RESIDENT=steps,own[,drawn] fixes the half-sweeps of a launch and the words a
workgroup owns (own at least the plane's words: one workgroup and no halo) and
whether the masks are formed by a launch of their own;
SMC_RESIDENT=0 keeps one launch a half-sweep."""
import numpy as np
import pytest

import layout

pytestmark = pytest.mark.gpu

INF = float("inf")
CASES = [  # d, L, kind, heatbath, packed, J0, beta, sweeps, "steps,own"
    # one workgroup: edges whose rows split words, whose last word is partly
    # filled, and of whole words; chunks of one and of several half-sweeps
    (2, 4, 0, False, False, 1.0, 0.4406868, 6, "128,2048"),
    (2, 6, 1, False, False, 1.0, 0.9, 5, "3,2048"),
    (2, 10, 0, True, False, 1.0, 0.4406868, 4, "1,2048"),
    (2, 34, 1, True, False, 1.0, 0.7, 4, "5,2048"),
    (2, 64, 0, False, True, -1.0, 0.4406868, 7, "128,2048"),
    (2, 100, 1, False, False, -0.7, 0.8, 3, "4,2048"),
    (2, 256, 0, False, False, 1.0, 0.0, 2, "2,2048"),
    (2, 362, 0, False, False, 1.0, 0.5, 2, "1,2048"),       # 2048 words a colour: the most
    (3, 4, 1, False, False, 1.0, 0.8, 6, "128,2048"),
    (3, 6, 0, True, False, 1.0, 0.2216546, 4, "2,2048"),
    (3, 10, 1, True, False, 1.0, 1.0, 3, "3,2048"),
    (3, 18, 1, False, False, 1.0, INF, 3, "2,2048"),
    (3, 40, 1, False, False, 1.0, 1.0, 2, "1,2048"),
    (3, 64, 0, False, False, -1.0, 0.2216546, 2, "2,2048"),  # does not fit one: half-sweeps
    # bands with a halo: the plane's end inside a band, partly filled last
    # words, a last workgroup with fewer words, one half-sweep a launch
    (2, 100, 0, False, False, 1.0, 0.4406868, 5, "2,16"),
    (2, 100, 1, True, False, 1.0, 0.9, 3, "3,40"),
    (2, 102, 1, False, False, 1.0, 0.9, 4, "1,8"),
    (2, 128, 0, False, False, 1.0, 0.4406868, 70, "7,33"),   # more than 64 sweeps
    (2, 128, 1, False, True, 1.0, 1.2, 4, "4,64"),
    (2, 192, 0, True, False, 1.0, 0.4406868, 3, "6,100"),
    (2, 256, 0, False, True, 1.0, 0.4406868, 6, "4,128"),
    (3, 16, 1, False, False, 1.0, 1.0, 3, "2,24"),
    (3, 20, 1, True, False, 1.0, 0.8, 3, "3,16"),
    (3, 22, 0, False, False, 1.0, 0.2216546, 4, "2,60"),
    (3, 64, 1, False, False, 1.0, 1.0, 2, "2,64"),
    (3, 64, 1, False, True, -1.0, 1.0, 2, "4,100"),
    # the masks from memory: either shape, every class count, last words partly
    # filled, more steps than the masks held in LDS
    (2, 4, 0, False, False, 1.0, 0.4406868, 6, "128,2048,drawn"),
    (2, 100, 1, True, False, 1.0, 0.9, 3, "3,40,drawn"),
    (2, 102, 1, False, False, -1.0, 0.9, 4, "1,8,drawn"),
    (2, 256, 0, False, True, 1.0, 0.0, 5, "3,2048,drawn"),
    (2, 128, 0, False, False, 1.0, 0.4406868, 70, "7,33,drawn"),
    (3, 10, 1, True, False, 1.0, 1.0, 3, "3,2048,drawn"),
    (3, 22, 0, False, False, 1.0, INF, 4, "2,60,drawn"),
    (3, 64, 1, False, False, 1.0, 1.0, 2, "4,100,drawn"),
]


@pytest.mark.parametrize("d,L,kind,hb,packed,J0,beta,n,split", CASES)
def test_resident_sweeps_match_oracle(smc_gpu, oracle_mod, monkeypatch, d, L, kind, hb, packed, J0,
                                      beta, n, split):
    import torch
    print(f"resident d={d} L={L} kind={kind} hb={hb} packed={packed} J0={J0} {split}", flush=True)
    monkeypatch.setenv("SMC_RESIDENT", split)
    lat = smc_gpu.Lattice(d, 1, L, seed=L + n, J_kind=kind, J0=J0, heatbath=hb, packed=packed)
    ref = oracle_mod.OracleLattice(d, 1, L, L + n, J_kind=kind, J0=J0)
    obs = torch.zeros(8, dtype=torch.int64, device="cuda")
    lat.sweep(beta, 1)
    lat.sweep_measure(beta, n, obs)
    ref.sweep_rule(beta, n + 1, "heatbath" if hb else "metropolis")
    s = lat.spins
    if packed:
        s = smc_gpu.unpack_spins(s.view(-1))
    s = s.cpu().numpy().reshape(2, -1)
    assert np.array_equal(layout.to_natural(s, d, L), ref.s)
    o, r = lat.decode_obs(obs)[0], ref.measure()
    assert (o.E_int, o.M_int, o.sweep) == (r.E_int, r.M_int, n + 1) and o.E == r.E
    assert lat.t == n + 1


@pytest.mark.parametrize("d,L,kind,hb,packed", [
    (2, 1000, 0, False, False), (2, 1000, 1, True, False), (2, 2048, 1, False, False),
    (2, 2050, 0, False, False), (2, 4096, 0, False, True), (2, 4096, 0, True, False),
    (3, 64, 1, False, False), (3, 100, 0, False, False), (3, 128, 1, False, True),
    (3, 130, 0, True, False), (3, 256, 1, False, False)])
def test_planned_sweeps_match_half_sweeps(smc_gpu, monkeypatch, d, L, kind, hb, packed):
    """The split the library chooses by itself, at the counts of sweeps where
    the choice changes, against one launch a half-sweep."""
    import torch
    print(f"planned d={d} L={L} kind={kind} hb={hb} packed={packed}", flush=True)
    monkeypatch.setenv("SMC_RESIDENT", "0")
    half = smc_gpu.Lattice(d, 1, L, seed=5, J_kind=kind, heatbath=hb, packed=packed)
    monkeypatch.delenv("SMC_RESIDENT")
    lat = smc_gpu.Lattice(d, 1, L, seed=5, J_kind=kind, heatbath=hb, packed=packed)
    a = torch.zeros(8, dtype=torch.int64, device="cuda")
    b = torch.zeros_like(a)
    for n in (1, 2, 5, 10):
        lat.sweep_measure(0.6, n, a)
        half.sweep_measure(0.6, n, b)
        assert torch.equal(lat.spins, half.spins) and torch.equal(a, b), n
