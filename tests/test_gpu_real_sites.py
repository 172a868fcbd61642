"""Half-sweeps of real-valued updates, one or four sites a lane: rows of every
remainder (odd, two, a multiple of four), lattices below one workgroup and of
many, between the two kernels and against the float64 oracle."""
import numpy as np
import pytest
import torch

from test_gpu_continuous import _protocol

pytestmark = pytest.mark.gpu


def _lattice(smc, monkeypatch, d, n, L, kind, kernel):
    monkeypatch.setenv("SMC_BRICK", "0")
    for v in ("SMC_ISING_KERNEL", "SMC_CONT_KERNEL"):
        monkeypatch.delenv(v, raising=False)
    if kernel:
        monkeypatch.setenv("SMC_ISING_KERNEL" if n == 1 else "SMC_CONT_KERNEL", kernel)
    return smc.Lattice(d, n, L, 11, J_kind=kind, J_sigma=0.8, delta=1.3, renorm_every=0)


@pytest.mark.parametrize("d,L", [(2, 4), (2, 6), (2, 8), (2, 22), (2, 40), (2, 130), (2, 264), (2, 1102),
                                 (3, 4), (3, 6), (3, 8), (3, 10), (3, 16), (3, 30), (3, 56)])
def test_four_sites_a_lane_run_the_same_chain(smc_gpu, monkeypatch, d, L):
    print(f"FP32 couplings d={d} L={L}", flush=True)
    a, b = (_lattice(smc_gpu, monkeypatch, d, 1, L, 2, k) for k in (None, "site"))
    oa, ob = (torch.zeros(8, dtype=torch.int64, device="cuda") for _ in range(2))
    for _ in range(3):
        a.sweep_measure(0.7, 1, oa)
        b.sweep_measure(0.7, 1, ob)
        assert torch.equal(a.spins, b.spins)
        assert oa[1] == ob[1]
        e = float(oa.view(torch.float64)[2]), float(ob.view(torch.float64)[2])
        # N d terms below 8 summed in two orders
        assert abs(e[0] - e[1]) <= 2.0 ** -52 * 8 * d * (L ** d) ** 1.5
        assert e[0] == pytest.approx(_energy(a, d, L), rel=1e-11, abs=1e-9)


def _energy(lat, d, L):
    """Sum of -J s s over the bonds in float64 from the lattice's own arrays."""
    s = lat.spins.cpu().numpy().reshape(-1, 2, L ** d // 2).astype(np.float64)
    grid = np.empty((s.shape[0],) + (L,) * d)
    J = np.ones((d,) + (L,) * d)
    x = np.indices((L,) * d)          # axes z, y, x: the last is x
    colour = x.sum(0) & 1
    j = np.ravel_multi_index(tuple(x[:-1]) + (x[-1] // 2,), (L,) * (d - 1) + (L // 2,))
    for k in range(s.shape[0]):
        grid[k] = s[k][colour, j]
    if lat.J is not None:
        Jp = lat.J.cpu().numpy().reshape(d, 2, -1).astype(np.float64)
        for mu in range(d):
            J[mu] = Jp[mu][colour, j]
    return -sum(float((J[mu] * (grid * np.roll(grid, -1, axis=grid.ndim - 1 - mu)).sum(0)).sum())
                for mu in range(d))


@pytest.mark.parametrize("d,n,L,kind", [(2, 2, 6, 0), (2, 2, 22, 1), (2, 2, 1002, 0), (3, 2, 6, 2),
                                        (3, 2, 42, 0), (2, 3, 10, 0), (3, 3, 6, 1), (3, 3, 30, 2),
                                        (3, 3, 54, 0)])
def test_rows_of_odd_length(smc_gpu, oracle_mod, monkeypatch, d, n, L, kind):
    """Rows of L / 2 odd sites: the two sites of a draw may lie in two rows.
    Half-sweeps against the float64 oracle, and a measured sweep's record
    against the float64 sums of the state it left."""
    print(f"odd rows d={d} n={n} L={L} kind={kind}", flush=True)
    monkeypatch.setenv("SMC_BRICK", "0")
    if L < 100:
        _protocol(smc_gpu, oracle_mod, d, n, L, 0.6, 1.3, kind, False, "row")
    lat = _lattice(smc_gpu, monkeypatch, d, n, L, kind, None)
    obs = torch.zeros(8, dtype=torch.int64, device="cuda")
    lat.sweep_measure(0.6, 1, obs)
    f = obs.view(torch.float64)
    assert float(f[2]) == pytest.approx(_energy(lat, d, L), rel=1e-11, abs=1e-9)
    M = lat.spins.double().reshape(n, -1).sum(1)
    assert torch.allclose(f[3:3 + n], M, rtol=0, atol=1e-10 * L ** d)
