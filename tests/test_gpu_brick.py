"""Sweeps of bricks held in LDS: whatever the cut, the chain is that of the
half-sweep kernels bit for bit, and the record agrees to the rounding of a
double-precision sum taken in another order."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _run(smc, monkeypatch, brick, d, n, L, kind, calls, renorm):
    if brick is None:
        monkeypatch.delenv("SMC_BRICK", raising=False)
    else:
        monkeypatch.setenv("SMC_BRICK", brick)
    lat = smc.Lattice(d, n, L, 23, J_kind=kind, J0=-0.8 if kind == 1 else 1.0, J_sigma=0.7, delta=1.2,
                      renorm_every=renorm)
    obs = torch.zeros(8, dtype=torch.int64, device="cuda")
    out = []
    for k in calls:
        lat.sweep_measure(0.9, k, obs)
        out.append((lat.spins.clone(), obs.clone()))
    return out


# d, n, L, J kind, cut "sweeps,nx,ny,nz,V": whole lattices; bricks of uneven
# edges; one axis, then all cut; bricks as small as their halo allows
CUTS = [(2, 1, 16, 2, "9,1,1,1,2"), (2, 1, 64, 2, "2,1,3,1,4"), (2, 1, 50, 2, "1,3,4,1,1"),
        (3, 1, 12, 2, "9,1,1,1,2"), (3, 1, 14, 2, "1,1,2,2,1"), (3, 1, 40, 2, "2,2,5,5,2"),
        (2, 2, 30, 0, "9,1,1,1,1"), (2, 2, 36, 1, "3,2,2,1,2"), (2, 2, 96, 2, "4,2,3,1,4"),
        (3, 2, 16, 0, "1,2,2,2,4"), (3, 2, 18, 1, "2,1,2,2,1"), (3, 2, 20, 2, "2,1,2,2,2"),
        (2, 3, 20, 0, "9,1,1,1,2"), (2, 3, 44, 2, "2,2,2,1,2"), (3, 3, 10, 1, "9,1,1,1,1"),
        (3, 3, 24, 0, "2,2,2,3,2"), (3, 3, 26, 2, "1,1,3,4,1"), (3, 3, 4, 0, "5,1,1,1,2"),
        (2, 2, 4, 2, "5,1,1,1,1")]


@pytest.mark.parametrize("d,n,L,kind,cut", CUTS)
def test_bricks_run_the_same_chain(smc_gpu, monkeypatch, d, n, L, kind, cut):
    print(f"brick d={d} n={n} L={L} kind={kind} cut={cut}", flush=True)
    # renormalisations inside, at the end and across calls; odd and even
    # numbers of launches; single sweeps
    calls, renorm = (1, 2, 5, 4, 9, 3, 11), 7 if n == 2 else 0
    got = _run(smc_gpu, monkeypatch, cut, d, n, L, kind, calls, renorm)
    ref = _run(smc_gpu, monkeypatch, "0", d, n, L, kind, calls, renorm)
    for k, ((a, oa), (b, ob)) in enumerate(zip(got, ref)):
        assert torch.equal(a, b), f"spins after call {k}"
        assert torch.equal(oa[:2], ob[:2]) and oa[7] == ob[7], f"whole numbers of call {k}"
        x, y = oa.view(torch.float64)[2:7], ob.view(torch.float64)[2:7]
        # sums of at most N 2d terms of magnitude max|J| < 8 in two orders
        assert torch.allclose(x, y, rtol=0, atol=2.0 ** -52 * 16 * d * (L ** d) ** 1.5), f"sums of call {k}"


def test_chosen_cuts(smc_gpu, monkeypatch):
    """The cut the library picks, over the sizes where its choice changes."""
    for d, n, L, kind in [(2, 1, 32, 2), (2, 1, 130, 2), (2, 1, 512, 2), (3, 1, 40, 2), (3, 1, 62, 2),
                          (2, 2, 64, 0), (2, 2, 254, 0), (2, 2, 700, 0), (3, 2, 16, 0), (3, 2, 48, 0),
                          (3, 3, 12, 0), (3, 3, 30, 0), (3, 3, 64, 0)]:
        print(f"chosen d={d} n={n} L={L}", flush=True)
        got = _run(smc_gpu, monkeypatch, None, d, n, L, kind, (1, 10, 5), 100)
        ref = _run(smc_gpu, monkeypatch, "0", d, n, L, kind, (1, 10, 5), 100)
        for (a, _), (b, _) in zip(got, ref):
            assert torch.equal(a, b), (d, n, L)
