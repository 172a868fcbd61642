"""Bricks with halos in 3D -- cut along x, along all axes, one, two and four
positions a lane, each kind of coupling -- and the cuts the library picks: the
calls are asked which way they run, so none is compared with itself."""
import pytest
import torch

pytestmark = pytest.mark.gpu
NAMES = {1: "ising_bricks", 2: "xy_bricks", 3: "heisenberg_bricks"}


def _run(smc, monkeypatch, brick, d, n, L, kind, calls, expect=None):
    if brick is None:
        monkeypatch.delenv("SMC_BRICK", raising=False)
    else:
        monkeypatch.setenv("SMC_BRICK", brick)
    lat = smc.Lattice(d, n, L, 27, J_kind=kind, J0=-0.8 if kind == 1 else 1.0, J_sigma=0.7, delta=1.2,
                      renorm_every=0)
    obs = torch.zeros(8, dtype=torch.int64, device="cuda")
    out = []
    for k in calls:
        if expect:
            expect(k, lat.sweeps_kernel(k, True))
        lat.sweep_measure(0.9, k, obs)
        out.append((lat.spins.clone(), obs.clone()))
    return out


def _compare(got, ref, d, L):
    for k, ((a, oa), (b, ob)) in enumerate(zip(got, ref)):
        assert torch.equal(a, b), f"spins after call {k}"
        assert torch.equal(oa[:2], ob[:2]) and oa[7] == ob[7], f"whole numbers of call {k}"
        x, y = oa.view(torch.float64)[2:7], ob.view(torch.float64)[2:7]
        # sums of at most N 2d terms of magnitude max|J| < 8 in two orders
        assert torch.allclose(x, y, rtol=0, atol=2.0 ** -52 * 16 * d * (L ** d) ** 1.5), f"sums of call {k}"


# n, L, J kind, cut "sweeps,nx,ny,nz,V"; every call has more sweeps than a launch
@pytest.mark.parametrize("n,L,kind,cut", [
    (1, 20, 2, "2,5,5,4,1"), (1, 16, 2, "2,2,1,1,2"), (1, 32, 2, "3,4,4,7,4"), (1, 40, 2, "1,5,5,7,1"),
    (2, 24, 0, "2,3,2,4,4"), (2, 12, 1, "2,3,3,3,1"), (2, 40, 2, "2,5,5,7,2"), (2, 16, 0, "1,1,3,2,2"),
    (3, 20, 0, "2,5,5,7,1"), (3, 16, 1, "1,2,2,3,2"), (3, 12, 2, "2,3,3,4,2"), (3, 12, 0, "2,4,1,1,1")])
def test_cuts_in_3d(smc_gpu, monkeypatch, n, L, kind, cut):
    print(f"brick cut n={n} L={L} kind={kind} cut={cut}", flush=True)
    per = int(cut.split(",")[0])

    def bricks(k, way):
        assert way == (NAMES[n], -(-k // per))
    calls = (4, 5, 11)
    got = _run(smc_gpu, monkeypatch, cut, 3, n, L, kind, calls, bricks)
    ref = _run(smc_gpu, monkeypatch, "0", 3, n, L, kind, calls)
    _compare(got, ref, 3, L)


@pytest.mark.parametrize("d,n,L,kind", [(2, 1, 32, 2), (2, 1, 130, 2), (2, 1, 512, 2), (3, 1, 40, 2),
                                        (2, 2, 64, 0), (2, 2, 254, 1), (2, 2, 700, 0), (3, 2, 16, 2),
                                        (3, 2, 48, 0), (2, 3, 48, 0), (3, 3, 12, 1), (3, 3, 30, 0)])
def test_picked_cuts(smc_gpu, monkeypatch, d, n, L, kind):
    print(f"brick picked d={d} n={n} L={L} kind={kind}", flush=True)

    def bricks(k, way):  # (a short call may stay with half-sweeps)
        assert k < 10 or way[0] == NAMES[n] and way[1] <= k, way
    got = _run(smc_gpu, monkeypatch, None, d, n, L, kind, (10, 20, 5), bricks)
    ref = _run(smc_gpu, monkeypatch, "0", d, n, L, kind, (10, 20, 5),
               lambda k, way: way[1] == 2 * k or pytest.fail(str(way)))
    _compare(got, ref, d, L)
