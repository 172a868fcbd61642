"""Continuous spins: whichever kernel runs -- one site a lane, streaming with each
number of sites a lane, bricks -- the chain is the same bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu
VARS = ("SMC_CONT_KERNEL", "SMC_CONT_SPL", "SMC_CONT_ROWS", "SMC_BRICK", "SMC_XY_MARCH")


def _spins(smc, monkeypatch, env, d, n, L, kind, calls, **kw):
    for v in VARS:
        monkeypatch.delenv(v, raising=False)
    for v, x in env.items():
        monkeypatch.setenv(v, x)
    lat = smc.Lattice(d, n, L, 21, J_kind=kind, J0=0.9, J_sigma=0.6, delta=1.4, renorm_every=0, **kw)
    for k in calls:
        lat.sweep(0.8, k)
    return lat.spins.clone()


# either side of the lines between two and four sites a lane, by kind of coupling
@pytest.mark.parametrize("d,L,kind", [(3, 96, 0), (3, 104, 0), (3, 104, 1), (3, 112, 2), (3, 106, 1),
                                      (2, 1344, 1), (2, 1400, 0), (2, 1400, 1), (2, 1400, 2)])
def test_chosen_sites_a_lane(smc_gpu, monkeypatch, d, L, kind):
    print(f"sites a lane d={d} L={L} kind={kind}", flush=True)
    got = _spins(smc_gpu, monkeypatch, {"SMC_BRICK": "0"}, d, 2, L, kind, (2,))
    ref = _spins(smc_gpu, monkeypatch, {"SMC_CONT_KERNEL": "row"}, d, 2, L, kind, (2,))
    assert torch.equal(got, ref)


# every (dimension, components, kind of coupling), in the precise and the fast arithmetic
@pytest.mark.parametrize("fast", [False, True])
@pytest.mark.parametrize("d,n,kind", [(d, n, kind) for d in (2, 3) for n in (2, 3) for kind in (0, 1, 2)])
def test_every_kernel_runs_the_same_chain(smc_gpu, monkeypatch, d, n, kind, fast):
    print(f"cont kernels d={d} n={n} kind={kind} fast={fast}", flush=True)
    L, calls = (48, (3, 9)) if d == 2 else (16, (3, 9))
    ref = _spins(smc_gpu, monkeypatch, {"SMC_CONT_KERNEL": "row"}, d, n, L, kind, calls, fast_math=fast)
    ways = [{"SMC_CONT_KERNEL": "stream", "SMC_CONT_SPL": str(v), "SMC_CONT_ROWS": str(h)}
            for v in ((2, 4) if n == 2 else (1, 2)) for h in (4, 8)] + [{}]
    if not fast:
        # the whole lattice and bricks cut along y, with each number of positions a lane
        ways += [{"SMC_BRICK": f"{m},1,{ny},1,{v}"} for m, ny in ((9, 1), (2, 2)) for v in ((1, 2, 4) if n == 2 else (1, 2))]
    for env in ways:
        assert torch.equal(_spins(smc_gpu, monkeypatch, env, d, n, L, kind, calls, fast_math=fast), ref), env
