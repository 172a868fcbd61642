"""Passes of two sweeps over a 2D XY lattice: the chain of the half-sweep
kernels bit for bit, whatever the bands, and the record to the rounding of a
double-precision sum taken in another order."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _run(smc, monkeypatch, rows, L, calls, renorm):
    monkeypatch.setenv("SMC_BRICK", "0")
    if rows is None:
        monkeypatch.delenv("SMC_XY_MARCH", raising=False)
    else:
        monkeypatch.setenv("SMC_XY_MARCH", str(rows))
    lat = smc.Lattice(2, 2, L, 29, J0=0.9, delta=1.2, renorm_every=renorm)
    obs = torch.zeros(8, dtype=torch.int64, device="cuda")
    out = []
    for k in calls:
        lat.sweep_measure(0.9, k, obs)
        out.append((lat.spins.clone(), obs.clone()))
    lat.sweep(0.9, 3)
    out.append((lat.spins.clone(), obs.clone()))
    return out


# the shortest rows (64 groups of four sites: two segments of 32), segments of
# uneven width, uneven bands, bands of two rows, one band, the chosen bands
@pytest.mark.parametrize("L,rows", [(512, 36), (512, 2), (520, 36), (520, 10000), (1000, 34), (992, 7),
                                    (2048, 18), (1736, 50), (3000, None)])
def test_passes_run_the_same_chain(smc_gpu, monkeypatch, L, rows):
    print(f"xy passes L={L} rows={rows}", flush=True)
    calls, renorm = (2, 3, 4, 5, 1, 10), 11  # one and two sweeps a pass; a renormalisation inside and after
    got = _run(smc_gpu, monkeypatch, rows, L, calls, renorm)
    ref = _run(smc_gpu, monkeypatch, 0, L, calls, renorm)
    for k, ((a, oa), (b, ob)) in enumerate(zip(got, ref)):
        assert torch.equal(a, b), f"spins after call {k}"
        assert oa[7] == ob[7]
        x, y = oa.view(torch.float64)[2:7], ob.view(torch.float64)[2:7]
        assert torch.allclose(x, y, rtol=0, atol=2.0 ** -52 * 16 * (L * L) ** 1.5), f"sums of call {k}"
