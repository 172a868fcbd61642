"""One call of many sweeps of a lattice that a single workgroup holds: the chain
of the same sweeps made in shorter calls, spins and record bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu


# past 2^16 half-sweeps: FP32 couplings; vector spins without a renormalisation
# that would cut the call
@pytest.mark.parametrize("d,n,L,kind", [(2, 1, 4, 2), (3, 1, 6, 2), (2, 2, 4, 0), (3, 3, 4, 1)])
def test_long_calls_run_every_sweep(smc_gpu, d, n, L, kind):
    print(f"long call d={d} n={n} L={L} kind={kind}", flush=True)
    out = []
    for calls in ([33000], [11000] * 3):
        lat = smc_gpu.Lattice(d, n, L, 31, J_kind=kind, J_sigma=0.7, delta=1.2, renorm_every=0)
        obs = torch.zeros(8, dtype=torch.int64, device="cuda")
        for k in calls:
            lat.sweep_measure(0.3, k, obs)
        out.append((lat.spins.clone(), obs))
        assert lat.t == 33000
    (a, oa), (b, ob) = out
    assert torch.equal(a, b) and torch.equal(oa, ob)
