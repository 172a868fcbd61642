"""Short calls of chains of more pairs than lanes, either side of the lines between
the multi-pair and the LDS kernel: the same chains and sums by both."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _run(smc, d, L, kernel, monkeypatch, calls):
    if kernel:
        monkeypatch.setenv("SMC_CHAINS_KERNEL", kernel)
    else:
        monkeypatch.delenv("SMC_CHAINS_KERNEL", raising=False)
    gen = torch.Generator().manual_seed(3)
    J = 1.0 + 0.1 * torch.randn((d, 2, L ** d // 2), generator=gen)
    g = torch.randn((d, 2, L ** d // 2), generator=gen).double().cuda()
    ch = smc.Chains(d, L, 6, 11, J=J.cuda())
    centre = torch.full((1,), 0.25, dtype=torch.float64, device="cuda")
    out = []
    for n in calls:
        acc = ch.bond_zeros()
        cov, G = torch.zeros_like(g), torch.zeros(2, dtype=torch.float64, device="cuda")
        ch.sample(0.4, n, acc)
        ch.sample(0.4, n)
        ch.half_sweep(0.4, 0)
        ch.covariance(0.4, n, g, centre, cov, G)
        out.append((ch.spins.clone(), acc, cov, G))
    return out


@pytest.mark.parametrize("d,L,calls", [(2, 76, (1, 3, 4)), (2, 80, (1, 2, 9)), (2, 84, (1, 13, 14)), (2, 88, (1, 5, 6)),
                                       (2, 96, (1, 9)), (3, 14, (1, 2)), (3, 16, (1, 7, 8)), (3, 18, (1, 4, 5))])
def test_short_calls_by_either_kernel(smc_gpu, monkeypatch, d, L, calls):
    print(f"chains short d={d} L={L} {calls}", flush=True)
    got = _run(smc_gpu, d, L, None, monkeypatch, calls)
    ref = _run(smc_gpu, d, L, "lds", monkeypatch, calls)
    bonds = d * L ** d
    for n, (a, b) in zip(calls, zip(got, ref)):
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]), n
        # sums of 6 n samples of G - c, itself a sum over the bonds, in two orders
        scale = 6 * n * bonds * 4.0
        assert torch.allclose(a[2], b[2], rtol=0, atol=2.0 ** -52 * scale * 16), n
        assert torch.allclose(a[3], b[3], rtol=0, atol=2.0 ** -52 * scale * 16 * bonds), n
