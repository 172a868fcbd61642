"""The covariance replay from a kept start: the sums of the replay that moves
the chains, bit for bit, with the chains left where they are."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kernel", ["pair", "lds"])
@pytest.mark.parametrize("d,L,count,sweeps", [(2, 4, 3, 1), (2, 64, 20, 9), (2, 96, 5, 8), (3, 8, 17, 10)])
def test_replay_equals_covariance(smc_gpu, monkeypatch, d, L, count, sweeps, kernel):
    print(f"replay d={d} L={L} count={count} {kernel}", flush=True)
    if kernel == "lds":
        monkeypatch.setenv("SMC_CHAINS_KERNEL", "lds")
    gen = torch.Generator(device="cuda").manual_seed(3)
    shape = (d, 2, L ** d // 2)
    J = 1.0 + 0.2 * torch.randn(shape, generator=gen, device="cuda")
    g = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float64)
    centre = torch.full((1,), 0.7, dtype=torch.float64, device="cuda")
    ch = smc_gpu.Chains(d, L, count, 5, J=J)
    ch.sample(0.4, 3)
    start, t0 = ch.spins.clone(), ch.t
    cov = torch.zeros(shape, dtype=torch.float64, device="cuda")
    G = torch.zeros(2, dtype=torch.float64, device="cuda")
    ch.covariance(0.4, sweeps, g, centre, cov, G)
    # the chains move on, under other couplings
    ch.set_couplings(J * 0.5)
    ch.sample(0.4, 4)
    end, t_end, J_end = ch.spins.clone(), ch.t, ch.J.clone()
    for _ in range(2):  # into fresh buffers, whatever they hold
        cov2, G2 = ch.replay(0.4, sweeps, t0, J, start, g, centre)
        assert torch.equal(cov, cov2) and torch.equal(G, G2)
    assert torch.equal(ch.spins, end) and ch.t == t_end and torch.equal(ch.J, J_end)


@pytest.mark.parametrize("d,L,count,sweeps", [(3, 4, 9, 1), (3, 6, 5, 8), (3, 8, 7, 19), (3, 12, 3, 9), (3, 14, 2, 5),
                                              (3, 16, 2, 8), (3, 18, 3, 10), (2, 16, 6, 17), (2, 68, 3, 9),
                                              (2, 80, 2, 16), (2, 96, 2, 7)])
def test_covariance_pair_and_lds(smc_gpu, monkeypatch, d, L, count, sweeps):
    """Both kernels' samples and replays: the same chains; sums of the same
    terms in two orders (3D: one wave, several, the most lanes the pair kernel
    takes, and past them; both: two and three pairs a lane, all lanes full)."""
    print(f"covariance kernels d={d} L={L}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(4)
    shape = (d, 2, L ** d // 2)
    J = 1.0 + 0.2 * torch.randn(shape, generator=gen, device="cuda")
    g = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float64)
    centre = torch.full((1,), -0.3, dtype=torch.float64, device="cuda")
    out = []
    for kernel in ("pair", "lds"):
        if kernel == "lds":
            monkeypatch.setenv("SMC_CHAINS_KERNEL", "lds")
        else:
            monkeypatch.delenv("SMC_CHAINS_KERNEL", raising=False)
        ch = smc_gpu.Chains(d, L, count, 6, J=J)
        bonds = ch.bond_zeros()
        ch.sample(0.25, 2, bonds)
        ch.half_sweep(0.25, 1)
        cov = torch.zeros(shape, dtype=torch.float64, device="cuda")
        G = torch.zeros(2, dtype=torch.float64, device="cuda")
        ch.covariance(0.25, sweeps, g, centre, cov, G)
        out.append((ch.spins.clone(), cov, G, bonds))
    (sa, ca, Ga, ba), (sb, cb, Gb, bb) = out
    assert torch.equal(sa, sb) and torch.equal(ba, bb)
    most = float(g.abs().sum()) + 0.3          # of |G - centre|
    eps, S = 2.0 ** -52, count * sweeps
    err = eps * most * (d * L ** d + S) * S    # rounding of each G and of the sums over S samples
    assert float((ca - cb).abs().max()) <= err and abs(float(Ga[0] - Gb[0])) <= err
    assert abs(float(Ga[1] - Gb[1])) <= 2 * most * err


def test_replay_refuses_no_sweeps(smc_gpu):
    ch = smc_gpu.Chains(2, 8, 2, 5)
    z = torch.zeros((2, 2, 32), dtype=torch.float64, device="cuda")
    with pytest.raises(smc_gpu.SmcError):
        ch.replay(0.4, 0, 0, ch.J, ch.spins, z, torch.zeros(1, dtype=torch.float64, device="cuda"))
