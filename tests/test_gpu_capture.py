"""The first call of a new handle captured into a graph: every replay runs the
captured sweeps (their counters are fixed) on the state it finds, with eager work and
synchronisations in between, and matches the same sweeps called eagerly."""
import pytest
import torch

pytestmark = pytest.mark.gpu

LATTICES = [  # d, n, L, keywords, sweeps, the kernel expected
    (2, 1, 100, dict(), 20, "ising_resident"), (2, 1, 1000, dict(), 20, "ising_resident"),
    (2, 1, 1024, dict(heatbath=True), 20, "ising_resident"), (3, 1, 64, dict(J_kind=1), 20, "ising_resident"),
    (2, 1, 256, dict(packed=True), 20, "ising_resident"), (2, 1, 8192, dict(), 10, "ising_packed"),
    (2, 1, 2048, dict(fused=True), 3, "ising_fused"), (3, 1, 40, dict(J_kind=2, J_sigma=0.7), 20, "ising_bricks"),
    (2, 2, 256, dict(delta=1.2), 10, "xy_bricks"), (2, 2, 3000, dict(delta=1.2), 4, "xy_march"),
    (3, 3, 24, dict(delta=1.2, renorm_every=7), 10, "heisenberg_bricks"), (3, 3, 128, dict(delta=1.2), 3, "heisenberg_stream"),
    (2, 1, 256, dict(tile=16, hits=9), 2, "ising_tiles_ahead"), (2, 1, 512, dict(tile=128, hits=3), 2, "ising_tiles_packed"),
    (2, 1, 1024, dict(tile=256, hits=3), 2, "ising_tiles")]


@pytest.mark.parametrize("d,n,L,kw,sweeps,name", LATTICES)
def test_captured_sweeps(smc_gpu, d, n, L, kw, sweeps, name):
    print(f"capture d={d} n={n} L={L} {kw}", flush=True)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ref = smc_gpu.Lattice(d, n, L, 33, **kw)
        lat = smc_gpu.Lattice(d, n, L, 33, **kw)
        a = torch.zeros(8, dtype=torch.int64, device="cuda")
        b = torch.zeros_like(a)
    stream.synchronize()
    assert lat.sweeps_kernel(sweeps, True)[0] == name
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        lat.sweep_measure(0.6, sweeps, a)
    assert lat.t == sweeps
    for replay in range(3):
        with torch.cuda.stream(stream):
            graph.replay()
            ref.t = 0
            ref.sweep_measure(0.6, sweeps, b)
            same = torch.equal(lat.spins, ref.spins) and torch.equal(a, b)  # (synchronises)
            assert same, replay
            a.zero_()
        assert lat.measure().E == ref.measure().E


@pytest.mark.parametrize("d,L", [(2, 64), (2, 88), (3, 16), (3, 18)])
def test_captured_chains(smc_gpu, d, L):
    print(f"capture chains d={d} L={L}", flush=True)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        J = 1.0 + 0.1 * torch.randn((d, 2, L ** d // 2), device="cuda")
        g = torch.randn_like(J).double()
        c = torch.full((1,), 0.5, dtype=torch.float64, device="cuda")
        runs = []
        for _ in range(2):
            ch = smc_gpu.Chains(d, L, 5, 7, J=J)
            runs.append((ch, ch.bond_zeros(), torch.zeros_like(g), torch.zeros(2, dtype=torch.float64, device="cuda")))
    stream.synchronize()

    def calls(ch, acc, cov, G):
        ch.sample(0.4, 16, acc)
        ch.covariance(0.4, 16, g, c, cov, G)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        calls(*runs[0])
    for replay in range(3):
        with torch.cuda.stream(stream):
            graph.replay()
            runs[1][0].t = 0
            calls(*runs[1])
            for x, y in zip(runs[0][1:], runs[1][1:]):
                assert torch.equal(x, y), replay
            assert torch.equal(runs[0][0].spins, runs[1][0].spins), replay


@pytest.mark.parametrize("d,edges", [(3, [4, 10, 16, 24, 40]), (2, [8, 62, 100, 256])])
def test_captured_batch(smc_gpu, d, edges):
    print(f"capture batch d={d} {edges}", flush=True)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        made = [smc_gpu.Batch(d, edges, [0.4 + 0.2 * r for r in range(len(edges))], seed=3) for _ in range(2)]
        obs = [torch.zeros((2, len(edges), 8), dtype=torch.int64, device="cuda") for _ in range(2)]
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        made[0].sweep(4, obs[0], every=2)
    for replay in range(3):
        with torch.cuda.stream(stream):
            graph.replay()
            made[1].t = 0
            made[1].sweep(4, obs[1], every=2)
            assert torch.equal(made[0].spins, made[1].spins) and torch.equal(*obs), replay
            obs[0].zero_()
