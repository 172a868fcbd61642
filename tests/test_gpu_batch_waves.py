"""Batches with one, some and all of a workgroup's waves on a lattice each: the
chains and records of the one byte per site path."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("threads,count,edges", [
    (64, 40, [4, 10]), (256, 1024, [4]), (256, 1100, [4]),        # tiny: one and two a workgroup
    (256, 90, [10]), (256, 90, [4, 10]), (256, 2100, [4, 10]),    # others: four; beside tiny ones
    (256, 700, [4, 10, 24]), (256, 60, [24, 4]), (1024, 300, [4, 10]),  # beside single lattices
    (1024, 4097, [4]), (1024, 4099, [10]), (1024, 600, [4, 18])])  # all sixteen; at most eight
def test_lattices_a_workgroup(smc_gpu, monkeypatch, threads, count, edges, graph):
    print(f"batch waves threads={threads} count={count} edges={edges} graph={graph}", flush=True)
    out = []
    for packed in ("1", "0"):
        monkeypatch.setenv("SMC_BATCH_PACKED", packed)
        b = smc_gpu.Batch(3, [edges[r % len(edges)] for r in range(count)], [0.3 + 0.01 * (r % 50) for r in range(count)],
                          seed=9)
        b.set_schedule(threads, True)
        b.use_graph(graph)
        obs = torch.zeros((2, count, 8), dtype=torch.int64, device="cuda")
        b.sweep(4, obs, every=2)
        out.append((b.spins.clone(), obs))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
