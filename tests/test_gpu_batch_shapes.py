"""The batch's packed path over the edges where it can go wrong: rows that
split words, last words partly filled, one-wave lattices filling and not
filling a workgroup beside lattices with a workgroup of their own, either
dimension and coupling kind, against the oracle; with and without a graph."""
import numpy as np
import pytest

import layout

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("threads", [64, 256])
@pytest.mark.parametrize("d,kind,J0,L", [
    (2, 0, 1.0, [4, 6, 10, 34, 62, 64, 66, 90, 128, 100]),
    (2, 1, 1.0, [64, 30, 8, 102, 16, 12]),
    (2, 1, -1.0, [6, 44, 96]),
    (3, 1, 1.0, [4, 6, 8, 10, 14, 16, 18, 22, 12]),
    (3, 0, 1.0, [16, 16, 16, 16, 16, 20]),
    (3, 1, -1.0, [10, 26, 6])])
def test_packed_batch_shapes(smc_gpu, oracle_mod, d, kind, J0, L, threads, graph):
    import torch
    print(f"batch shapes d={d} kind={kind} J0={J0} L={L} threads={threads} graph={graph}", flush=True)
    n = len(L)
    beta = [(0.44 if d == 2 else 0.25) + 0.2 * (r % 4) for r in range(n)]
    b = smc_gpu.Batch(d, L, beta, seed=91, J_kind=kind, J0=J0)
    b.threads = threads
    b.use_graph(graph)
    words = [-(-(e ** d // 2) // 32) for e in L]
    assert [b.packed(r) for r in range(n)] == [w <= 2 * threads for w in words]
    obs = torch.zeros((2, n, 8), dtype=torch.int64, device=b.device)
    b.sweep(2)
    b.sweep(4, obs, every=2)
    recs = smc_gpu.Lattice.decode_obs(obs)
    for r in range(n):
        ref = oracle_mod.OracleLattice(d, 1, L[r], 91, J_kind=kind, J0=J0, replica=r)
        for m, k in ((0, 4), (1, 2)):
            ref.sweep(beta[r], k)
            o = ref.measure()
            got = recs[m * n + r]
            assert (got.E_int, got.M_int, got.sweep) == (o.E_int, o.M_int, 2 * m + 4), (r, L[r])
        assert np.array_equal(layout.to_natural(b.spins_of(r).cpu().numpy(), d, L[r]), ref.s), (r, L[r])
