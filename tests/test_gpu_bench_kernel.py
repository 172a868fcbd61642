"""The benchmark line names the kernel that its calls ran, and counts its launches."""
import os
import sys

import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench

pytestmark = pytest.mark.gpu

ISING2 = dict(d=2, n=1, seed=1, beta=0.4406868)
CASES = [  # workload, arguments, kernel, launches a call
    (dict(ISING2, L=64), ["--heatbath"], "ising_resident", 1),
    (dict(ISING2, L=64), ["--heatbath", "--sweeps-per-step", "1"], "ising_resident", 1),
    (dict(ISING2, L=8192), ["--heatbath"], "ising_resident", 10),
    (dict(ISING2, L=8192), [], "ising_packed", 20),
    (dict(ISING2, L=512), ["--tile", "64", "--hits", "20"], "ising_tiles_ahead", 20),
    (dict(ISING2, L=8192), ["--tile", "16", "--hits", "1"], "ising_tiles_packed", 20),
    (dict(ISING2, L=384), ["--tile", "96", "--hits", "2"], "ising_tiles", 20),
    (dict(d=2, n=2, L=3000, seed=1, beta=1.1, delta=1.2, renorm=100), [], "xy_march", 6),
    (dict(d=2, n=2, L=64, seed=1, beta=1.1, delta=1.2, renorm=100), [], "xy_bricks", None),
]


@pytest.mark.parametrize("wl,extra,name,launches", CASES)
def test_line_names_the_kernel_of_its_calls(smc_gpu, monkeypatch, wl, extra, name, launches):
    import torch
    print(f"bench line {wl} {extra}", flush=True)
    monkeypatch.setattr(sys, "argv", ["bench.py", "--steps", "2", "--warmup", "1", "--cpu-seconds", "0",
                                      "--no-int8-line", "--no-autotune"] + extra)
    seen = []
    inner = smc_gpu.Lattice.sweeps_kernel
    monkeypatch.setattr(smc_gpu.Lattice, "sweeps_kernel",
                        lambda self, n, measured=False: seen.append(inner(self, n, measured)) or seen[-1])
    r = bench.run_lattice(bench.parse(), wl, torch, smc_gpu)
    assert r["config"]["kernel"] == r["roofline"]["kernel"] == name == seen[0][0]
    assert launches in (None, seen[0][1])
    assert abs(r["roofline"]["kernel_avg_us"] * seen[0][1] / 1e3 - r["ms_per_step"]) <= 1e-3 * (1 + seen[0][1])
