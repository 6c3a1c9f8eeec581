"""The surrogate pusher's work items (half tiles of 256 particles from a queue) at their edges: every
particle is pushed once, as the oracle pushes it."""
import numpy as np
import pytest

from paper_2609_17661_amd import Pic1D

from . import parity
from .test_gpu_mlp import _mlp_cfg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("counts", [(1, 0), (255, 256), (257, 511), (512, 513), (769, 3)])
def test_step_parity_at_half_tile_counts(counts):
    print("half tiles", counts, flush=True)
    cfg = _mlp_cfg(61, n_cells=64, ppc=1, init="empty", pairs=False)
    cfg["lines"].append(dict(cfg["lines"][0], n_cells=40))
    sim = Pic1D(cfg)
    rng = np.random.default_rng(62)
    for line in (0, 1):
        for s in (0, 1):
            n = counts[(s + line) & 1]
            gam = 10.0 ** rng.uniform(0, 3, n)
            u = (np.where(rng.random(n) < 0.5, -1, 1) * np.sqrt(gam**2 - 1)).astype(np.float32)
            sim.set_particles(line, s, rng.integers(0, sim.n_cells(line), n), rng.uniform(0.01, 0.99, n).astype(np.float32),
                              u, np.arange(n, dtype=np.uint64) * np.uint64(4) + np.uint64(2 * line + s))
    ocfg = parity.oracle_config(cfg)
    before_n = sim.moments(0)["counters"]["pushed"]
    for _ in range(2):
        before = parity.snapshot(sim)
        sim.step(1)
        rep, _ = parity.compare_step(ocfg, before, parity.snapshot(sim))
        print(rep, flush=True)
        assert rep["excused"] <= max(3, 1e-3 * rep["compared"])
    assert before_n == 0 and sim.moments(0)["counters"]["pushed"] <= 2 * sum(counts)
