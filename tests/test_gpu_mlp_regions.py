"""Photon records of the surrogate pusher: an append region's fill follows from the particles, not from
which wavefront takes which item of the queue."""
import numpy as np
import pytest

from oracle import mlp as omlp
from paper_2609_17661_amd import Pic1D, workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("attempt", range(3))
def test_every_region_filled_to_its_last_record(attempt):
    # 256 items of 256 leptons, each of which scatters (the network's outputs are constants: no force,
    # a rate far above one event a step) into a photon that converts; a region holds 256 records
    # (the least, at these capacities): one item fills one region, two in one would overflow it; cells near a
    # foot of the line, all in the stochastic regime
    print("regions", attempt, flush=True)
    n, cells = 65536, 64
    cfg = workloads.small(n_cells=cells, ppc=1, init="empty", rics="mlp", pairs=True, j_twist=0.0, nmax_over_n0=1e7,
                          sort_interval=0, capacity=[2 * n, n, 256, 256])
    cfg["mlp_params"] = np.zeros(omlp.N_PARAM, np.float32)
    cfg["mlp_norm"] = np.array([-30.0, 9.0, 0.0, 1.0, 1.0, 1.0], np.float32)
    sim = Pic1D(cfg)
    i = np.arange(n)
    sim.set_particles(0, 0, (4 + i * 16 // n).astype(np.int32), (i % 64 / 64).astype(np.float32),
                      np.where(i % 2 == 0, 1e4, -1e4).astype(np.float32), i.astype(np.uint64))
    sim.step(1)
    c = sim.moments(0)["counters"]
    print(c, flush=True)
    assert c["events"] == n and c["pairs_created"] == n and c["pushed"] == n
    sim.close()
