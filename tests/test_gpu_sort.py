"""The cell sort at the edges of its tiles, windows and scans: particles at rest in random order
keep every value and come out in bin order."""
import numpy as np
import pytest

from paper_2609_17661_amd import Pic1D, workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cells,count,sub", [
    (2, 1, 8),              # one particle
    (64, 4095, 1),          # one short of a tile, one window
    (64, 4096, 8),          # a tile
    (256, 4097, 32),        # one more; 8,192 bins: four windows
    (512, 20000, 32),       # 16,384 bins: the most windows
    (520, 20000, 32),       # beyond: straight to the global bins
    (1024, 9000, 8),        # the longest line scanned by one block
    (1025, 9000, 8),        # beyond: chunks over blocks
])
def test_sort_keeps_particles_and_orders_them(cells, count, sub):
    print("sort", cells, count, sub, flush=True)
    cfg = workloads.small(n_cells=cells, ppc=1, init="empty", rics="off", j_twist=0.0, pairs=False,
                          capacity=[count + 1, count // 3 + 1, 300, 300])
    cfg["lines"].append(dict(cfg["lines"][0], n_cells=3))
    cfg["sort_interval"] = 1
    sim = Pic1D(cfg)
    sim.set_sort_granularity(sub)
    rng = np.random.default_rng(count)
    put = {}
    for line, s, n in ((0, 0, count), (0, 1, count // 3), (1, 0, 7), (1, 3, 2)):
        p = dict(cell=rng.integers(0, cells if line == 0 else 3, n).astype(np.int32),
                 off=(rng.integers(0, 1 << 24, n) * 2.0**-24).astype(np.float32),
                 u=(rng.integers(-50, 50, n) * 1e-30).astype(np.float32),      # too slow to move
                 id=rng.permutation(n).astype(np.uint64) + np.uint64(1 << 40))
        sim.set_particles(line, s, p["cell"], p["off"], p["u"], p["id"])
        put[line, s] = p
    sim.step(1)
    for (line, s), p in put.items():
        got = sim.get_particles(line, s)
        key = got["cell"] * sub + np.minimum(np.floor(got["off"] * np.float32(sub)).astype(np.int64), sub - 1)
        assert np.all(np.diff(key) >= 0)
        a, b = np.argsort(p["id"]), np.argsort(got["id"])
        for k in p:
            assert np.array_equal(p[k][a], got[k][b]), k
