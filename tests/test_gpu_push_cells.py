"""What the particle kernel reads and writes per cell, at its edges: the field beside the walls, table
rows that a cell straddles or that are clamped, columns at both ends of the table, deposits into the
window's cells beyond the walls.  One step against the oracle."""
import numpy as np
import pytest

from paper_2609_17661_amd import Pic1D, workloads

from . import parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rics,cells,ns,nlg,gamma_max", [
    ("off", 2, 512, 256, 1e3),
    ("exact", 3, 512, 256, 1e3),
    ("table", 2, 2, 64, 1e3),           # two rows, every cell at a clamped end
    ("table", 3, 512, 256, 1e3),        # many rows a cell: every particle forms its own
    ("table", 130, 40, 256, 1e3),       # cells between two rows, straddling one, and at the ends
    ("table", 130, 40, 9, 3e8),         # momenta beyond the last column
    ("table", 700, 512, 256, 1.5),      # the first columns
])
def test_cells_at_the_edges(rics, cells, ns, nlg, gamma_max):
    print("cells", rics, cells, ns, nlg, gamma_max, flush=True)
    cfg = workloads.small(n_cells=cells, ppc=24, rics=rics, gamma_max=gamma_max, table_ns=ns, table_nlg=nlg, pairs=True)
    sim = Pic1D(cfg)
    rng = np.random.default_rng(cells)
    sim.set_field(0, rng.normal(0.0, 1e-3, cells))
    for _ in range(2):
        before = parity.snapshot(sim)
        sim.step(1)
        rep, _ = parity.compare_step(parity.oracle_config(cfg), before, parity.snapshot(sim))
        print(rep, flush=True)
        assert rep["excused"] <= max(2, rep["compared"] // 50)
    sim.close()
