"""Parts of tiles against whole tiles (of the default tile with the other deposit window, which no rule
divides): the same bits, at tile counts on both sides of the switches and across a change of count."""
import numpy as np
import pytest

from paper_2609_17661_amd import Pic1D, workloads

from .test_gpu_push_parts import _moments

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rics,cells,ppc,graph", [
    ("table", 3, 1, 0),            # one item, nearly empty
    ("exact", 64, 40, 0),          # a few tiles: quarters
    ("off", 700, 200, 3),          # 547: quarters from graphs
    ("table", 3000, 300, 0),       # 3,516 tiles: halves
    ("exact", 3000, 300, 3),
    ("off", 3000, 300, 0),
    ("table", 9000, 300, 0),       # 10,547
    ("table", 15000, 300, 0),      # 17,579: whole tiles of themselves
])
def test_parts_and_whole_tiles_give_the_same_results(rics, cells, ppc, graph):
    print("whole", rics, cells, ppc, graph, flush=True)
    cfg = workloads.small(n_cells=cells, ppc=ppc, rics=rics, pairs=True, atmosphere=cells < 1000, nmax_over_n0=4.0,
                          gamma_max=1e4, sort_interval=3,
                          capacity=[4 * cells * ppc + 20000, 4 * cells * ppc + 20000, 600_000, 600_000])
    out = []
    for whole in (False, True):
        sim = Pic1D(cfg)
        if whole:
            sim.set_push_shape(5, 8, 64)
        if graph:
            sim.set_graph(graph)
        sim.step(4)
        # fewer particles: another number of parts from here on
        if cells == 3000:
            for s in (0, 1):
                p = sim.get_particles(0, s)
                keep = np.argsort(p["id"])[: cells * 40]
                sim.set_particles(0, s, *(p[k][keep] for k in ("cell", "off", "u", "id")))
        sim.step(7)
        out.append(_moments(sim))
        sim.close()
    for a, b in zip(*out):
        assert np.array_equal(a, b)
