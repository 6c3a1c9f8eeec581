"""Which particle kernel a step launches, and when graphs are captured, as the number of tiles changes."""
import pytest

from . import launches

pytestmark = pytest.mark.gpu


def test_graphs_are_kept_across_the_switch_of_parts(tmp_path):
    # 768 and 16,384 tiles are the switches at 256 CUs; the state goes to either side of the first and back
    r = launches.run(tmp_path, """
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    few, many = 2 * n_cu * 512 // 2, 4 * n_cu * 512 // 2        # per species: 2 and 4 tiles a CU
    cells = 2048
    cfg = workloads.small(n_cells=cells, ppc=1, init="empty", rics="table", j_twist=0.0, pairs=False, sort_interval=3,
                          capacity=[many + 256, many + 256, 256, 256])
    sim = Pic1D(cfg)
    i = np.arange(many)
    part = ((i * cells // many).astype(np.int32), (i % 64 / 64).astype(np.float32), np.zeros(many, np.float32),
            i.astype(np.uint64))
    sim.set_graph(3)
    captured, kernels = [], []
    for k in range(12):
        n = few if k % 2 else many
        for s in (0, 1):
            sim.set_particles(0, s, *(a[many // n - 1::many // n] for a in part))
        assert sum(sim.moments(0)["count"]) == 2 * n
        shim.forget()
        sim.step(6)
        captured.append(shim.n_graphs())
        kernels.append(pushes())
    result = dict(captured=captured, kernels=kernels, step=sim.moments(0)["step"])
    sim.close()
    """)
    assert r["step"] == 72
    # one per live buffer set (a sort within each graph) and number of parts, in the first calls on either side
    assert r["captured"] == [2, 2] + [0] * 10
    assert r["kernels"][0] == [[2, 4, 128, 2]] and r["kernels"][1] == [[2, 2, 128, 4]]


@pytest.mark.parametrize("graph", [0, 10])
def test_a_long_call_follows_the_number_of_tiles(tmp_path, graph):
    # an empty line that the atmosphere fills in the first step: 0 tiles when the call begins, more
    # than 3 a CU for the rest of it
    r = launches.run(tmp_path, f"""
    graph = {graph}
    """ + """
    cells, ppc = 700, 800
    cfg = workloads.small(r_eq=8.0, n_cells=cells, ppc=ppc, init="empty", rics="table", atmosphere=True, pairs=False,
                          sort_interval=10, capacity=[256, 256, 4_000_000, 4_000_000])
    sim = Pic1D(cfg)
    if graph:
        sim.set_graph(graph)
    pushes()
    sim.step(1500)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    count = sim.moments(0)["count"]
    result = dict(kernels=pushes(), tiles=sum((c + 511) // 512 for c in count) / n_cu)
    sim.close()
    """)
    assert 3 < r["tiles"] <= 64
    assert r["kernels"] == [[2, 2, 128, 4], [2, 4, 128, 2]]
