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


def test_the_shape_that_the_tuner_reports_runs_what_it_timed(tmp_path):
    # a small state: quarters of tiles by default, also after the default shape is set by hand and after a
    # change of the tile and back; whole tiles in any other shape
    r = launches.run(tmp_path, """
    cfg = workloads.small(n_cells=512, ppc=64, rics="table", pairs=False, sort_interval=5)
    sim = Pic1D(cfg)
    def kernels(*shape):
        if shape:
            sim.set_push_shape(*shape)
        shim.forget()
        sim.step(2)
        return pushes()
    result = [kernels(), kernels(5, 8, 128), kernels(5, 16, 128), kernels(5, 8, 64), kernels(5, 8, 128)]
    tune = sim.autotune(2)
    sim.step(2)
    shim.forget()
    sim.step(2)
    tuned = pushes()
    again = Pic1D(cfg)
    again.set_push_shape(tune["push_blocks_per_cu"], tune["push_ppt"], tune["deposit_window"])
    shim.forget()
    again.step(2)
    result += [tuned, pushes()]
    """)
    quarters = [[2, 2, 128, 4]]
    assert r[:5] == [quarters, quarters, [[2, 16, 128, 1]], [[2, 8, 64, 1]], quarters]
    assert r[5] == r[6]


def test_the_tiles_of_a_new_size_are_counted_at_once(tmp_path):
    # 2.5 tiles a CU of 16 particles a lane are 5 of 8: halves, from the first step after the change
    r = launches.run(tmp_path, """
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    cells, n = 2048, n_cu * 1280
    cfg = workloads.small(n_cells=cells, ppc=1, init="empty", rics="exact", j_twist=0.0, pairs=False, sort_interval=0,
                          capacity=[n + 256, n + 256, 256, 256])
    sim = Pic1D(cfg)
    i = np.arange(n)
    for s in (0, 1):
        sim.set_particles(0, s, (i * cells // n).astype(np.int32), (i % 64 / 64).astype(np.float32),
                          np.zeros(n, np.float32), i.astype(np.uint64))
    sim.set_push_shape(6, 16, 32)
    sim.step(1)
    pushes()
    sim.set_push_shape(6, 8, 32)
    sim.step(1)
    result = pushes()
    """)
    assert r == [[1, 4, 32, 2]]
