"""A state frozen by an error inside a call of many steps, with sorts queued behind the error: its
particles are the ones of the step that was not completed, however many steps the call asked for."""
import numpy as np
import pytest

from paper_2609_17661_amd import Pic1D, Pic1dError, workloads
from paper_2609_17661_amd.pic1d import STATUS

pytestmark = pytest.mark.gpu

CELLS, PPC = 64, 40


def _sim(rics="exact"):
    # a hot line whose cascade outgrows its segments; one crowded cell annihilates in every step, so
    # that the other buffer set holds candidate records
    cfg = workloads.small(n_cells=CELLS, ppc=PPC, rics=rics, gamma_max=1e4, pairs=True, conversion="immediate",
                          nmax_over_n0=8.0, sort_interval=1, avg_start_step=0,
                          capacity=[3 * CELLS * PPC, 3 * CELLS * PPC, 0, 0])
    sim = Pic1D(cfg)
    for s in (0, 1):
        p = sim.get_particles(0, s)
        crowd = np.arange(PPC * 5, dtype=np.int32)
        sim.set_particles(0, s, np.r_[p["cell"], np.full(crowd.size, 30, np.int32)],
                          np.r_[p["off"], (crowd % 64 / 64).astype(np.float32)],
                          np.r_[p["u"], np.zeros(crowd.size, np.float32)],
                          np.r_[p["id"], (1 << 50) + crowd.astype(np.uint64) * 2 + s])
    return sim


def _until_error(sim, steps):
    for n in steps:
        try:
            sim.step(n)
        except Pic1dError as e:
            return STATUS[e.code]
    return None


def _particles(sim):
    out = []
    for s in (0, 1):
        p = sim.get_particles(0, s)
        order = np.argsort(p["id"])
        out.append({k: p[k][order] for k in p})
    return out


@pytest.mark.parametrize("rics", ["off", "exact", "table"])
@pytest.mark.parametrize("ahead,graph", [(40, 0), (41, 0), (40, 4), (40, 5), (1100, 0), (1101, 4)])
def test_particles_after_an_error_in_a_long_call(rics, ahead, graph):
    # (no pairs are made without scattering: a momentum that leaves the float range instead)
    want = "ENONFINITE" if rics == "off" else "ECAPACITY"
    print("frozen", rics, ahead, graph, flush=True)
    one, many = _sim(rics), _sim(rics)
    # the step of the error, from a state that is stepped singly and asked for nothing behind it
    k = 0
    if rics == "off":
        k = 4
        for sim in (one, many):
            sim.step(k)
            E = sim.get_field(0)
            E[CELLS // 2:] = 1e300
            sim.set_field(0, E)
    else:
        probe = _sim(rics)
        while _until_error(probe, [1]) is None:
            k += 1
            assert k < ahead
        probe.close()
        assert k > 0                     # a sort has taken place
        one.step(k)
    before = _particles(one)
    assert _until_error(one, [1]) == want
    if graph:
        many.set_graph(graph)
    assert _until_error(many, [ahead]) == want
    a, b = _particles(one), _particles(many)
    m = many.moments(0)
    assert m["step"] == k and one.moments(0)["step"] == k
    assert m["avg_steps"] == k and one.moments(0, average=True)["avg_steps"] == k
    for s in (0, 1):
        print("species", s, "step", k, "live", a[s]["id"].size, b[s]["id"].size, m["count"][s], flush=True)
        for p in (a[s], b[s]):
            assert 0 < p["id"].size <= m["count"][s]
            assert np.unique(p["id"]).size == p["id"].size and np.isin(p["id"], before[s]["id"]).all()
            assert (p["cell"] >= 0).all() and (p["cell"] < CELLS).all()
        if want == "ECAPACITY":          # the push was complete, the appends do not count
            for q in a[s]:
                assert np.array_equal(a[s][q], b[s][q]), q
    one.close()
    many.close()
