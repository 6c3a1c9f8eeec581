"""Photon conversion at record counts on both sides of its chunk sizes, on one line and on several,
against the oracle: the pairs created, their ids, cells and momenta."""
import numpy as np
import pytest

from oracle import pic
from paper_2609_17661_amd import Pic1D, workloads

from . import parity

pytestmark = pytest.mark.gpu


def config(cells, per_line):
    return workloads.small(n_cells=cells, ppc=1, init="empty", pairs=True, j_twist=0.0, kT_keV=2.0,
                           nmax_over_n0=1e7,
                           capacity=[2 * per_line + 4096, 2 * per_line + 4096, 256, 256])


def particles(line, n, cells):
    rng = np.random.default_rng(n + line)
    u = rng.uniform(2e2, 2e3, n).astype(np.float32) * np.where(rng.random(n) < 0.5, 1, -1).astype(np.float32)
    return (rng.integers(0, cells, n).astype(np.int32), rng.random(n).astype(np.float32), u,
            np.arange(1, n + 1, dtype=np.uint64) * np.uint64(3) + np.uint64(line))


# some 0.7 records a particle and one block a CU: one record a thread up to 65,536 records on
# 256 CUs, then two, three and four, and several chunks a block above 262,144
@pytest.mark.parametrize("lines,n", [(1, 7), (1, 900), (3, 900), (1, 120_000), (1, 220_000), (2, 150_000), (1, 500_000)])
def test_conversion_at_record_counts(lines, n):
    print("conversion", lines, n, flush=True)
    cells = 64
    cfg = config(cells, n)
    cfg["lines"] = [dict(cfg["lines"][0], r_eq=4.0 + 0.5 * li) for li in range(lines)]
    sim = Pic1D(cfg)
    for li in range(lines):
        sim.set_particles(li, 0, *particles(li, n, cells))
    before = parity.snapshot(sim)
    sim.step(1)
    after = parity.snapshot(sim)
    made = [sim.moments(li)["counters"]["pairs_created"] for li in range(lines)]
    sim.close()

    ocfg = parity.oracle_config(cfg)
    st = parity.oracle_from_snapshot(ocfg, before)
    marginal = [len(parity._marginal_parents(ocfg, st, li)[0]) for li in range(lines)]
    pic.step(st)
    pairs = [c["pairs_created"] for c in st.counters]
    print(made, pairs, marginal, flush=True)
    assert sum(pairs) > 0.1 * n and sum(marginal) < 0.01 * lines * n + 5
    assert all(abs(g - w) <= x for g, w, x in zip(made, pairs, marginal))
    for li in range(lines):
        for s in (0, 1):
            got, want = after["lines"][li]["parts"][s], st.parts[li][s]
            # a marginal decision is worth one particle on either side
            assert np.unique(got["id"]).size == got["id"].size
            assert np.setxor1d(got["id"], want["id"]).size <= 2 * marginal[li]
            _, a, b = np.intersect1d(got["id"], want["id"], return_indices=True)
            new = ~np.isin(got["id"][a], before["lines"][li]["parts"][s]["id"])
            x = got["cell"][a][new].astype(np.float64) + got["off"][a][new]
            assert np.abs(x - want["x"][b][new]).max() <= 2 * parity.XTOL
            # set from an energy: compared through it
            g, w = (np.hypot(1.0, v) for v in (got["u"][a][new].astype(np.float64), want["u"][b][new]))
            assert (np.abs(g - w) <= parity.GTOL * w * 10).all()
