"""Annihilation where many particles carry one id, so that all keys of a cell are equal and lie on one side
of its threshold: the cells searched in full are bounded, and the limit holds a step later."""
import time

import numpy as np
import pytest

from paper_2609_17661_amd import Pic1D, workloads

pytestmark = pytest.mark.gpu


def test_one_id_for_all_particles():
    cells, per_cell = 8192, 400
    n = cells * per_cell
    n_max = 2 * per_cell - 2                 # one pair a cell: 29 of 400 keys are recorded on average
    cfg = workloads.small(n_cells=cells, ppc=1, init="empty", rics="off", j_twist=0.0, pairs=False, nmax_over_n0=n_max,
                          capacity=[n, n, 256, 256])
    sim = Pic1D(cfg)
    cell = np.repeat(np.arange(cells, dtype=np.int32), per_cell)
    for s in (0, 1):
        sim.set_particles(0, s, cell, np.full(n, 0.5, np.float32), np.zeros(n, np.float32),
                          np.full(n, 12345 + s, np.uint64))
    for k in range(3):
        a = time.perf_counter()
        sim.step(1)
        m = sim.moments(0)
        over = int((m["n"].sum(axis=0) > n_max).sum())
        print("step", k, "seconds", time.perf_counter() - a, "cells over the limit", over, m["count"], flush=True)
        # 1,024 cells are searched, the others wait for the step in which all candidates are recorded
        assert over == (cells - 1024 if k == 0 else 0)
    live = [np.bincount(sim.get_particles(0, s)["cell"], minlength=cells) for s in (0, 1)]
    assert np.array_equal(*live)
    sim.close()
