"""Pair annihilation's candidate threshold and its selection at their edges, against the oracle:
particles at rest on a line without field or current, so that a step does nothing but annihilate."""
import numpy as np
import pytest

from oracle import philox, pic
from paper_2609_17661_amd import Pic1D, workloads

from . import parity

pytestmark = pytest.mark.gpu


def _print(*a):
    print(*a, flush=True)


def _sim(n_max):
    # n0 = 1 per cell: n_max is the same whole number in float32 and float64
    cfg = workloads.small(n_cells=6, ppc=1, init="empty", rics="off", j_twist=0.0, pairs=False, nmax_over_n0=n_max,
                          capacity=[4096, 4096, 256, 256])
    return cfg, Pic1D(cfg)


def _check(cfg, sim, k):
    before = parity.snapshot(sim)
    sim.step(1)
    rep, _ = parity.compare_step(parity.oracle_config(cfg), before, parity.snapshot(sim))
    c = sim.moments(0)["counters"]
    _print(rep, c["annihilated"])
    assert rep["excused"] == 0 and c["annihilated"] == k


def _place(sim, s, cells, ids):
    rng = np.random.default_rng(s + 5)
    sim.set_particles(0, s, cells, rng.random(len(ids)).astype(np.float32), np.zeros(len(ids), np.float32), ids)


@pytest.mark.parametrize("m,k", [(1, 1), (28, 1), (29, 1), (64, 1), (65, 3), (200, 30), (300, 120), (520, 60), (700, 520)])
def test_selection_at_record_counts(m, k):
    # N = 2 m particles in a cell and n_max = N - 2 k: k pairs go.  The threshold admits about
    # k + 8 k^1/2 + 20 records of a species (all m of them up to that): one register a lane up to
    # 64, eight up to 512, memory beyond
    _print("records", m, k)
    cfg, sim = _sim(2 * m - 2 * k if m > k else 0.5)
    for s in (0, 1):
        _place(sim, s, np.full(m, 3), np.arange(m, dtype=np.uint64) * 7 + s + 11)
    _check(cfg, sim, k)


def _keys(cfg, ids):
    return pic.annihilation_keys(0, ids, *philox.seed_key(cfg["seed"]))


@pytest.mark.parametrize("low", [0, 1])
def test_cell_whose_keys_all_exceed_the_threshold(low):
    # k = 2 of m = 200: the threshold lies at 33.3/200 of the key range; with `low` keys of the
    # electrons below it, fewer than k are recorded and the whole cell has to be
    _print("above the threshold", low)
    cfg, sim = _sim(397)
    ids = np.arange(1, 3000, dtype=np.uint64)
    frac = _keys(cfg, ids).astype(np.float64) / 2.0**64
    high = ids[frac > 0.2][:200 - low]
    few = ids[frac < 0.1][:low]
    _place(sim, 0, np.full(200, 2), np.concatenate([high, few]))
    _place(sim, 1, np.full(200, 2), np.arange(5000, 5200, dtype=np.uint64))
    _check(cfg, sim, 2)


def test_equal_high_key_words():
    # two ids whose keys share their high word, the smallest of a cell that loses one pair: the
    # low word decides
    cfg, sim = _sim(98)
    ids = np.arange(1, 600001, dtype=np.uint64)
    keys = _keys(cfg, ids)
    hi = keys >> np.uint64(32)
    order = np.argsort(hi, kind="stable")
    at = np.nonzero((np.diff(hi[order].astype(np.int64)) == 0) & (hi[order][1:] < 2**31))[0]
    assert at.size > 0
    pair = order[at[0]:at[0] + 2]
    rest = ids[np.nonzero(hi > hi[pair[0]])[0][:48]]
    _print("equal high words", hex(int(keys[pair[0]])), hex(int(keys[pair[1]])))
    _place(sim, 0, np.full(50, 4), np.concatenate([rest[:20], ids[pair], rest[20:]]))
    _place(sim, 1, np.full(50, 4), np.arange(700000, 700050, dtype=np.uint64))
    _check(cfg, sim, 1)


@pytest.mark.parametrize("per_cell", [37, 1390, 1401])
def test_gather_at_either_pass_length(per_cell):
    # the gather takes four particles a thread, or eight from 8,388,608 particles on (256 CUs); ragged
    # segments, every cell over the limit: the k pairs of the smallest keys go
    _print("gather", per_cell)
    cells, k = 3000, 3
    n = cells * per_cell
    cfg = workloads.small(n_cells=cells, ppc=1, init="empty", rics="off", j_twist=0.0, pairs=False,
                          nmax_over_n0=2 * per_cell - 2 * k, capacity=[n + 64, n + 64, 256, 256])
    sim = Pic1D(cfg)
    ids = [np.arange(n, dtype=np.uint64) * np.uint64(5) + np.uint64(s + 1) for s in (0, 1)]
    cell = np.repeat(np.arange(cells, dtype=np.int32), per_cell)
    for s in (0, 1):
        _place(sim, s, cell, ids[s])
    sim.step(1)
    for s in (0, 1):
        keys = _keys(cfg, ids[s]).reshape(cells, per_cell)
        gone = np.argsort(keys, axis=1)[:, :k] + per_cell * np.arange(cells)[:, None]
        want = np.delete(ids[s], gone.ravel())
        got = sim.get_particles(0, s)["id"]
        np.testing.assert_array_equal(np.sort(got), want)
    assert sim.moments(0)["counters"]["annihilated"] == k * cells
    sim.close()
