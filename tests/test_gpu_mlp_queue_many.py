"""The surrogate pusher's queue with more items than wavefronts, over lines and species in turn, alone and
beside lines on their tables: every particle is pushed once in every step and comes out as it does from
states of so few items that no wavefront takes a second one."""
import math

import numpy as np
import pytest

from paper_2609_17661_amd import Pic1D

from .test_gpu_mlp import _fallback_cfg

pytestmark = pytest.mark.gpu

RADII = (4.0, 40.0, 4.0, 40.0, 4.0)
CELLS = 700
PIECES = 10
STEPS = 2


def _cfg(tol):
    cfg = _fallback_cfg(tol, RADII, n_cells=CELLS, ppc=1)
    cfg.update(pairs=False, frozen_field=True, gravity=False, sort_interval=0)
    for ln in cfg["lines"]:
        ln.update(init="empty", capacity=[140_000, 140_000, 256, 60_000])
    return cfg


def _particles():
    rng = np.random.default_rng(83)
    out = {}
    for line in range(len(RADII)):
        for s, n in ((0, 130_001 - 777 * line), (1, 120_000 + 511 * line), (3, 40_003 + line)):
            gam = 10.0 ** rng.uniform(0, 3.5, n)
            u = np.where(rng.random(n) < 0.5, -1, 1) * np.sqrt(gam**2 - 1) * (1.0 if s < 3 else 1e-2)
            cell = rng.integers(0, CELLS, n).astype(np.int32)
            if line < 3:             # in order, as after a sort; the others deposit from all over the line
                cell.sort()
            out[line, s] = (cell, rng.random(n).astype(np.float32) * np.float32(0.999), u.astype(np.float32),
                            np.arange(n, dtype=np.uint64) * np.uint64(20) + np.uint64(4 * line + s))
    return out


def _run(tol, parts):
    sim = Pic1D(_cfg(tol))
    for (line, s), p in parts.items():
        sim.set_particles(line, s, *p)
    E = np.random.default_rng(84).normal(0.0, 1e-2, CELLS)
    pushed = np.zeros((len(RADII), 2), np.int64)
    for line in range(len(RADII)):
        sim.set_field(line, E)
    for _ in range(STEPS):
        for line in range(len(RADII)):
            count = sim.moments(line)["count"]
            pushed[line] += (sum(count), count[3])
        sim.step(1)
    mom = []
    for line in range(len(RADII)):
        m = sim.moments(line)
        assert (m["counters"]["pushed"], m["counters"]["pushed_ions"]) == tuple(pushed[line])
        mom.append((m["n"], m["j"], m["counters"]["limited"], m["counters"]["events"], m["counters"]["absorbed"]))
    got = {}
    for k in parts:
        p = sim.get_particles(*k)
        order = np.argsort(p["id"])
        got[k] = {q: p[q][order] for q in p}
    uses = [sim.rics_line_info(line)[1] for line in range(len(RADII))]
    sim.close()
    return got, mom, uses


@pytest.mark.parametrize("mixed", [False, True])
def test_many_items_a_wavefront(mixed):
    tol = 1e30
    if mixed:
        sim = Pic1D(_cfg(tol))
        e = [sim.rics_line_info(line)[0] for line in (0, 1)]
        sim.close()
        tol = math.sqrt(e[0] * e[1])
    parts = _particles()
    items = sum((p[0].size + 255) // 256 for p in parts.values())
    print("queue, mixed", mixed, "items", items, flush=True)
    assert items > 2 * 2048                           # two wavefronts per SIMD of 256 CUs
    whole, mom, uses = _run(tol, parts)
    assert len(set(uses)) == (2 if mixed else 1)
    pieces = []
    for k in range(PIECES):
        pieces.append(_run(tol, {key: tuple(a[k::PIECES] for a in p) for key, p in parts.items()}))
        assert pieces[-1][2] == uses
    for key in parts:
        for q in ("id", "cell", "off", "u"):
            a = np.concatenate([pc[0][key][q] for pc in pieces])
            order = np.argsort(np.concatenate([pc[0][key]["id"] for pc in pieces]))
            assert np.array_equal(whole[key][q], a[order]), (key, q)
    for line in range(len(RADII)):
        n, j, *counts = mom[line]
        parts_of = [pc[1][line] for pc in pieces]
        assert np.array_equal(n, sum(p[0] for p in parts_of))
        # sums in fixed point, exact; a rounding to float64 each
        jsum = sum(p[1] for p in parts_of)
        assert np.abs(j - jsum).max() <= 2 * PIECES * 2.0**-53 * sum(np.abs(p[1]) for p in parts_of).max()
        assert counts == [sum(p[2 + i] for p in parts_of) for i in range(3)]
    print("events", [m[3] for m in mom], "limited", [m[2] for m in mom], flush=True)
