"""The 32-bit slot arithmetic of the kernels at segments of up to 2^31 - 256 slots, and the tags by which
the annihilation compares particles with counts, in a host build."""
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_17661_amd", "csrc")
MAIN = r"""
#include <cstdio>
#include "slots.h"
int main() {
    char op;
    long long a, b, c;
    while (std::scanf(" %c %lld %lld %lld", &op, &a, &b, &c) == 4) {
        const int x = (int)(unsigned)a, y = (int)b, z = (int)c;
        if (op == 'g') std::printf("%u\n", pic1d::cell_tag((unsigned)a, (unsigned)b));
        else std::printf("%d\n", op == 't' ? pic1d::tiles_of(x, y) : op == 's' ? (int)pic1d::slot_in(x, y) : (int)pic1d::slots_in(x, y, z));
    }
}
"""
CAP = 2**31 - 256                      # the largest accepted capacity


@pytest.fixture(scope="module")
def slots(tmp_path_factory):
    d = tmp_path_factory.mktemp("slots")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", CSRC, "-o", str(d / "main"), str(d / "main.cpp")], check=True)

    def run(rows):
        inp = "\n".join(" ".join(map(str, r)) for r in rows)
        out = subprocess.run([str(d / "main")], input=inp, capture_output=True, text=True, check=True).stdout.split()
        return [int(v) for v in out]
    return run


def test_tiles_of_large_segments(slots):
    counts = [0, 1, 255, 256, 257, 4095, 4096, 4097, 2**31 - 4097, 2**31 - 4096, 2**31 - 4095, 2**31 - 1024, CAP - 1, CAP]
    rows = [("t", n, t, 0) for n in counts for t in (256, 512, 1024, 2048, 4096)]
    assert slots(rows) == [-(-n // t) for _, n, t, _ in rows]


def test_slots_of_a_counter_that_passed_the_sign(slots):
    # an allocation counter counts on past the capacity, by at most 2^30 a step
    at = [0, 1, 255, 256, CAP - 1, CAP, 2**31 - 1, 2**31, 2**31 + 5, 2**31 + 2**30]
    rows = [("s", a, cap, 0) for a in at for cap in (256, CAP)]
    assert slots(rows) == [int(a < cap) for _, a, cap, _ in rows]
    rows = [("r", a, n, cap) for a in at for n in (0, 1, 256, 1024) for cap in (256, CAP)]
    assert slots(rows) == [int(a + n <= cap) for _, a, n, cap in rows]


def test_tags_find_particles_in_other_cells(slots):
    # a count that does not match shows, whatever other cells do to make up for it
    cells = 3000
    tag = np.array([slots([("g", c0 + c, s, 0) for c in range(cells)]) for c0, s in ((0, 0), (0, 1), (2**27 - cells, 1))],
                   dtype=np.uint64)
    for t in tag:
        assert np.unique(t).size == cells and not (t == 0).any()
        rng = np.random.default_rng(5)
        count = rng.integers(0, 1000, cells).astype(np.uint64)
        particles = np.repeat(np.arange(cells), count.astype(int))
        assert int(t[particles].sum()) % 2**32 == int((count * t).sum()) % 2**32
        # one particle in another cell (every distance), two swapped against one between them, and
        # longer patterns that a linear tag would miss
        for d in range(1, cells):
            assert ((t[d:] - t[:-d]) % 2**32 != 0).all()
        for w in ((1, -2, 1), (1, -1, -1, 1), (1, -3, 3, -1), (2, -4, 2)):
            total = sum(np.int64(k) * t[i:cells - len(w) + i + 1].astype(np.int64) for i, k in enumerate(w))
            assert (total % 2**32 != 0).all(), w
    assert ((tag[0] - tag[1]) % 2**32 != 0).all()
