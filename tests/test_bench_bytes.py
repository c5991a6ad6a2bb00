"""bench.py credits each phase of a step with the bytes of the kernels that run under its name (no GPU needed)."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import bench  # noqa: E402
import workloads as W  # noqa: E402
from oracle.geometry import build_tables  # noqa: E402


@pytest.mark.parametrize("case", [W.small_case_3d(16), W.small_case(64, 32, kind="sin")], ids=["3d", "2d"])
def test_work_lists_from_the_tables(case):
    T = build_tables(case.grid, case.shapes, case.params)
    n, d = case.grid.n, case.grid.ndim
    sets = bench.ghost_sets({"gidx": T.gidx, "ap": T.ap}, n)

    def cell(c):
        return [int(c // np.prod(n[:a], dtype=np.int64)) % n[a] for a in range(d)]

    def index(q):
        return sum(q[a] * int(np.prod(n[:a], dtype=np.int64)) for a in range(d))

    def cross(c):
        out = {int(c)}
        for a in range(d):
            for s in (1, -1):
                q = cell(c)
                q[a] += s
                if a < d - 1:
                    q[a] %= n[a]
                if 0 <= q[a] < n[a]:
                    out.add(index(q))
        return out

    points = set(T.gidx.tolist()) | set(T.ap.reshape(-1).tolist())
    faces = set()
    for c in T.gidx.tolist():
        for a in range(d):
            q = cell(c)
            q[a] = (q[a] - 1) % n[a]
            faces |= {(a, c), (a, index(q))}
    assert sets == {"ghosts": len(T.gidx), "points": len(points), "faces": len(faces),
                    "point_cells": len(set().union(*[cross(c) for c in points])),
                    "patch": len(set().union(*[cross(c) for c in T.gidx.tolist()]))}


@pytest.mark.parametrize("scheme", ["semi", "explicit", "momentum"])
def test_the_point_stencils_are_credited_where_they_run(scheme):
    """phi~ at the listed points runs in the face pass of the step before, so the cells it reads count there."""
    sets = {"ghosts": 100, "points": 700, "point_cells": 1500, "patch": 300, "faces": 500}
    more = dict(sets, point_cells=3000)

    def b(name, s):
        return bench.algorithmic_bytes(name, 1 << 24, 3, 8, s, False, scheme)

    assert b("ghost_dphi", more) == b("ghost_dphi", sets)
    fill = "ns_vel_fill" if scheme == "momentum" else "ghost_fills"
    assert b(fill, more) - b(fill, sets) == 1500 * 8 * (1 if scheme == "explicit" else 2)


def test_the_explicit_update_reads_phi_below_a_million_cells():
    none = {"ghosts": 0, "points": 0, "point_cells": 0, "patch": 0, "faces": 0}
    small, large = 1 << 18, 1 << 20
    per = [bench.algorithmic_bytes("explicit_update", c, 3, 8, none, False, "explicit") / c for c in (small, large)]
    assert per[0] == 8 * 8 and per[1] == 7 * 8 + 0.25
