"""GPU: members of a batch take their tile heights from the batch's size and the fixed-size solves where
there is one; every member steps as it does alone, bit for bit."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def chib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_00350_amd import chib as m
    return m


SETS = {
    "every line length": [(64, 32), (128, 64), (256, 128), (512, 256), (1024, 512)],
    "narrower than a tile": [(16, 8), (32, 16), (64, 32)],
    "past two million cells": 4 * [(1024, 512)] + [(128, 64), (512, 256)],
    "line-tiled member": [(2048, 1024), (256, 128)],      # too wide for the y-march
}


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("name", sorted(SETS))
def test_members_step_like_single_states(chib, name, precision):
    def states():
        out = []
        for i, (nx, ny) in enumerate(SETS[name]):
            case = W.small_case(nx, ny, kind="flat", theta_deg=60.0 + 10 * i, seed=i)
            g = case.grid
            geo = chib.Geometry.build(g.n, g.lo, g.hi, case.shapes, case.params)
            st = chib.State(geo, case.params, precision)
            rng = np.random.default_rng(20 + i)
            st.set_initial(case.initial_fields()[0], [0.2 * rng.standard_normal(g.shape) for _ in range(2)])
            if name == "line-tiled member":
                sh = st.shapes()
                sh[0] = [1, 8, 2]
                st.set_shapes(sh)
            out.append(st)
        return out

    singles, members = states(), states()
    b = chib.Batch(members)
    print("batch widths", name, precision, flush=True)
    b.step(5)
    b.sync()
    for s, m in zip(singles, members):
        s.step(5)
        for f in (chib.FIELD_C, chib.FIELD_C_PREV, chib.FIELD_U, chib.FIELD_V):
            a = s.get(f)
            assert np.isfinite(a).all()
            assert np.array_equal(a, m.get(f))
