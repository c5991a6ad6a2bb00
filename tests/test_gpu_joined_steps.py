"""GPU: steps taken in one call join the face pass with the next step's ghost patch; the result is that
of the same steps taken one call at a time, bit for bit."""
import dataclasses

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


def _flow(case):
    return dataclasses.replace(case, params=dataclasses.replace(case.params, navier_stokes=True, dt=2e-5))


CASES = {
    "2d": lambda: W.small_case(128, 64, kind="sin"),
    "2d_dynamic": lambda: W.small_case(64, 32, kind="circle", Vs=0.5),
    "2d_no_velocity_fill": lambda: W.small_case(64, 32, kind="tilted", velocity_fill=False),
    "2d_wall_longer_than_a_block": lambda: W.small_case(1024, 512, kind="flat"),
    "2d_flow": lambda: _flow(W.small_case(64, 32, kind="sin")),
    "3d": lambda: W.small_case_3d(32),
    "3d_z_march": lambda: dataclasses.replace(
        W.small_case_3d(32), grid=W.Grid((256, 32, 32), (-16.0, -2.0, -2.0), (16.0, 2.0, 2.0))),
    "3d_flow": lambda: _flow(W.small_case_3d(32)),
}


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("name", sorted(CASES))
def test_joined_steps(chib, name, precision):
    case = CASES[name]()
    g = case.grid
    geo = chib.Geometry.build(g.n, g.lo, g.hi, case.shapes, case.params)
    C0, _ = case.initial_fields()
    rng = np.random.default_rng(3)
    faces = [0.2 * rng.standard_normal(g.shape) for _ in range(g.ndim)]
    out = []
    for calls in ((1,) * 7, (7,), (2, 4, 1)):
        st = chib.State(geo, case.params, precision)
        st.set_initial(C0, faces)
        if name == "3d_z_march":
            st.set_shapes([[1, 8, 3], [3, 8, 1], [3, 8, 1], [3, 8, 1]])
        for n in calls:
            st.step(n)
        out.append([st.get(f) for f in (chib.FIELD_C, chib.FIELD_C_PREV, chib.FIELD_CI)]
                   + [st.get(chib.FIELD_U + a) for a in range(g.ndim)])
        assert all(np.isfinite(f).all() for f in out[-1])
    for other in out[1:]:
        for a, b in zip(out[0], other):
            assert np.array_equal(a, b)
