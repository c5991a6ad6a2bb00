"""GPU: the 3D explicit step that forms phi on the way (grids from 2^20 cells) and the sixteen-lane dynamic
ghost fill, against the FP64 oracle on the same tables.

Tolerances as in the other parity tests: FP64 1e-9 of each field's scale, FP32 1e-4 for these few steps."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from oracle.geometry import build_tables
from oracle.solver import OracleState

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def chib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_00350_amd import chib as m
    return m


def _pair(chib, grid, prm, shapes, centre, radius, precision):
    T = build_tables(grid, shapes, prm)
    geo = chib.Geometry.from_tables(grid.n, grid.lo, grid.hi, T.gidx, T.normal, T.dn, T.gamma, T.ap, T.w, T.alpha)
    st = chib.State(geo, prm, precision)
    C0, _ = W.droplet_field(grid, centre, radius, prm.Cn, 1e-3, 5)
    rng = np.random.default_rng(7)
    faces = [0.2 * rng.standard_normal(grid.shape) for _ in grid.n]
    st.set_initial(C0, faces)
    return st, OracleState(grid, prm, T, C0, faces)


def _errors(chib, st, orc):
    e = [float(np.max(np.abs(st.get(chib.FIELD_C) - orc.C)))]
    for a, f in enumerate(orc.faces):
        e.append(float(np.max(np.abs(st.get(chib.FIELD_U + a) - f)) / np.max(np.abs(f))))
    return e


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("wall", [True, False])
@pytest.mark.parametrize("n", [(64, 8, 2048), (128, 128, 64), (256, 256, 16)])
def test_fused_explicit_step(chib, n, wall, precision):
    h = 1.0 / 32
    grid = W.Grid(n, (0.0, 0.0, 0.0), tuple(v * h for v in n))
    prm = W.Params(Cn=1.2 * h, Pe=100.0, theta_deg=60.0, dt=2e-6, slip_length=0.02, explicit=True, subgrid=10)
    mid = tuple(0.5 * v for v in grid.hi)
    shapes = [W.Shape(W.SPHERE, mid + (2.5 * h,))] if wall else []
    st, orc = _pair(chib, grid, prm, shapes, mid, 5.0 * h, precision)
    for k in (1, 3):        # the first step has no previous rate
        st.step(k)
        orc.step(k)
        e = _errors(chib, st, orc)
        print("[gpu]", n, wall, precision, len(orc.T.gidx), e, flush=True)
        assert max(e) <= (1e-9 if precision == 64 else 1e-4)


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("d", [2, 3])
def test_dynamic_fill(chib, d, precision):
    case = W.small_case(128, 64, kind="circle", theta_deg=70.0) if d == 2 else W.small_case_3d(32, theta_deg=70.0)
    prm = dataclasses.replace(case.params, Vs=0.5, subgrid=20)
    st, orc = _pair(chib, case.grid, prm, case.shapes, case.droplet_centre, case.droplet_radius, precision)
    st.step(5)
    orc.step(5)
    e = _errors(chib, st, orc) + [float(np.max(np.abs(st.get(chib.FIELD_CI) - orc.CI)))]
    print("[gpu]", d, precision, e, flush=True)
    assert max(e) <= (1e-9 if precision == 64 else 1e-4)
