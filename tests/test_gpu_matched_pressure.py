"""GPU: fluids of one density take their pressure from the divergence formed inside the transform, in both dimensions
and precisions, and a step matches the FP64 oracle (FP64 within 1e-9 of each field's scale; FP32 within 1e-4 for C
and 1e-3 of the largest velocity, as in the other parity tests of the coupled step)."""
import dataclasses

import numpy as np
import pytest

import workloads as W
from oracle.geometry import build_tables, face_fractions
from oracle.solver import OracleState

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def chib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_00350_amd import chib as m
    return m


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("n", [(64, 32), (128, 64), (512, 256), (32, 16, 32), (64, 16, 32)])
def test_matched_fluids(chib, n, precision):
    h, d = 1.0 / 32, len(n)
    grid = W.Grid(n, (0.0,) * d, tuple(v * h for v in n))
    prm = W.Params(Cn=1.3 * h, Pe=50.0, Re=10.0, Ca=0.2, theta_deg=60.0, slip_length=0.02, dt=1e-4, navier_stokes=True,
                   subgrid=10)
    p = (0.0, 0.0, 2.6 * h, 0.0, 0.0, 1.0) if d == 3 else (0.0, 2.6 * h, 0.0, 0.0, 1.0, 0.0)
    shapes = [W.Shape(W.HALFPLANE, p)]
    T, fa = build_tables(grid, shapes, prm), face_fractions(grid, shapes, prm)
    geo = chib.Geometry.from_tables(grid.n, grid.lo, grid.hi, T.gidx, T.normal, T.dn, T.gamma, T.ap, T.w, T.alpha)
    geo.set_face_fractions(fa)
    C0, _ = W.droplet_field(grid, tuple(0.5 * v for v in grid.hi), 4.0 * h, prm.Cn, 1e-3, 5)
    faces = [0.05 * np.random.default_rng(13 + a).standard_normal(grid.shape) for a in range(d)]

    def names(params):
        st = chib.State(geo, params, precision)
        st.set_initial(C0, faces)
        print("[gpu] matched", n, precision, params.rho1, flush=True)
        return st, st.step_timed(4)

    st, kernels = names(prm)
    assert "ns_div_poisson" in kernels and "ns_pressure_rhs" not in kernels
    orc = OracleState(grid, prm, T, C0, faces, face_alpha=fa)
    orc.step(4)
    u = max(float(np.max(np.abs(f))) for f in orc.faces)
    assert np.max(np.abs(st.get(chib.FIELD_C) - orc.C)) <= (1e-9 if precision == 64 else 1e-4)
    for a in range(d):
        assert np.max(np.abs(st.get(chib.FIELD_U + a) - orc.faces[a])) <= (1e-9 if precision == 64 else 1e-3) * u
    _, kernels = names(dataclasses.replace(prm, rho1=0.5))
    assert "ns_pressure_rhs" in kernels and "ns_div_poisson" not in kernels
