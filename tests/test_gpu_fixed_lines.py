"""GPU: transform kernels compiled for 64-, 128- and 512-point lines give the bits of the runtime-size
kernels, whose per-line arithmetic is the same, and match the oracle."""
import numpy as np
import pytest

import workloads as W
from oracle.geometry import build_tables, face_fractions
from oracle.solver import OracleState, derived_coefficients, spectral_solve

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def chib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_00350_amd import chib as m
    return m


def _state(chib, n, precision):
    d = len(n)
    grid = W.Grid(n, (0.0,) * d, tuple(v / 64.0 for v in n))
    prm = W.Params(Cn=0.02, Pe=100.0, dt=1e-4)
    T = build_tables(grid, [], prm)
    geo = chib.Geometry.from_tables(grid.n, grid.lo, grid.hi, T.gidx, T.normal, T.dn, T.gamma, T.ap, T.w)
    st = chib.State(geo, prm, precision)
    st.set_initial(np.zeros(grid.shape))
    return grid, prm, st


# every axis at each length, and the narrowest grid that a tile of adjacent columns fits
@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("n", [(64, 64, 64), (128, 128, 128), (32, 64, 128), (32, 512, 64), (512, 64, 512),
                               (64, 128), (128, 512), (512, 64)])
def test_fixed_lines(chib, n, precision):
    grid, prm, st = _state(chib, n, precision)
    Q = np.random.default_rng(11).standard_normal(grid.shape) * 1e9
    cols = 4 if precision == 64 else 5
    default = 8 if precision == 64 else 16

    def shapes(drop):
        r = [16 if m == 128 else default for m in n]
        lb = [cols - (m == 512) - drop for m in n]
        return [[2, 8, 1], [lb[1], r[1], 1], [lb[-1], r[-1], 1], [(2 if n[0] == 512 else 4) - drop, r[0], 1]]

    print("fixed-size lines", n, precision, shapes(0), flush=True)
    st.set_shapes(shapes(0))
    fixed = np.asarray(st.stage(chib.STAGE_SOLVE, Q))
    st.set_shapes(shapes(1))
    runtime = np.asarray(st.stage(chib.STAGE_SOLVE, Q))
    assert np.array_equal(fixed, runtime)
    _, al, a = derived_coefficients(prm)
    ref = spectral_solve(Q, grid, al, a)
    assert np.max(np.abs(fixed - ref)) <= (1e-12 if precision == 64 else 1e-4) * np.max(np.abs(ref))


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("n", [(16, 8), (64, 32), (1024, 512), (8, 8, 8), (32, 32, 64), (64, 64, 64),
                               (128, 128, 64), (256, 128, 128), (512, 256, 32)])
def test_default_shapes_fit(chib, n, precision):
    """The shapes a new state takes from its grid's size: the solve at them against the oracle."""
    grid, prm, st = _state(chib, n, precision)
    Q = np.random.default_rng(12).standard_normal(grid.shape) * 1e9
    print("default shapes", n, precision, flush=True)
    out = np.asarray(st.stage(chib.STAGE_SOLVE, Q))
    _, al, a = derived_coefficients(prm)
    ref = spectral_solve(Q, grid, al, a)
    assert np.max(np.abs(out - ref)) <= (1e-12 if precision == 64 else 1e-4) * np.max(np.abs(ref))


# the divergence of the velocity formed on the way into the x transform (fluids of one density)
@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("n", [(64, 64, 64), (128, 64, 64), (512, 64, 64)])
def test_fixed_lines_of_the_divergence(chib, n, precision):
    h = 1.0 / 32
    g = W.Grid(n, (0.0, 0.0, 0.0), tuple(v * h for v in n))
    prm = W.Params(Cn=1.3 * h, Pe=50.0, Re=10.0, Ca=0.2, theta_deg=60.0, slip_length=0.02, dt=1e-4,
                   navier_stokes=True, subgrid=10)
    wall = [W.Shape(W.HALFPLANE, (0.0, 0.0, 2.6 * h, 0.0, 0.0, 1.0))]
    T = build_tables(g, wall, prm)
    geo = chib.Geometry.from_tables(g.n, g.lo, g.hi, T.gidx, T.normal, T.dn, T.gamma, T.ap, T.w, T.alpha)
    geo.set_face_fractions(face_fractions(g, wall, prm))
    rng = np.random.default_rng(4)
    C0 = np.tanh(rng.standard_normal(g.shape))
    faces = [0.1 * rng.standard_normal(g.shape) for _ in range(3)]
    out = []
    for drop in (0, 1):
        st = chib.State(geo, prm, precision)
        sh = st.shapes()
        sh[3] = [(2 if n[0] == 512 else 4) - drop, 16 if n[0] == 128 or precision == 32 else 8, 1]
        st.set_initial(C0, faces)
        st.set_shapes(sh)
        print("divergence", n, precision, sh, flush=True)
        st.step(2)
        out.append([st.get(f) for f in (chib.FIELD_C, chib.FIELD_U, chib.FIELD_V, chib.FIELD_P)])
    for a, b in zip(*out):
        assert np.isfinite(a).all()
        assert np.array_equal(a, b)


# the line-tiled rhs of 64- to 512-point lines: tiles that fill the block once, twice, or in part.  Three steps
# at a wall, within 1e-9 of the oracle in FP64 and 1e-4 in FP32 as in the other parity tests
@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("n", [(64, 16, 32), (128, 8, 32), (256, 8, 16), (512, 8, 16)])
def test_rhs_of_fixed_lines(chib, n, precision):
    h = 1.0 / 32
    g = W.Grid(n, (0.0, 0.0, 0.0), tuple(v * h for v in n))
    prm = W.Params(Cn=1.3 * h, Pe=50.0, theta_deg=60.0, slip_length=0.02, dt=1e-4)
    T = build_tables(g, [W.Shape(W.HALFPLANE, (0.0, 0.0, 2.6 * h, 0.0, 0.0, 1.0))], prm)
    geo = chib.Geometry.from_tables(g.n, g.lo, g.hi, T.gidx, T.normal, T.dn, T.gamma, T.ap, T.w, T.alpha)
    C0, _ = W.droplet_field(g, tuple(0.5 * v for v in g.hi), 4.0 * h, prm.Cn, 1e-3, 5)
    rng = np.random.default_rng(6)
    faces = [0.05 * rng.standard_normal(g.shape) for _ in range(3)]
    out = []
    for lt in (1, 2, 3, 4, 5):
        st = chib.State(geo, prm, precision)
        sh = st.shapes()
        sh[0] = [lt, 8, 1]
        st.set_shapes(sh)
        st.set_initial(C0, faces)
        print("rhs lines", n, precision, lt, flush=True)
        st.step(3)
        out.append(np.asarray(st.get(chib.FIELD_C)))
    orc = OracleState(g, prm, T, C0, faces)
    orc.step(3)
    assert np.max(np.abs(out[0] - orc.C)) <= (1e-9 if precision == 64 else 1e-4)
    for o in out[1:]:
        assert np.array_equal(o, out[0])
