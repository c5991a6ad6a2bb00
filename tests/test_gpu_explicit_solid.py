"""GPU: what the solid holds behind its ghost layer reaches no fluid cell in the explicit step.  The fluxes, phi
(whose ghosts take the mirror value) and both fills read fluid and ghost cells only, so a run whose deep solid
cells start as NaN matches the same run with finite values there, bit for bit, on every other cell; and the
finite run matches the FP64 oracle (1e-9, FP32 1e-4, as in the other parity tests)."""
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


# the first three sizes form phi on the way (from 2^20 cells), in chunks of 16, 8 and 4 planes; a flat wall at the
# height given in cells puts its ghost plane inside a chunk, below its first plane or on it, and more ghosts into
# a plane of a tile than it has threads
@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("n,flat", [((64, 8, 2048), None), ((64, 8, 2048), 15.6), ((128, 128, 64), None),
                                    ((256, 256, 16), 2.6), ((256, 256, 16), 3.6), ((256, 256, 16), 4.6),
                                    ((64, 32, 32), 3.6), ((64, 32), 3.6)])
def test_deep_solid_reaches_no_fluid(chib, n, flat, precision):
    h, d = 1.0 / 32, len(n)
    grid = W.Grid(n, (0.0,) * d, tuple(v * h for v in n))
    prm = W.Params(Cn=1.2 * h, Pe=100.0, theta_deg=60.0, dt=2e-6, slip_length=0.02, explicit=True, subgrid=10)
    mid = tuple(0.5 * v for v in grid.hi)
    if flat is None:
        shapes = [W.Shape(W.SPHERE, mid + (3.5 * h,))]
    elif d == 3:
        shapes = [W.Shape(W.HALFPLANE, (0.0, 0.0, flat * h, 0.0, 0.0, 1.0))]
    else:
        shapes = [W.Shape(W.HALFPLANE, (0.0, flat * h, 0.0, 0.0, 1.0, 0.0))]
    T = build_tables(grid, shapes, prm)
    geo = chib.Geometry.from_tables(grid.n, grid.lo, grid.hi, T.gidx, T.normal, T.dn, T.gamma, T.ap, T.w, T.alpha)
    C0, _ = W.droplet_field(grid, mid, 5.0 * h, prm.Cn, 1e-3, 5)
    rng = np.random.default_rng(7)
    faces = [0.2 * rng.standard_normal(grid.shape) for _ in n]
    deep = np.array(T.csolid).copy()
    deep.reshape(-1)[T.gidx] = False
    assert deep.any()
    out = []
    for fill in (None, np.nan):
        C = C0.copy()
        if fill is not None:
            C[deep] = fill
        st = chib.State(geo, prm, precision)
        st.set_initial(C, faces)
        print("[gpu] deep solid", n, flat, precision, fill, flush=True)
        for k in (1, 3):        # the first step has no previous rate
            st.step(k)
        out.append([st.get(chib.FIELD_C)[~deep]] + [st.get(chib.FIELD_U + a) for a in range(d)])
    orc = OracleState(grid, prm, T, C0, faces)
    orc.step(4)
    tol = 1e-9 if precision == 64 else 1e-4
    assert np.max(np.abs(out[0][0] - orc.C[~deep])) <= tol
    for a, f in enumerate(orc.faces):
        assert np.max(np.abs(out[0][1 + a] - f)) <= tol * np.max(np.abs(f))
    for a, b in zip(*out):
        assert np.array_equal(a, b)
