"""GPU: the tuner times every kernel once.  On 3D lines of 64 to 512 cells the line-tiled rhs is the same kernel with one
cell in flight as with two, so it never reports two; other grids may take either."""
import numpy as np
import pytest

import workloads as W
from oracle.geometry import build_tables

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def chib():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2104_00350_amd import chib as m
    return m


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("n", [(64, 16, 16), (64, 64, 64), (128, 32, 32), (256, 8, 16), (512, 8, 16), (32, 32, 32)])
def test_no_candidate_twice(chib, n, precision):
    grid = W.Grid(n, (0.0,) * 3, tuple(v / 64.0 for v in n))
    prm = W.Params(Cn=0.02, Pe=100.0, dt=1e-4)
    T = build_tables(grid, [], prm)
    geo = chib.Geometry.from_tables(grid.n, grid.lo, grid.hi, T.gidx, T.normal, T.dn, T.gamma, T.ap, T.w)
    st = chib.State(geo, prm, precision)
    st.set_initial(np.zeros(grid.shape))
    picks = [st.tune(2)[0][2] for _ in range(4)]
    print("[gpu] cells in flight", n, precision, picks, flush=True)
    assert n[0] == 32 or 2 not in picks
