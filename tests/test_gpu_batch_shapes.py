"""GPU: a batch runs its members with launch shapes of its own; what the members step with alone stays as it was,
while the batch lives and after it, and no batch changes a result."""
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


def _states(chib, sizes, precision):
    out = []
    for i, (nx, ny) in enumerate(sizes):
        case = W.small_case(nx, ny, kind="flat", theta_deg=60.0 + 10 * i, seed=i)
        g = case.grid
        st = chib.State(chib.Geometry.build(g.n, g.lo, g.hi, case.shapes, case.params), case.params, precision)
        rng = np.random.default_rng(20 + i)
        st.set_initial(case.initial_fields()[0], [0.2 * rng.standard_normal(g.shape) for _ in range(2)])
        out.append(st)
    return out


@pytest.mark.parametrize("precision", [64, 32])
def test_members_keep_their_shapes(chib, precision):
    states = _states(chib, [(64, 32), (128, 64), (512, 256)], precision)
    chosen = states[1].shapes()
    chosen[3][0] = 2
    states[1].set_shapes(chosen)
    before = [s.shapes() for s in states]
    b = chib.Batch(states)
    print("[gpu] batch shapes", precision, before, flush=True)
    assert [s.shapes() for s in states] == before
    b.step(3)
    b.sync()
    b.close()
    assert [s.shapes() for s in states] == before


# a batch takes one rhs kernel for all its members: the marching one only where every member is narrow enough
@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("sizes", [[(2048, 1024), (64, 32), (128, 64), (256, 128), (512, 256), (1024, 512)],
                                   [(256, 128), (2048, 1024)]])
def test_mixed_widths_at_default_shapes(chib, sizes, precision):
    singles, members = _states(chib, sizes, precision), _states(chib, sizes, precision)
    b = chib.Batch(members)
    print("[gpu] mixed widths", precision, sizes, flush=True)
    b.step(5)
    b.sync()
    for s, m in zip(singles, members):
        s.step(5)
        for f in (chib.FIELD_C, chib.FIELD_C_PREV, chib.FIELD_U, chib.FIELD_V):
            a = s.get(f)
            assert np.isfinite(a).all()
            assert np.array_equal(a, m.get(f))


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("n", [(64, 32), (256, 128), (512, 256), (1024, 512)])
def test_rhs_kernels_of_2d_grids_agree(chib, n, precision):
    """Line-tiled with one and two cells in flight, and marching: one step, bit for bit."""
    out = []
    for u in (1, 2, 3):
        st = _states(chib, [n], precision)[0]
        sh = st.shapes()
        sh[0] = [1, 8, u]
        st.set_shapes(sh)
        print("[gpu] rhs kernels", n, precision, u, flush=True)
        st.step(1)
        out.append(st.get(chib.FIELD_C))
    for o in out[1:]:
        assert np.array_equal(out[0], o)
