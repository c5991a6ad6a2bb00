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
