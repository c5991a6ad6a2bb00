"""GPU: the velocity fill is one computation, whether it runs alone (when fields are set) or joined with the fill of C
(at the end of a step, alone or in a batch): filled faces that a step fills again match the same faces set and
filled anew, bit for bit.  With the static condition it reads the faces only."""
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


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("d", [2, 3])
def test_velocity_fill_alone_and_joined(chib, d, precision):
    case = W.small_case(128, 64, kind="circle", slip_length=0.05) if d == 2 else W.small_case_3d(32)
    g = case.grid
    geo = chib.Geometry.build(g.n, g.lo, g.hi, case.shapes, case.params)
    rng = np.random.default_rng(9)
    faces = [rng.standard_normal(g.shape) for _ in range(d)]
    C0 = case.initial_fields()[0]

    def state(f):
        st = chib.State(geo, case.params, precision)
        st.set_initial(C0, f)
        return st

    def filled(st):
        st.step(0)
        return [st.get(chib.FIELD_U + a) for a in range(d)]

    first = state(faces)
    once = filled(first)                     # the fill alone
    assert any(np.any(a != b.astype(a.dtype)) for a, b in zip(once, faces))
    print("[gpu] velocity fill", d, precision, len(once), flush=True)
    alone = filled(state(once))              # and again, alone
    first.step(1)                            # and again, joined
    for a, b in zip(alone, [first.get(chib.FIELD_U + a) for a in range(d)]):
        assert np.array_equal(a, b)
    if d == 2:                               # and again, in a batch
        member = state(faces)
        b = chib.Batch([member, state(faces)])
        b.step(1)
        b.sync()
        for a, f in zip(alone, [member.get(chib.FIELD_U + a) for a in range(d)]):
            assert np.array_equal(a, f)
