"""GPU: the solve stage takes fields that are aligned to their elements only, as any slice of a larger device
buffer is: the result is that of an aligned copy, bit for bit."""
import ctypes as C

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


# line lengths with a fixed-size transform, and one without
@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("n", [(32, 64, 64), (64, 64, 64), (128, 64, 64), (256, 64, 64), (512, 64, 64), (256, 128)])
def test_solve_of_an_unaligned_field(chib, n, precision):
    d = len(n)
    grid = W.Grid(n, (0.0,) * d, tuple(v / 64.0 for v in n))
    prm = W.Params(Cn=0.02, Pe=100.0, dt=1e-4)
    T = build_tables(grid, [], prm)
    geo = chib.Geometry.from_tables(grid.n, grid.lo, grid.hi, T.gidx, T.normal, T.dn, T.gamma, T.ap, T.w)
    st = chib.State(geo, prm, precision)
    st.set_initial(np.zeros(grid.shape))
    r = 16 if n[0] == 128 or precision == 32 else 8
    sh = st.shapes()
    sh[3] = [3 if n[0] == 256 else 2 if n[0] == 512 else 4, r, 1]      # the fixed-size tile of the x pass
    st.set_shapes(sh)
    Q = np.random.default_rng(11).standard_normal(grid.shape) * 1e9
    ref = st.stage(chib.STAGE_SOLVE, Q)
    src = torch.zeros(st.cells + 4, dtype=st.torch_dtype, device=st.device)
    dst = torch.zeros(st.cells + 4, dtype=st.torch_dtype, device=st.device)
    src[1:1 + st.cells] = torch.as_tensor(Q.reshape(-1)).to(device=st.device, dtype=st.torch_dtype)
    torch.cuda.synchronize()
    print("[gpu] unaligned solve", n, precision, src[1:].data_ptr() & 15, flush=True)
    chib.check(chib.lib.ch_ib_stage(st.h, chib.STAGE_SOLVE, C.c_void_p(src[1:].data_ptr()),
                                    C.c_void_p(dst[1:].data_ptr())))
    assert np.array_equal(dst[1:1 + st.cells].cpu().numpy().reshape(grid.shape), ref)
    assert not dst[0].item() and not dst[1 + st.cells:].any().item()
