"""The checking and folding passes over operands that are far from square: one
row, rows of one to nine chunks of 8, few rows of many, and row strides that
are not 16-byte aligned."""
import numpy as np
import pytest
import torch

import oracle as O
import synth

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (3, 7), (5000, 1), (70000, 8), (9000, 9), (2100, 72), (33, 20000), (1, 30011), (257, 2049), (300, 3)]


@pytest.fixture(scope="module")
def mpr():
    import paper_2409_17658_amd as m

    m.lib()
    m.init(0)
    return m


@pytest.mark.parametrize("padded", [True, False])
@pytest.mark.parametrize("shape", SHAPES)
def test_every_entry_is_checked(mpr, shape, padded):
    """One finite entry above MPR_FMAX is found wherever it lies, and MPR_FMAX
    and infinity are not mistaken for one."""
    rows, cols = shape
    X = np.full((rows, cols), 0x7FFF, dtype=np.uint16)
    X[::2, ::3] = mpr.INF
    other = mpr.to_device(np.zeros((cols, 2), dtype=np.uint16))
    A = mpr.to_device(X) if padded else torch.from_numpy(X).cuda()
    C = mpr.alloc_matrix(rows, 2)
    at = {(0, 0), (rows - 1, cols - 1), (rows // 2, cols // 2), (rows // 3, max(0, cols - 9)), (rows - 1, 0)}
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    mpr.minplus_gemm(A, other, C=C, d_status=st)
    assert int(st.item()) == 0
    for i, j in at:
        keep = A[i, j].item()
        A[i, j] = 0x8000
        st.zero_()
        mpr.minplus_gemm(A, other, C=C, d_status=st)
        assert int(st.item()) == 3
        A[i, j] = keep


@pytest.mark.parametrize("padded", [True, False])
@pytest.mark.parametrize("shape", SHAPES)
def test_fold_of_any_shape(mpr, shape, padded):
    """The right operand K x N with its rows' offsets, some rows empty, against
    the product of the unfolded matrices."""
    K, N = shape
    X, Y = synth.random_matrix(2, K, 3, 0, 50, 0.2), synth.random_matrix(K, N, 4, 0, 50, 0.2)
    X[:, K // 2] = 1
    rng = np.random.default_rng(K)
    R = rng.integers(1000, 1100, K)
    if K > 2:
        Y[1], R[1] = mpr.INF, mpr.ROW_NONE
    wide = O.from_u16(Y)
    full = np.where(wide == O.INF, O.INF, wide + np.where(R == mpr.ROW_NONE, 0, R)[:, None])
    A = mpr.to_device(X)
    B = mpr.to_device(Y) if padded else torch.from_numpy(Y).cuda()
    C, Rc = mpr.minplus_gemm_norm(A, B, Rb=torch.from_numpy(R).cuda())
    Nw, Rw = O.normalise(O.minplus(O.from_u16(X), full))
    assert np.array_equal(C.cpu().numpy(), O.to_u16(Nw)) and np.array_equal(Rc.cpu().numpy(), Rw)
