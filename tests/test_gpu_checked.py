"""Products that are checked on the way (minplus_gemm with check=True) at the
ends of the sizes that one block takes, read on another stream as soon as the
call has returned."""
import numpy as np
import pytest
import torch

import oracle as O
import synth

pytestmark = pytest.mark.gpu

# 1024 pairs of outputs and K = 127 in one block; one pair or one value more
# than it takes; K = 128 and outputs of the level form and of a VALU tile.
SHAPES = [(32, 64, 127), (31, 66, 127), (1024, 2, 3), (1024, 1, 8), (1, 2048, 7), (1, 2047, 8), (32, 65, 16),
          (1025, 1, 1), (33, 33, 33), (32, 64, 128), (300, 500, 90), (700, 900, 1000)]


@pytest.fixture(scope="module")
def mpr():
    import paper_2409_17658_amd as m

    m.lib()
    m.init(0)
    return m


@pytest.mark.parametrize("padded", [True, False])
@pytest.mark.parametrize("shape", SHAPES)
def test_checked_product_is_done_when_it_returns(mpr, shape, padded):
    M, N, K = shape
    other = torch.cuda.Stream()
    for lo, hi in ((0, 40), (0x7FF0, 0x7FFF)):
        print("checked product", shape, padded, (lo, hi), flush=True)
        X, Y = synth.random_matrix(M, K, 5, lo, hi, 0.2), synth.random_matrix(K, N, 6, lo, hi, 0.2)
        ref = O.to_u16(O.minplus(O.from_u16(X), O.from_u16(Y)))
        if padded:
            A, B = mpr.to_device(X), mpr.to_device(Y)
        else:
            A, B = torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda()
        C = mpr.alloc_matrix(M, N, fill=7)
        torch.cuda.synchronize()
        mpr.minplus_gemm(A, B, C=C)
        with torch.cuda.stream(other):
            got = C.clone()
        other.synchronize()
        assert np.array_equal(got.cpu().numpy(), ref)
        for bad in (A, B):
            keep = bad[-1, -1].item()
            bad[-1, -1] = 0x8000
            with pytest.raises(mpr.MprError) as e:
                mpr.minplus_gemm(A, B, C=C)
            assert e.value.status == 3
            bad[-1, -1] = keep
