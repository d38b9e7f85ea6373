"""The product on the matrix cores (values 0..30 as powers of two) at the
edges of its blocks, slices and value range: the default configuration
against the explicit uint16 configuration 0 (another kernel, itself checked
against the oracle), bit for bit, and against the oracle on sampled rows."""
import numpy as np
import pytest
import torch

import oracle as O
import synth

pytestmark = pytest.mark.gpu

# (rows, columns, inner): K of whole and partial slices of 64, tiles of 64 and
# of 128 (from 256 tiles of 128 x 128 on) with and without remainders.
SHAPES = [(1, 4, 128), (64, 64, 129), (65, 67, 191), (130, 5, 200), (2048, 2048, 128), (2049, 2051, 135),
          (1, 33000, 160), (33000, 4, 137)]
# (least, largest, infinite): all sums in the levels; minima in, operands out
# of them; sums up to 44 and 45 (the ends of the float range); minima past
# 30; past 2048; nothing finite.
LAWS = [(0, 15, 0.3), (0, 200, 0.25), (22, 22, 0.99), (22, 23, 0.99), (14, 40, 0.3), (1500, 0x7FFF, 0.2), (0, 1, 1.0)]


@pytest.fixture(scope="module")
def mpr():
    import paper_2409_17658_amd as m

    m.lib()
    m.init(0)
    return m


def _law(rows, cols, seed, law):
    lo, hi, inf = law
    return synth.random_matrix(rows, cols, seed, lo, hi, inf)


@pytest.mark.parametrize("padded", [True, False])
@pytest.mark.parametrize("law", LAWS)
def test_level_product(mpr, law, padded):
    for i, (M, N, K) in enumerate(SHAPES):
        print("level product", law, padded, (M, N, K), flush=True)
        X, Y = _law(M, K, 1 + i, law), _law(K, N, 50 + i, law)
        if padded:
            A, B = mpr.to_device(X), mpr.to_device(Y)
        else:
            A, B = torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda()
        ref = mpr.minplus_gemm(A, B, cfg=0)
        assert torch.equal(mpr.minplus_gemm(A, B), ref)
        assert torch.equal(mpr.minplus_gemm(A, B, spare=True), ref)
        rows = sorted({0, M // 2, M - 1})
        assert np.array_equal(ref.cpu().numpy()[rows], O.to_u16(O.minplus(O.from_u16(X[rows]), O.from_u16(Y))))


def test_level_product_mixed_blocks(mpr):
    """One block out of the levels among blocks inside them, an all-infinite
    row and column, and single finite pairs at the ends of K."""
    n = 300
    X, Y = _law(n, n, 7, (0, 9, 0.5)), _law(n, n, 8, (0, 9, 0.5))
    X[70:75] = 900
    X[200], Y[:, 3] = mpr.INF, mpr.INF
    X[10], X[11] = mpr.INF, mpr.INF
    X[10, 0], X[11, n - 1] = 30, 29
    A, B = mpr.to_device(X), mpr.to_device(Y)
    assert np.array_equal(mpr.minplus_gemm(A, B).cpu().numpy(), O.to_u16(O.minplus(O.from_u16(X), O.from_u16(Y))))


# Chains whose rows stay in the levels; leave them (f16, then uint16 blocks);
# carry offsets past 0x7FFF; have no finite value at all.
STEP_LAWS = [(0, 31, 0.25), (0, 60, 0.9), (2100, 3000, 0.2), (0x7000, 0x7FFF, 0.3), (0, 9, 0.997)]


@pytest.mark.parametrize("law", STEP_LAWS)
def test_level_batch_steps(mpr, law):
    """A batch run step by step on the matrix cores (largest chain >= 192
    states), tile edges and chains of different lengths, against the
    oracle's chains."""
    print("level batch", law, flush=True)
    sizes = [(257, 5), (129, 7), (8, 3), (320, 1), (65, 2), (192, 6)]
    chains, refs = [], []
    for i, (n, e) in enumerate(sizes):
        X = _law(n, n, 900 + i, law)
        if i % 2:  # rows that are not 16-byte aligned
            A, N = torch.from_numpy(X).cuda(), torch.empty((n, n), dtype=torch.int16, device="cuda").view(torch.uint16)
        else:
            A, N = mpr.to_device(X), mpr.alloc_matrix(n, n)
        chains.append((A, e, N, torch.empty(n, dtype=torch.int64, device="cuda")))
        refs.append(O.power_chain(O.from_u16(X), e))
    ws = mpr.workspace(mpr.batch_workspace_size(chains))
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    mpr.batch_plan(chains, ws)
    for _ in range(2):  # the launch prepares all its state itself
        mpr.batch_launch(ws, st)
        assert int(st.item()) == 0
        for (_, _, N, R), (Nr, Rr) in zip(chains, refs):
            assert np.array_equal(N.cpu().numpy(), O.to_u16(Nr)) and np.array_equal(R.cpu().numpy(), Rr)


def test_level_batch_overflow_is_reported(mpr):
    """A row whose canonical values pass 0x7FFF: refused by the panel form
    (configuration 0) and by the step-by-step form alike."""
    n, e = 200, 4
    X = np.full((n, n), mpr.INF, dtype=np.uint16)
    X[np.arange(n), (np.arange(n) + 1) % n] = 0x7FFF
    X[np.arange(n), np.arange(n)] = 0
    status = []
    for cfg in (0, -1):
        mpr.set_batch_config(cfg)
        try:
            chain = (mpr.to_device(X), e, mpr.alloc_matrix(n, n), torch.empty(n, dtype=torch.int64, device="cuda"))
            ws = mpr.workspace(mpr.batch_workspace_size([chain]))
            st = torch.zeros(1, dtype=torch.int32, device="cuda")
            mpr.batch_plan([chain], ws)
            mpr.batch_launch(ws, st)
            status.append(int(st.item()))
        finally:
            mpr.set_batch_config(-1)
    assert status == [3, 3]


@pytest.mark.parametrize("n", [8, 11, 33, 72, 100, 129, 200])
def test_level_sparse_steps(mpr, n):
    """Compressed-K steps at the edges of their lists: blocks of 32 and of 64
    listed rows and more, a last group of fewer than 8 rows, a block of
    columns without entries, row strides of n; in a workspace full of ones,
    so a read past a list would not pass unnoticed."""
    for i, (inf, e) in enumerate([(0.9, 5), (0.3, 4), (0.995, 3)]):
        print("level sparse", n, inf, flush=True)
        X = synth.random_matrix(n, n, 300 + n + i, 0, 12, inf)
        if i == 2:
            X[:, 64:128] = mpr.INF
        A = torch.from_numpy(X).cuda() if i else mpr.to_device(X)
        N = torch.empty((n, n), dtype=torch.int16, device="cuda").view(torch.uint16)
        ws = mpr.workspace(mpr.power_workspace_size(n, e, mpr.CHAIN) + 256 + mpr.sparse_plan_bytes(A)).fill_(255)
        N, R = mpr.minplus_power(A, e, mpr.CHAIN_SPARSE, N_out=N, ws=ws)
        Nr, Rr = O.power_chain(O.from_u16(X), e)
        assert np.array_equal(N.cpu().numpy(), O.to_u16(Nr)) and np.array_equal(R.cpu().numpy(), Rr)


@pytest.mark.parametrize("shape", [(1, 1, 1), (3, 2, 7), (33, 33, 33), (127, 129, 127), (128, 128, 8), (129, 127, 9),
                                   (700, 900, 100)])
def test_small_products_and_their_check(mpr, shape):
    """The default product below the level form's sizes (tiny outputs, one
    thread per two columns, and the next size up), checked on the way: inputs
    at MPR_FMAX pass, one entry above it in either operand is refused."""
    M, N, K = shape
    for law in ((0, 40, 0.35), (0x7FF0, 0x7FFF, 0.2)):
        print("small product", shape, law, flush=True)
        X, Y = _law(M, K, 5, law), _law(K, N, 6, law)
        ref = O.to_u16(O.minplus(O.from_u16(X), O.from_u16(Y)))
        for A, B in ((mpr.to_device(X), mpr.to_device(Y)), (torch.from_numpy(X).cuda(), torch.from_numpy(Y).cuda())):
            assert np.array_equal(mpr.minplus_gemm(A, B).cpu().numpy(), ref)
            for bad in (A, B):
                keep = bad[-1, -1].item()
                bad[-1, -1] = 0x8000
                with pytest.raises(mpr.MprError) as e:
                    mpr.minplus_gemm(A, B)
                assert e.value.status == 3
                bad[-1, -1] = keep


@pytest.mark.parametrize("pipeline", [False, True])
@pytest.mark.parametrize("spread", [0, 25, 40, 300])
def test_period_search_in_bytes_and_past_them(mpr, spread, pipeline):
    """A period search keeps its powers in bytes while their values stay
    within 30 (spread 0, 25) and starts again when one does not (40: past the
    first power, 300: at once); period, traces and the observer's calls equal
    those of the dense search, which holds 16 bits throughout."""
    n, kmax = 75, 40
    X = np.full((n, n), mpr.INF, dtype=np.uint16)
    rng = np.random.default_rng(spread)
    for i in range(n):  # strongly connected, period 3, sparse
        X[i, (i + 1) % n] = rng.integers(0, 3)
        X[i, rng.integers(0, n)] = rng.integers(0, max(spread, 3) // 2 + 1)
    X[5, 6] = spread
    A = mpr.to_device(X)
    mpr.set_period_progress(lambda k, t: heard.append((k, t)))
    try:
        got = []
        for sparse in (False, True):
            heard = []
            mu, lam, c, tr = mpr.find_period(A, kmax, slots=30, sparse=sparse, pipeline=pipeline)
            assert [k for k, _ in heard] == list(range(1, kmax + 1))
            got.append((mu, lam, c, tr.tolist(), heard))
        assert got[0] == got[1]
    finally:
        mpr.set_period_progress(None)
    On = O.power_chain(O.from_u16(X), 7)
    assert int(O.trace(*On)) == got[1][3][7] if got[1][3][7] != mpr.ROW_NONE else True


@pytest.mark.parametrize("n", [8, 9, 15, 16, 17, 33, 63, 64, 65])
@pytest.mark.parametrize("top", [7, 30, 60])
def test_small_period_search(mpr, n, top):
    """Searches of at most 64 states take a power in one workgroup (65: not):
    the same period and traces as the dense search, the traces of the oracle's
    powers, for odd and even n, empty rows, and values past the byte range."""
    kmax = 24
    rng = np.random.default_rng(n + top)
    X = np.full((n, n + 5), mpr.INF, dtype=np.uint16)
    for i in range(n - 1):  # the last row is empty
        X[i, (i + 1) % (n - 2)] = rng.integers(0, 4)
        X[i, rng.integers(0, n)] = rng.integers(0, top + 1)
    X[n // 2, 0] = top
    A = mpr.to_device(X)[:, :n]
    want = mpr.find_period(A, kmax, slots=30, sparse=False)
    On = O.from_u16(X[:, :n])
    for pipeline in (False, True):
        got = mpr.find_period(A, kmax, slots=30, sparse=True, pipeline=pipeline)
        assert got[:3] == want[:3] and got[3].tolist() == want[3].tolist()
    for k in (1, 2, 5):
        assert got[3][k] == int(O.trace(*O.power_chain(On, k)))  # one value for "none" on both sides


@pytest.mark.parametrize("n", [66, 80, 1023, 1025, 4095, 4097, 8193])
def test_period_search_byte_passes(mpr, n):
    """The pass over a power in bytes at the ends of the sizes of its forms
    (2, 4 and 16 groups a thread, and more), with ragged last groups and rows:
    traces and period equal the dense search's."""
    kmax = 7
    rng = np.random.default_rng(n)
    X = np.full((n, n), mpr.INF, dtype=np.uint16)
    r = np.arange(n - 1)  # the last row is empty
    X[r, (r + 1) % 5 + (r // 5) * 5 % (n - 5)] = rng.integers(0, 4, n - 1)
    X[r, rng.integers(0, n, n - 1)] = rng.integers(0, 6, n - 1)
    A = mpr.to_device(X)
    want = mpr.find_period(A, kmax, slots=9, sparse=False)
    got = mpr.find_period(A, kmax, slots=9, sparse=True, pipeline=True)
    assert got[:3] == want[:3] and got[3].tolist() == want[3].tolist()
    assert any(t != mpr.ROW_NONE for t in got[3][1:])


@pytest.mark.parametrize("shape", [(300, 260, 1000), (2048, 2048, 193), (64, 70, 257), (2304, 2050, 128)])
@pytest.mark.parametrize("late", [False, True])
def test_blocks_that_give_up_early(mpr, shape, late):
    """Blocks whose first slices hold values past the levels leave the pass over
    K at once, or (late: only the first columns of K hold small values) after
    it; the product is the same."""
    M, N, K = shape
    X, Y = synth.random_matrix(M, K, 31, 0, 3000, 0.25), synth.random_matrix(K, N, 32, 0, 3000, 0.25)
    if late:
        X[:, : K // 2] = np.minimum(X[:, : K // 2], 9)
        Y[: K // 2] = np.minimum(Y[: K // 2], 9)
    A, B = mpr.to_device(X), mpr.to_device(Y)
    want = mpr.minplus_gemm(A, B, cfg=0, check=False)
    got = mpr.minplus_gemm(A, B, check=False)
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
