"""The block shapes that products, chain steps and batches take between 160
and 255 tiles of 128 x 128, and 128 x 256 blocks with ragged edges, with values
in the levels, past them, and past 2048: against the uint16 configuration 0
(itself checked against the oracle)."""
import numpy as np
import pytest
import torch

import oracle as O
import synth

pytestmark = pytest.mark.gpu

SHAPES = [(1700, 1730, 135), (1000, 3333, 300), (2500, 2570, 135), (2049, 6200, 192)]
LAWS = [(0, 15, 0.3), (0, 200, 0.25), (22, 23, 0.99), (14, 40, 0.3), (0, 3000, 0.25), (1000, 10000, 0.2),
        (1500, 0x7FFF, 0.2), (0, 1, 1.0)]


@pytest.fixture(scope="module")
def mpr():
    import paper_2409_17658_amd as m

    m.lib()
    m.init(0)
    return m


def _same(a, b):
    return torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("law", LAWS)
def test_products(mpr, law):
    for i, (M, N, K) in enumerate(SHAPES):
        print("blocks", law, (M, N, K), flush=True)
        lo, hi, inf = law
        X, Y = synth.random_matrix(M, K, 1 + i, lo, hi, inf), synth.random_matrix(K, N, 50 + i, lo, hi, inf)
        A = mpr.to_device(X) if i % 2 else torch.from_numpy(X).cuda()
        B = mpr.to_device(Y)
        ref = mpr.minplus_gemm(A, B, cfg=0)
        assert _same(mpr.minplus_gemm(A, B), ref)
        assert _same(mpr.minplus_gemm(A, B, spare=True), ref)
        rows = [0, 127, 128, M - 1]
        assert np.array_equal(ref.cpu().numpy()[rows], O.to_u16(O.minplus(O.from_u16(X[rows]), O.from_u16(Y))))


def test_products_of_mixed_blocks(mpr):
    """Rows past the levels in some blocks only, columns in others."""
    for M, N, K in SHAPES:
        X, Y = synth.random_matrix(M, K, 3, 0, 9, 0.4), synth.random_matrix(K, N, 4, 0, 9, 0.4)
        X[130:300] = np.where(X[130:300] == mpr.INF, mpr.INF, X[130:300] + 2500)
        Y[:, 900:1100] = np.where(Y[:, 900:1100] == mpr.INF, mpr.INF, Y[:, 900:1100] + 700)
        X[M - 1], Y[:, N - 2] = mpr.INF, mpr.INF
        A, B = mpr.to_device(X), mpr.to_device(Y)
        assert _same(mpr.minplus_gemm(A, B), mpr.minplus_gemm(A, B, cfg=0))


# Sizes whose products past the levels have a launch of their own (128 x 256
# blocks would leave CUs idle), and, launched to leave room, outputs of few
# columns, also fewer than 8.
PAST_SHAPES = [(3000, 3001, 136, False), (3050, 2900, 128, False), (33000, 9, 137, True), (33000, 8, 128, True),
               (33000, 7, 130, True), (2300, 2200, 200, True)]


@pytest.mark.parametrize("shape", PAST_SHAPES)
def test_products_past_the_levels(mpr, shape):
    """Whole products past the levels, mostly infinite ones, and ones of which
    some or most rows are: the same bits whichever launch takes a block."""
    M, N, K, spare = shape
    for law in LAWS + [(0, 20, 0.97), (900, 1100, 0.9)]:
        print("past the levels", shape, law, flush=True)
        lo, hi, inf = law
        X, Y = synth.random_matrix(M, K, 5, lo, hi, inf), synth.random_matrix(K, N, 6, lo, hi, inf)
        small = synth.random_matrix(M, K, 7, 0, 9, 0.2)
        for rows in (0, M // 10, 9 * M // 10):
            X[:rows] = small[:rows]
            A, B = mpr.to_device(X), mpr.to_device(Y)
            assert _same(mpr.minplus_gemm(A, B, spare=spare), mpr.minplus_gemm(A, B, cfg=0))


@pytest.mark.parametrize("shape", PAST_SHAPES[:2])
def test_products_partly_past_the_levels(mpr, shape):
    """Blocks in the levels beside ones for either VALU form, whose borders are no
    tile's: the launch behind computes whole tiles of them."""
    M, N, K, spare = shape
    X, Y = synth.random_matrix(M, K, 8, 0, 9, 0.2), synth.random_matrix(K, N, 9, 0, 9, 0.2)
    for at, size, more in [(100, 300, 600), (500, 700, 20000), (1300, 65, 600), (1500, 1, 20000), (M - 130, 130, 600)]:
        X[at : at + size] = np.where(X[at : at + size] == mpr.INF, mpr.INF, X[at : at + size] + more)
        Y[:, at + 90 : at + 90 + size] = np.where(
            Y[:, at + 90 : at + 90 + size] == mpr.INF, mpr.INF, Y[:, at + 90 : at + 90 + size] + more)
    A, B = mpr.to_device(X), mpr.to_device(Y)
    assert _same(mpr.minplus_gemm(A, B, spare=spare), mpr.minplus_gemm(A, B, cfg=0))


STEP_LAWS = [(0, 31, 0.25), (0, 60, 0.9), (2100, 3000, 0.2), (0x7000, 0x7FFF, 0.3), (0, 3000, 0.2)]


def _chain(mpr, A, e):
    """A^e by products of configuration 0 and normalisations."""
    N = A.clone()
    R = mpr.normalise(N)
    for _ in range(e - 1):
        N = mpr.minplus_gemm(N, A, cfg=0, check=False)
        R = mpr.normalise(N, R_in=R)
    return N, R


@pytest.mark.parametrize("n", [900, 1700, 2100])
@pytest.mark.parametrize("law", STEP_LAWS)
def test_chain_steps(mpr, n, law):
    """Chain steps normalised late (a workspace with room for their minima)."""
    lo, hi, inf = law
    A = mpr.to_device(synth.random_matrix(n, n, n, lo, hi, inf))
    for e in (2, 4):
        ws = mpr.workspace(mpr.power_workspace_size(n, e, mpr.CHAIN) + 32 * n + 4096)
        N, R = mpr.minplus_power(A, e, mpr.CHAIN, ws=ws)
        Nr, Rr = _chain(mpr, A, e)
        assert _same(N, Nr) and torch.equal(R, Rr)


@pytest.mark.parametrize("law", STEP_LAWS)
def test_batch_steps(mpr, law):
    """A batch of more than 256 tiles of 128 x 256, beside small chains."""
    lo, hi, inf = law
    chains, want = [], []
    for i, (n, e) in enumerate([(4101, 3), (300, 5), (1300, 2), (9, 4)]):
        A = mpr.to_device(synth.random_matrix(n, n, 70 + i, lo, hi, inf))
        chains.append((A, e, mpr.alloc_matrix(n, n), torch.empty(n, dtype=torch.int64, device="cuda")))
        want.append(_chain(mpr, A, e))
    mpr.batch_power(chains)
    for (_, _, N, R), (Nr, Rr) in zip(chains, want):
        assert _same(N, Nr) and torch.equal(R, Rr)


def test_batch_overflow_is_reported(mpr):
    n, e = 4101, 3
    X = np.full((n, n), mpr.INF, dtype=np.uint16)
    X[np.arange(n), (np.arange(n) + 1) % n] = 0x7FFF
    X[np.arange(n), np.arange(n)] = 0
    chain = (mpr.to_device(X), e, mpr.alloc_matrix(n, n), torch.empty(n, dtype=torch.int64, device="cuda"))
    with pytest.raises(mpr.MprError) as err:
        mpr.batch_power([chain])
    assert err.value.status == 3


@pytest.mark.parametrize("count", [7, 8, 21, 33])
def test_batch_of_many_small_chains(mpr, count):
    """Chains that go eight at a time, one to an XCD, beside ones that do not;
    within an eight they end at different powers and differ in size."""
    rng = np.random.default_rng(count)
    chains, want = [], []
    for i in range(count):
        n, e = (int(rng.integers(8, 400)), int(rng.integers(1, 7))) if i != 3 else (900, 4)
        X = synth.random_matrix(n, n, 100 * count + i, 0, 25 if i % 5 else 2600, 0.25)
        A = mpr.to_device(X)
        chains.append((A, e, mpr.alloc_matrix(n, n), torch.empty(n, dtype=torch.int64, device="cuda")))
        want.append(_chain(mpr, A, e))
    ws = mpr.workspace(mpr.batch_workspace_size(chains)).fill_(255)
    mpr.batch_plan(chains, ws)
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    stream = torch.cuda.Stream()
    graph = mpr.batch_graph_create(ws, st, stream)
    for launch in (lambda: mpr.batch_launch(ws, st), lambda: (torch.cuda.synchronize(), mpr.graph_launch(graph, stream))) * 2:
        for _, _, N, R in chains:
            N.view(torch.int16).fill_(9)
            R.fill_(9)
        launch()
        torch.cuda.synchronize()
        assert int(st.item()) == 0
        for (_, _, N, R), (Nr, Rr) in zip(chains, want):
            assert _same(N, Nr) and torch.equal(R, Rr)
    mpr.graph_destroy(graph)
