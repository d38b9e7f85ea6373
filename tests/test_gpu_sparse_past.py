"""Compressed-K steps whose values leave the matrix-core levels, wholly or in
some tiles: below 7000 states their tiles are computed where they are, from
there on by the entry-list form.  Chains (rows normalised as the next step
reads them, and by a pass of their own) and period searches against the tile
form of the step."""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mpr():
    import paper_2409_17658_amd as m

    m.lib()
    m.init(0)
    yield m
    m.set_sparse_form("auto")


def _same(a, b):
    return torch.equal(a.view(torch.int16), b.view(torch.int16))


def _matrix(mpr, n, law):
    lo, hi, inf = law
    X = synth.random_matrix(n, n, 40 + n, lo, hi, inf)
    X[:, 128:192] = mpr.INF  # columns without an entry
    X[5] = mpr.INF
    if lo == 0 and hi > 100:  # some row panels and column blocks stay in the levels
        X[300:600] = np.where(X[300:600] == mpr.INF, mpr.INF, X[300:600] % 7)
        X[:, 640:700] = np.where(X[:, 640:700] == mpr.INF, mpr.INF, X[:, 640:700] % 5)
    return mpr.to_device(X)


# all past the levels, some, none; offsets past 0x7FFF; mostly past 2047
LAWS = [(100, 900, 0.97), (0, 3000, 0.97), (0, 12, 0.97), (0x7000, 0x7FFF, 0.98), (1500, 9000, 0.8)]


@pytest.mark.parametrize("law", LAWS)
@pytest.mark.parametrize("n", [72, 700, 1999, 7000, 7603])
def test_chains_past_the_levels(mpr, n, law):
    A = _matrix(mpr, n, law)
    for e in (2, 3, 5):
        print("sparse past", n, law, e, flush=True)
        mpr.set_sparse_form("tiles")
        Nr, Rr = mpr.minplus_power(A, e, mpr.CHAIN_SPARSE)
        mpr.set_sparse_form("auto")
        late = mpr.workspace(mpr.power_workspace_size(n, e, mpr.CHAIN) + 256 + mpr.sparse_plan_bytes(A)).fill_(255)
        N, R = mpr.minplus_power(A, e, mpr.CHAIN_SPARSE, ws=late)
        assert _same(N, Nr) and torch.equal(R, Rr)
        if n < 7000:  # a workspace of the worst case: a pass of its own normalises every step
            each = mpr.workspace(mpr.power_workspace_size(n, e, mpr.CHAIN_SPARSE)).fill_(255)
            N, R = mpr.minplus_power(A, e, mpr.CHAIN_SPARSE, ws=each)
            assert _same(N, Nr) and torch.equal(R, Rr)


@pytest.mark.parametrize("n", [72, 700, 7003])
def test_period_search_past_the_levels(mpr, n):
    """A search that starts again in 16 bits, with its traces and period."""
    X = np.full((n, n), mpr.INF, dtype=np.uint16)
    rng = np.random.default_rng(n)
    i = np.arange(n)
    X[i, (i + 1) % 3 + i // 3 * 3 % (n - 3)] = rng.integers(0, 900, n)
    X[i, rng.integers(0, n, n)] = rng.integers(0, 2500, n)
    A = mpr.to_device(X)
    got = []
    for form in ("tiles", "auto"):
        mpr.set_sparse_form(form)
        mu, lam, c, tr = mpr.find_period(A, 8, slots=4, sparse=True)
        got.append((mu, lam, c, tr.tolist()))
    assert got[0] == got[1]


def test_steps_that_come_back_into_the_levels(mpr):
    """Costs that are large in one step only: a first power far past the levels
    whose products are not."""
    n = 7100
    X = np.full((n, n), mpr.INF, dtype=np.uint16)
    i = np.arange(n)
    X[:, 0] = 5000 + i % 3
    X[0] = i % 9
    X[i, i] = 4000
    A = mpr.to_device(X)
    for e in (2, 3, 4, 7):
        mpr.set_sparse_form("tiles")
        Nr, Rr = mpr.minplus_power(A, e, mpr.CHAIN_SPARSE)
        mpr.set_sparse_form("auto")
        N, R = mpr.minplus_power(A, e, mpr.CHAIN_SPARSE)
        assert _same(N, Nr) and torch.equal(R, Rr)
