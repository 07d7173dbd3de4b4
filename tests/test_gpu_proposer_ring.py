"""Host arrays of the proposer travel through a small ring of pinned slots: calls
at the edges of a slot, of the ring and of the pinned outputs give the rows'
results whatever the parts they travel in; a refused inference writes nothing, and
input and output may share memory."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SLOT = 1 << 18   # floats


@pytest.fixture(scope="module")
def morap():
    from paper_2305_04397_amd import morap as m
    return m


@pytest.mark.parametrize("n_in,d,n", [
    (1024, 512, 255), (1024, 512, 256), (1024, 512, 257), (1024, 512, 1024), (1024, 512, 1025),  # slots and the ring
    (1024, 512, 8191), (1024, 512, 8192), (1024, 512, 8193),                                    # pinned outputs or not
    (1, 1, SLOT), (1, 1, SLOT + 1), (1, 1, 8 * SLOT + 1), (37, 3, 4 * SLOT // 37 + 5),
    (2000, 3, 300), (1030, 600, 1800), (1030, 2, 100),                                          # layer by layer
])
def test_rows_in_any_number_of_parts(morap, n_in, d, n):
    rng = np.random.default_rng(n)
    X = rng.normal(0, 1, (n, n_in)).astype(np.float32)
    with morap.Context(0) as ctx:
        ctx.proposer_init(n_in, d, seed=2)
        P = ctx.proposer_infer(X, d)
        assert np.abs(P.sum(1) - 1).max() <= 1e-5
        for r in {0, n // 3, n - 1}:     # a row's result is its own, alone or among others
            assert np.array_equal(ctx.proposer_infer(X[r:r + 1], d)[0], P[r])
        assert np.array_equal(ctx.proposer_infer(X, d), P)


@pytest.mark.parametrize("n_in,d,n", [(62, 30, 4096), (300, 40, 2 * SLOT // 300 + 1), (1024, 512, 700), (1100, 20, 500), (62, 30, 9)])
def test_steps_over_several_slots(morap, n_in, d, n):
    """Loss and gradients of all rows are the weighted sums of the parts'."""
    rng = np.random.default_rng(n)
    X = rng.normal(0, 1, (n, n_in)).astype(np.float32)
    T = rng.dirichlet(np.ones(d), n).astype(np.float32)
    with morap.Context(0) as ctx:
        ctx.proposer_init(n_in, d, seed=2)
        loss, grads = ctx.proposer_step(X, T)
        again, g2 = ctx.proposer_step(X, T)
        assert again == loss and np.array_equal(g2, grads)
        h = n // 2
        (la, ga), (lb, gb) = ctx.proposer_step(X[:h], T[:h]), ctx.proposer_step(X[h:], T[h:])
        assert loss == pytest.approx((h * la + (n - h) * lb) / n, rel=1e-5)
        # (each part rounds its output gradients, scaled by its own row count, to BF16)
        scale = np.abs(grads).max()
        assert np.abs(grads - (h * ga + (n - h) * gb) / n).max() <= 2 ** -7 * scale


def test_refused_inference_writes_nothing_and_arrays_may_overlap(morap):
    n_in, d, n = 64, 64, 9000
    rng = np.random.default_rng(1)
    X = rng.normal(0, 1, (n, n_in)).astype(np.float32)
    ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)  # noqa: E731
    with morap.Context(0) as ctx:
        ctx.proposer_init(n_in, d, seed=2)
        want = ctx.proposer_infer(X, d)
        bad = X.copy()
        bad[-1, -1] = np.nan
        out = np.full((n, d), 7, np.float32)
        assert morap.lib.morap_proposer_infer(ctx._h, ptr(bad), n, ptr(out)) == morap.E_INVALID
        assert (out == 7).all()
        buf = X.copy()
        assert morap.lib.morap_proposer_infer(ctx._h, ptr(buf), n, ptr(buf)) == 0
        assert np.array_equal(buf, want)
