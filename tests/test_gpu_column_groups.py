"""Several columns a workgroup where they stop at different sweeps, and fewer
columns than a workgroup's widest group: the LDS iterations against the batched
sweeps, every value of every column the same bits.  (A group of columns is taken
only where a solve has more (product, column) pairs than twice the device's
compute units.)"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def morap():
    from paper_2305_04397_amd import morap as m
    return m


@pytest.fixture()
def ctx(morap):
    c = morap.Context(0)
    yield c
    c.close()


def _rows(rng, n, entries, leave=0.05):
    """n states of two rows of that many entries over any states."""
    R = 2 * n
    p = rng.random((R, entries)) + 0.05
    p *= (1 - leave) / p.sum(1, keepdims=True)
    return {"state_row": np.arange(0, R + 1, 2), "row_ptr": np.arange(0, R * entries + 1, entries),
            "col": rng.integers(0, n, R * entries).astype(np.int32), "prob": p.ravel(),
            "rew": np.stack([-rng.uniform(0.5, 2.0, R), rng.uniform(0, leave, R)], 1),
            "to_done": np.ones(R), "init": n // 3}


def _unlike_weights(K, nI, nJ):
    """Rows whose cost weight falls a hundredfold from one column to the next
    and back after four: the columns of a group stop far apart."""
    W = np.zeros((K, nI + nJ))
    s = 0.9 * 100.0 ** -(np.arange(K) % 4)
    W[:, :nI] = s[:, None] / nI
    W[:, nI:] = ((1 - s) / nJ)[:, None]
    return W / W.sum(1, keepdims=True)


def _same_everywhere(ctx, morap, W, nI, nJ, prec, schedule, resident, eps=1e-6):
    K, M = len(W), nI * nJ
    c1, s1 = ctx.solve(W, morap.Options(eps_vi=eps, precision=prec))
    x1 = [[ctx.get_values(k, m) for k in range(K)] for m in range(M)]
    c0, s0 = ctx.solve(W, morap.Options(eps_vi=eps, precision=prec, schedule=schedule))
    assert s0["resident_models"] == 0 and s1["resident_models"] == resident
    assert np.array_equal(c1, c0)
    for f in ("backups", "sweeps", "max_pair_sweeps", "floor_stops"):
        assert s1[f] == s0[f], f
    for m in range(M):
        for k in range(K):
            assert np.array_equal(x1[m][k], ctx.get_values(k, m)), (k, m)


@pytest.mark.parametrize("prec,sizes", [("f32", (4927, 4928, 4929, 9919, 9920, 9921)),
                                        ("f64", (2300, 4799, 4800, 4801, 9663, 9664))])
@pytest.mark.parametrize("entries", [2, 4])
def test_streamed_rows_whose_columns_stop_apart(ctx, morap, prec, sizes, entries):
    """Sizes on both sides of the limits of four, two and one columns, numbers of
    slices that the waves do not share evenly, and small ones: a wave that
    has stored a stopped column's values goes on with the next sweep while
    others still store."""
    rng = np.random.default_rng(entries)
    sizes = (300, 700, 1100) + sizes
    models = [_rows(rng, n, entries) for n in sizes]
    ctx.load_models(models, len(sizes), 1)
    _same_everywhere(ctx, morap, _unlike_weights(64, len(sizes), 1), len(sizes), 1, prec, 16, len(sizes))
