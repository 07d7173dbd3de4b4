"""A refused training step leaves nothing on its way: the rows' upload runs while
the targets are checked, and its source is the caller's array (large calls) or
pinned memory that the next call writes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_in", [(3000, 1024), (12000, 1024)])   # 3 and 12 million floats: staged, and not
def test_refused_targets_leave_the_stream_idle(n, n_in):
    import torch
    from paper_2305_04397_amd import morap
    rng = np.random.default_rng(n)
    X = rng.normal(0, 1, (n, n_in)).astype(np.float32)
    T = np.full((n, 2), 0.5, np.float32)
    stream = torch.cuda.Stream()
    with morap.Context(0, stream=stream) as ctx:
        ctx.proposer_init(n_in, 2, seed=3)
        good, g0 = ctx.proposer_step(X, T)
        for bad in (-0.5, np.nan, 2.0):
            B = T.copy()
            B[0, 1] = bad
            with pytest.raises(morap.MorapError) as e:
                ctx.proposer_step(X, B)
            assert e.value.code == morap.E_INVALID
            assert stream.query()
        # (input refused behind rows that were fine)
        Y = X.copy()
        Y[-1, -1] = np.inf
        for call in (lambda: ctx.proposer_step(Y, T), lambda: ctx.proposer_infer(Y, 2)):
            with pytest.raises(morap.MorapError):
                call()
            assert stream.query()
        again, g1 = ctx.proposer_step(X, T)
        assert again == good and np.array_equal(g0, g1)
