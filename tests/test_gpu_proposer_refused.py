"""A refused training step leaves nothing on its way: the rows' upload runs while
the targets are checked, and its source is the caller's array (large calls) or
pinned memory that the next call writes."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_in", [(3000, 1024), (12000, 1024)])   # 3 and 12 million floats: staged, and not
def test_refused_targets_leave_the_stream_idle(n, n_in):
    from paper_2305_04397_amd import morap
    hip = ctypes.CDLL("libamdhip64.so")   # (the runtime the library itself loaded)
    hip.hipStreamQuery.argtypes = hip.hipStreamDestroy.argtypes = [ctypes.c_void_p]
    stream = ctypes.c_void_p()
    assert hip.hipSetDevice(0) == 0 and hip.hipStreamCreateWithFlags(ctypes.byref(stream), 1) == 0

    def idle():
        return hip.hipStreamQuery(stream) == 0
    rng = np.random.default_rng(n)
    X = rng.normal(0, 1, (n, n_in)).astype(np.float32)
    T = np.full((n, 2), 0.5, np.float32)
    with morap.Context(0, stream=stream.value) as ctx:
        ctx.proposer_init(n_in, 2, seed=3)
        good, g0 = ctx.proposer_step(X, T)
        for bad in (-0.5, np.nan, 2.0):
            B = T.copy()
            B[0, 1] = bad
            with pytest.raises(morap.MorapError) as e:
                ctx.proposer_step(X, B)
            assert e.value.code == morap.E_INVALID
            assert idle()
        # (input refused behind rows that were fine)
        Y = X.copy()
        Y[-1, -1] = np.inf
        for call in (lambda: ctx.proposer_step(Y, T), lambda: ctx.proposer_infer(Y, 2)):
            with pytest.raises(morap.MorapError):
                call()
            assert idle()
        again, g1 = ctx.proposer_step(X, T)
        assert again == good and np.array_equal(g0, g1)
    assert hip.hipStreamDestroy(stream) == 0
