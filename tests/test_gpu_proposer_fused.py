"""The proposer's fused kernels (networks of up to 1,024 inputs and 512
outputs) against the layer-by-layer kernels of larger networks.

The same network runs on both: padded with inputs that are zero and have zero
weights to 1,025 inputs, it takes the layer-by-layer path.  The padding adds
exact zeros after the other terms, and both paths accumulate a product over
its inputs in ascending steps of 32, so probabilities and losses are
bit-identical; gradients sum over the rows in another FP32 order, which the
standard summation bound covers (rounded BF16 operands are the same ones)."""
import ctypes

import numpy as np
import pytest

from oracle import mlp

pytestmark = pytest.mark.gpu
HID, U = 256, 2.0 ** -24
BIG = 1025


def _pad(flat, n_in, d):
    out = np.zeros((HID, BIG), np.float32)
    out[:, :n_in] = flat[:HID * n_in].reshape(HID, n_in)
    return np.concatenate([out.ravel(), flat[HID * n_in:]])


def _params(flat, n_in, d):
    sizes, out, o = (n_in, HID, HID, HID, d), [], 0
    for fi, fo in zip(sizes[:-1], sizes[1:]):
        out.append((flat[o:o + fo * fi].reshape(fo, fi).astype(np.float64), flat[o + fo * fi:o + fo * fi + fo]))
        o += fo * fi + fo
    return out


@pytest.mark.parametrize("n,n_in,d", [(1, 4, 1), (15, 33, 16), (16, 32, 17), (17, 62, 30), (32, 64, 65), (33, 5, 256),
                                      (545, 62, 30), (40, 1024, 512), (100, 151, 300)])
def test_fused_network_equals_the_layer_by_layer_one(n, n_in, d):
    from paper_2305_04397_amd import morap
    rng = np.random.default_rng(n * 7 + n_in + d)
    X = rng.normal(0, 1, (n, n_in)).astype(np.float32)
    T = rng.dirichlet(np.full(d, 0.3), size=n).astype(np.float32)
    XB = np.zeros((n, BIG), np.float32)
    XB[:, :n_in] = X
    with morap.Context(0) as a, morap.Context(0) as b:
        a.proposer_init(n_in, d, seed=n)
        flat = a.proposer_params()
        flat[-d:] = rng.normal(0, 0.1, d)
        a.proposer_set_params(flat)
        b.proposer_init(BIG, d, seed=1)
        b.proposer_set_params(_pad(flat, n_in, d))
        mu, sd = rng.normal(0, 0.2, n_in).astype(np.float32), rng.uniform(0.5, 2, n_in).astype(np.float32)
        a.proposer_set_input_norm(mu, sd)
        b.proposer_set_input_norm(np.concatenate([mu, np.zeros(BIG - n_in, np.float32)]),
                                  np.concatenate([sd, np.ones(BIG - n_in, np.float32)]))
        assert np.array_equal(a.proposer_infer(X, d), b.proposer_infer(XB, d))
        la, ga = a.proposer_step(X, T, apply=False)
        lb, gb = b.proposer_step(XB, T, apply=False)
        assert la == lb
        # |G| and |H| of the bound from the oracle (a few BF16 units more)
        params = _params(flat, n_in, d)
        xs = (X - mu) / sd
        P, (acts, _) = mlp.forward([(mlp.to_bf16(W), c) for W, c in params], xs, act_round=mlp.to_bf16)
        gl = np.abs(P - T) / n + 2.0 ** -8 / n
        # the order of the padded gradient, without the padding's
        gb = np.concatenate([gb[:HID * BIG].reshape(HID, BIG)[:, :n_in].ravel(), gb[HID * BIG:]])
        pa, pb = _params(ga, n_in, d), _params(gb, n_in, d)
        for l in range(3, -1, -1):
            k = 1.1 * 2 * (n + 32) * U
            H = np.abs(acts[l]) + 2.0 ** -6
            assert (np.abs(pa[l][0] - pb[l][0]) <= k * (gl.T @ H) + 1e-30).all(), l
            assert (np.abs(pa[l][1] - pb[l][1]) <= k * gl.sum(0) + 1e-30).all(), l
            gl = gl @ np.abs(params[l][0]) * (1 + 2.0 ** -6)
        # one update: every copy of the weights follows it (n_in inputs only)
        a.proposer_step(X, T, apply=True, lr=1e-2)
        b.proposer_set_params(_pad(a.proposer_params(), n_in, d))
        assert np.array_equal(a.proposer_infer(X, d), b.proposer_infer(XB, d))


@pytest.mark.parametrize("offset", [0, 1000, -900])
def test_noalloc_output_may_overlap_its_input(offset):
    """W_out inside, behind and before X in one allocation: the outputs of
    separate buffers."""
    from paper_2305_04397_amd import morap
    h = ctypes.CDLL("libamdhip64.so")
    h.hipMalloc.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_size_t]
    h.hipFree.argtypes = [ctypes.c_void_p]
    h.hipMemcpy.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]
    n, n_in, d = 300, 62, 30
    X = np.random.default_rng(3).normal(0, 1, (n, n_in)).astype(np.float32)
    with morap.Context(0) as c:
        c.proposer_init(n_in, d, seed=5)
        ref = c.proposer_infer(X, d)
        p = ctypes.c_void_p()
        assert h.hipMalloc(ctypes.byref(p), 1 << 20) == 0
        try:
            x = p.value + 65536
            assert h.hipMemcpy(x, X.ctypes.data, X.nbytes, 1) == 0
            c.proposer_infer_noalloc(x, n, x + 4 * offset)
            assert h.hipDeviceSynchronize() == 0
            out = np.zeros((n, d), np.float32)
            assert h.hipMemcpy(out.ctypes.data, x + 4 * offset, out.nbytes, 2) == 0
        finally:
            h.hipFree(p)
        assert np.array_equal(out, ref)


@pytest.mark.parametrize("n_in,d,n", [(62, 30, 1056), (62, 30, 1057), (62, 30, 8448), (62, 30, 8449), (500, 20, 1000),
                                      (1, 1, 70000)])
def test_inference_of_host_rows_in_parts(n_in, d, n):
    """Rows are independent: a call that goes in several launches gives what
    calls of a few rows each give; a row that is not finite in the last part
    refuses the call, and the next one is served."""
    from paper_2305_04397_amd import morap
    rng = np.random.default_rng(n)
    X = rng.normal(0, 1, (n, n_in)).astype(np.float32)
    with morap.Context(0) as c:
        c.proposer_init(n_in, d, seed=3)
        P = c.proposer_infer(X, d)
        for r in sorted({0, n // 3, n // 2, n - 40}):
            assert np.array_equal(P[r:r + 40], c.proposer_infer(X[r:r + 40], d)), r
        bad = X.copy()
        bad[-1, -1] = np.inf
        with pytest.raises(morap.MorapError) as e:
            c.proposer_infer(bad, d)
        assert e.value.code == morap.E_INVALID
        assert np.array_equal(c.proposer_infer(X, d), P)
