"""Policies and evaluations of assigned pairs in LDS (one workgroup per pair)
at the edges of their register steps and beyond what LDS holds, against the
oracle: policies greedy for its converged values off ties, values equal to the
exact evaluation of the device's own policies."""
import dataclasses

import numpy as np
import pytest

from oracle import product, vi
from tests.test_gpu_resident import _corridor

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


@pytest.mark.parametrize("sizes", [(1, 64, 511, 512, 513), (1024, 1025, 1536), (1537, 2048, 2049), (2560, 2561),
                                   (3584, 3585, 5100), (9900, 10400)])
@pytest.mark.parametrize("prec,from_values", [("f64", False), ("f32", True)])
def test_policies_and_values(ctx, morap, sizes, prec, from_values):
    """Column k assigns the task to agent k: one instance of every size.  The
    evaluation stops at a change of 1e-10; a state of these grids is left
    after fewer than 1e4 steps in expectation, so its error is below 1e-6."""
    wl = _corridor(sizes, width=100)
    n = len(sizes)
    ctx.build_products(wl)
    rng = np.random.default_rng(n)
    W = rng.dirichlet(np.ones(n + 1), size=n)
    o = morap.Options(eps_vi=1e-10 if prec == "f64" else 1e-6, eps_eval=1e-10, precision=prec,
                      eval_from_values=from_values)
    ctx.solve(W, o)
    o = dataclasses.replace(o, eps_vi=1e-10)
    r, st = ctx.evaluate(np.arange(n)[:, None], o)
    assert st["eval_sweeps"] > 0 and st["polish_sweeps"] > 0
    for k, size in enumerate(sizes):
        p = product.build_product(wl.agents[k], wl.tasks[0], wl.letters[k][0])
        assert p.n_states == size
        mu = ctx.get_policy(k, 0, size).astype(np.int64)
        assert (mu >= 0).all()
        ex = vi.evaluate_exact(p, mu)
        assert r[k, k] == pytest.approx(ex[p.init, 0], rel=1e-6, abs=1e-6)
        assert r[k, n] == pytest.approx(ex[p.init, 1], rel=1e-6, abs=1e-6)
        a, b = np.array([W[k, k], W[k, n]]) / (W[k, k] + W[k, n])
        x, _ = vi.value_iteration(p, np.array([a]), np.array([b]), 1e-11)
        best, gap = vi.q_gaps(p, vi.q_values(p, x[:, 0], a, b)[:, 0])
        clear = gap > 1e-6
        assert not (clear & (mu != best)).any(), (k, size)


def test_unreachable_goal_is_improper(ctx, morap):
    """No action leads to done: under a probability-only weight the values
    converge (to 0) and the attractor ranks no state."""
    wl = _corridor((40,))
    wl = dataclasses.replace(wl, letters=[[np.zeros(41, np.int32)]])
    ctx.build_products(wl)
    with pytest.raises(morap.MorapError) as e:
        ctx.support(np.array([[0.0, 1.0]]), morap.Options(eps_vi=1e-8, precision="f64"))
    assert e.value.code == morap.E_IMPROPER


def test_evaluation_over_its_sweep_limit(ctx, morap):
    """NOT_CONVERGED names the column; the policies stay readable and the
    context goes on."""
    wl = _corridor((300,))
    ctx.build_products(wl)
    W = np.array([[0.5, 0.5]])
    o = morap.Options(eps_vi=1e-9, precision="f64")
    ctx.solve(W, o)
    with pytest.raises(morap.MorapError) as e:
        ctx.evaluate(np.zeros((1, 1), np.int32), dataclasses.replace(o, eps_vi=1e-1, max_sweeps=8, check_every=2))
    assert e.value.code == morap.E_NOT_CONVERGED
    r, _ = ctx.evaluate(np.zeros((1, 1), np.int32), o)
    assert np.isfinite(r).all() and r[0, 1] == pytest.approx(1.0, abs=1e-6)
