"""Several columns a workgroup where they stop at different sweeps, and fewer
columns than a workgroup's widest group: the LDS iterations against the batched
sweeps, every value of every column the same bits.  (A group of columns is taken
only where a solve has more (product, column) pairs than twice the device's
compute units.)"""
import dataclasses

import numpy as np
import pytest

from workloads import make_workload, dirichlet_weights
from workloads.gridworld import make_agent

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


def _batched(blocks, K):
    """A batched sweep of one lane group of the padded width."""
    Kp = 1
    while Kp < K:
        Kp *= 2
    return ({1: 19, 2: 20, 4: 22} if blocks else {1: 1, 2: 2, 4: 4})[Kp]


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("K", [1, 2, 3])
@pytest.mark.parametrize("form", ["blocks", "rows"])
def test_fewer_columns_than_a_group(ctx, morap, form, prec, K):
    """One to three columns of more products than twice the compute units: no
    group reaches past the columns the buffers hold.  Products of every kernel:
    small, larger (sorted by block; streamed rows), one of the batched sweeps."""
    wl = make_workload(1)
    rng = np.random.default_rng(K)
    sides = [3 + i % 4 for i in range(22)] + [64]
    agents = [make_agent(rng, np.ones((s, s), bool), 0, 0.1, rng.uniform(1, 3, 5)) for s in sides]
    tasks = [wl.tasks[0]] * 24
    letters = [[np.where(np.arange(s * s) == s * s - 1, 1 + j % 2, 0).astype(np.int32) for j in range(24)] for s in sides]
    for rows, s in zip(letters, sides):
        for j, lab in enumerate(rows):
            lab[s * s // 2 + j % 2] = 2 - j % 2
            lab[0] = 0
    wl = dataclasses.replace(wl, agents=agents, tasks=tasks, letters=letters)
    nI, nJ = len(sides), 24
    if form == "blocks":
        ctx.build_products(wl)
    else:
        ctx.load_models([morap.product_host(a, t, letters[i][j]) for i, a in enumerate(agents)
                         for j, t in enumerate(tasks)], nI, nJ)
    W = dirichlet_weights(np.random.default_rng(K), K, nI + nJ)
    _same_everywhere(ctx, morap, W, nI, nJ, prec, _batched(form == "blocks", K), nI * nJ)
    # a query's later passes start from the values before
    t = np.concatenate([np.full(nI, -300.0), np.full(nJ, 0.9)])
    q = [ctx.query(t, eps=1e-3, max_iter=4, opts=morap.Options(eps_vi=1e-7, precision=prec, schedule=sched), warm_start=True)
         for sched in (0, _batched(form == "blocks", 1))]
    assert q[0]["verdict"] == q[1]["verdict"] and q[0]["iterations"] == q[1]["iterations"]
    assert np.allclose(q[0]["t_up"], q[1]["t_up"], rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("K", [64, 1])
def test_larger_products_before_the_largest(ctx, morap, K):
    """FP32 products of four, two and one columns a workgroup, each followed by
    one of nearly 40,000 states in the records: what a wave reads ahead past its
    product's last step names LDS rows that its own launch does not have."""
    rng = np.random.default_rng(K)
    agents, letters = [], []
    for n in (3700, 39200, 9700, 39500, 19000, 39700, 3585):
        free = np.zeros((-(-(n + 1) // 200), 200), bool)
        free.ravel()[:n + 1] = True
        a = make_agent(rng, free, 0, 0.1, rng.uniform(1.0, 3.0, 5))
        lab = np.zeros(a.n_states, np.int32)
        lab[-1] = 1
        agents.append(a)
        letters.append([lab])
    base = make_workload(1)
    task = dataclasses.replace(base.tasks[0], kind="reach", k=1, n_locs=2, n_letters=2, q0=0,
                               delta=np.array([[0, 1], [1, 1]], np.int32), accepting=np.array([0, 1], np.uint8),
                               waypoints_uv=np.zeros((0, 2, 2)), avoid_uv=None)
    wl = dataclasses.replace(base, agents=agents, tasks=[task], letters=letters)
    ctx.build_products(wl)
    n = len(agents)
    W = dirichlet_weights(np.random.default_rng(K), K, n + 1)
    _same_everywhere(ctx, morap, W, n, 1, "f32", 37 if K == 64 else 19, n)
