"""Value iteration with the values in LDS (the solver's own choice for
products that fit a workgroup) against the batched neighbourhood-block sweep
(a fixed schedule): the same bits in every value, the same stopping sweeps,
backups and floor stops, at the edges of its register steps and column
groups."""
import dataclasses

import numpy as np
import pytest

from workloads import make_workload, tiny_workload, dirichlet_weights
from workloads.gridworld import Task, Workload, make_agent

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


def _corridor(sizes, width=None):
    """One agent per size on a grid of that many cells plus the goal (the
    last cell), one reach task: products of exactly `size` live states."""
    agents, letters = [], []
    rng = np.random.default_rng(len(sizes))
    for n in sizes:
        w = min(n + 1, width or 32)
        h = -(-(n + 1) // w)
        free = np.zeros((h, w), bool)
        free.ravel()[:n + 1] = True
        a = make_agent(rng, free, 0, 0.1, rng.uniform(1.0, 3.0, 5))
        lab = np.zeros(a.n_states, np.int32)
        lab[-1] = 1
        agents.append(a)
        letters.append([lab])
    task = Task(kind="reach", k=1, n_locs=2, n_letters=2, q0=0, delta=np.array([[0, 1], [1, 1]], np.int32),
                accepting=np.array([0, 1], np.uint8), waypoints_uv=np.zeros((0, 2, 2)), avoid_uv=None)
    return Workload(name="corridors", agents=agents, tasks=[task], letters=letters)


def _compare(ctx, morap, wl, K, prec, eps, schedule, seed=0, resident=None):
    nI, nJ = wl.n_agents, wl.n_tasks
    W = dirichlet_weights(np.random.default_rng(seed), K, nI + nJ)
    W[0] = np.eye(nI + nJ)[nI]        # a probability alone: every cost weight is 0
    c1, s1 = ctx.solve(W, morap.Options(eps_vi=eps, precision=prec))
    models = range(nI * nJ)
    cols = sorted({0, K // 2, K - 1})
    x1 = {(k, m): ctx.get_values(k, m) for m in models for k in cols}
    c0, s0 = ctx.solve(W, morap.Options(eps_vi=eps, precision=prec, schedule=schedule))
    assert s0["resident_models"] == 0
    assert s1["resident_models"] == (nI * nJ if resident is None else resident)
    assert np.array_equal(c1, c0)
    for f in ("backups", "sweeps", "max_pair_sweeps", "floor_stops"):
        assert s1[f] == s0[f], f
    assert s1["bytes"] + s1["bytes_tail"] == pytest.approx(s0["bytes"], rel=1e-12)
    for (k, m), x in x1.items():
        assert np.array_equal(x, ctx.get_values(k, m)), (k, m)
    return s1


def _block(morap, K):
    """A neighbourhood-block variant of one lane group of min(Kp, 64) columns."""
    Kp = 1
    while Kp < K:
        Kp *= 2
    return {1: 19, 2: 20, 4: 22, 8: 25, 16: 28, 32: 31}.get(Kp, 37)


@pytest.mark.parametrize("sizes", [(1, 2, 63, 64, 65), (511, 512, 513), (1024, 1025), (1536, 1537), (2048, 2049),
                                   (2560, 2561), (3583, 3584)])
@pytest.mark.parametrize("prec,K", [("f32", 64), ("f32", 3), ("f32", 1)])
def test_register_steps_f32(ctx, morap, sizes, prec, K):
    wl = _corridor(sizes)
    ctx.build_products(wl)
    _compare(ctx, morap, wl, K, prec, 1e-6, _block(morap, K), seed=K)


@pytest.mark.parametrize("sizes", [(1, 64, 511, 512), (513, 1024), (1025, 1536), (1537, 2048), (2049, 2560), (2561,)])
@pytest.mark.parametrize("K", [1, 5, 40])
def test_register_steps_f64(ctx, morap, sizes, K):
    wl = _corridor(sizes)
    ctx.build_products(wl)
    _compare(ctx, morap, wl, K, "f64", 1e-9, _block(morap, K), seed=K)


@pytest.mark.parametrize("prec,K", [("f32", 64), ("f32", 1), ("f64", 5)])
def test_larger_products(ctx, morap, prec, K):
    """Products beyond the first kernel: states sorted by block, one iterate
    in LDS, four, two or one columns per workgroup."""
    wl = _corridor((100, 2049, 3585, 4161, 9700, 11000, 19000), width=80)
    ctx.build_products(wl)
    _compare(ctx, morap, wl, K, prec, 1e-6, _block(morap, K), seed=K)


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_largest_products_take_the_batched_sweeps(ctx, morap, prec):
    """Products beyond a workgroup's LDS beside products within it."""
    wl = _corridor((100, 3000, 21000, 39000, 45000), width=200)
    ctx.build_products(wl)
    st = _compare(ctx, morap, wl, 64, prec, 1e-6, 37, resident=4 if prec == "f32" else 2)
    assert 18 < st["variant"] <= 40


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_many_products(ctx, morap, prec):
    """More column groups than workgroups fit at once (several columns each)."""
    wl = make_workload(2, n_agents=5, n_tasks=12)
    ctx.build_products(wl)
    _compare(ctx, morap, wl, 70, prec, 1e-6, 37)


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_general_blocks(ctx, morap, prec):
    """Blocks outside the grid pattern, costs that differ between states, and
    a self-successor in another location: the general form."""
    rng = np.random.default_rng(3)
    base = tiny_workload(3, 2, 1, width=6, height=5, kinds=("reach",), k=1)
    # costs per state
    wl = dataclasses.replace(base, agents=[dataclasses.replace(a, cost=rng.uniform(1, 3, a.cost.size))
                                           for a in base.agents])
    ctx.build_products(wl)
    _compare(ctx, morap, wl, 8, prec, 1e-7, 25)
    # a counting automaton that advances while the agent stays on a waypoint
    delta = np.array([[0, 1], [1, 2], [2, 3], [3, 3]], dtype=np.int32)
    wl = dataclasses.replace(base, tasks=[Task(kind="count", k=3, n_locs=4, n_letters=2, q0=0, delta=delta,
                                               accepting=np.array([0, 0, 0, 1], np.uint8),
                                               waypoints_uv=np.zeros((0, 2, 2)), avoid_uv=None)])
    for i, a in enumerate(wl.agents):
        lab = np.zeros(a.n_states, np.int32)
        lab[[1, 5]] = 1
        lab[a.init] = 0
        wl.letters[i][0] = lab
    ctx.build_products(wl)
    _compare(ctx, morap, wl, 8, prec, 1e-7, 25)
    # two actions over four successors, the state itself not among them
    n = 700
    succ = (np.arange(n)[:, None, None] + np.array([[1, 7, 50, 333], [333, 50, 1, 7]])) % n
    ptr = np.arange(0, 8 * n + 1, 4)
    a = dataclasses.replace(base.agents[0], n_actions=2, cells=np.arange(n, dtype=np.int32), init=0,
                            sa_ptr=ptr.astype(np.int32), succ=succ.ravel().astype(np.int32),
                            prob=np.tile([0.4, 0.3, 0.2, 0.1], 2 * n), cost=np.tile([1.0, 2.0], n))
    wl = Workload(name="wide", agents=[a, a], tasks=base.tasks, letters=[[(np.arange(n) % 97 == 5).astype(np.int32)]] * 2)
    ctx.build_products(wl)
    _compare(ctx, morap, wl, 64, prec, 1e-7, 37)


def test_sweep_limit_and_long_solves(ctx, morap):
    """Solves longer than one launch give the same bits; one over its sweep
    limit is NOT_CONVERGED and names pairs, and the context goes on."""
    # an agent that moves on with probability 5e-4: tens of thousands of sweeps
    n = 6
    wl = _corridor((n - 1,))
    nxt = np.minimum(np.arange(n) + 1, n - 1)
    chain = dataclasses.replace(wl.agents[0], n_actions=1, sa_ptr=np.arange(0, 2 * n + 1, 2, dtype=np.int32),
                                succ=np.stack([np.arange(n), nxt], 1).ravel().astype(np.int32),
                                prob=np.tile([0.9995, 0.0005], n), cost=np.full(n, 1.0))
    slow = dataclasses.replace(wl, agents=[chain])
    ctx.build_products(slow)
    st = _compare(ctx, morap, slow, 4, "f64", 1e-9, 22)
    assert st["max_pair_sweeps"] > 2 * 4096
    W = dirichlet_weights(np.random.default_rng(1), 4, 2)
    for limit in (10, 5000):
        with pytest.raises(morap.MorapError) as e:
            ctx.solve(W, morap.Options(eps_vi=1e-9, precision="f64", max_sweeps=limit))
        assert e.value.code == morap.E_NOT_CONVERGED and "column" in str(e.value)
    c, _ = ctx.solve(W, morap.Options(eps_vi=1e-9, precision="f64"))
    assert np.isfinite(c).all()


def test_costs_too_large_for_the_matrix_path(ctx, morap):
    """Larger FP32 products of costs above 1e25 take the batched sweeps (a
    slot an action does not reach must add nothing); smaller ones stay."""
    wl = _corridor((100, 4000), width=80)
    huge = dataclasses.replace(wl, agents=[dataclasses.replace(a, cost=a.cost * 1e26) for a in wl.agents])
    ctx.build_products(huge)
    _compare(ctx, morap, huge, 4, "f32", 1e-6, 22, resident=1)
