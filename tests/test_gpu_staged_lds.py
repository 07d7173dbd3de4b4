"""Stage retirement with the values in LDS (the solver's own choice when every
product fits a workgroup) against the batched sweeps of the same iteration (a
fixed schedule): the same bits in every value, the same retiring sweeps (their
backups, bytes and floor stops), at the edges of steps, column groups, stages
and launches."""
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


def _block(K):
    Kp = 1
    while Kp < K:
        Kp *= 2
    return {1: 19, 2: 20, 4: 22, 8: 25, 16: 28, 32: 31}.get(Kp, 37)


def _corridor(sizes, width=32, slip=0.1):
    """Products of exactly `size` states: that many cells plus the goal."""
    agents, letters = [], []
    rng = np.random.default_rng(len(sizes))
    for n in sizes:
        w = min(n + 1, width)
        free = np.zeros((-(-(n + 1) // w), w), bool)
        free.ravel()[:n + 1] = True
        agents.append(make_agent(rng, free, 0, slip, rng.uniform(1.0, 3.0, 5)))
        lab = np.zeros(agents[-1].n_states, np.int32)
        lab[-1] = 1
        letters.append([lab])
    task = Task(kind="reach", k=1, n_locs=2, n_letters=2, q0=0, delta=np.array([[0, 1], [1, 1]], np.int32),
                accepting=np.array([0, 1], np.uint8), waypoints_uv=np.zeros((0, 2, 2)), avoid_uv=None)
    return Workload(name="corridors", agents=agents, tasks=[task], letters=letters)


def _compare(ctx, morap, wl, K, prec, eps, seed=0, lds=True):
    ctx.build_products(wl)
    nI, nJ = wl.n_agents, wl.n_tasks
    W = dirichlet_weights(np.random.default_rng(seed), K, nI + nJ)
    W[0] = np.eye(nI + nJ)[nI]        # a probability alone: every cost weight is 0
    c1, s1 = ctx.solve_staged(W, morap.Options(eps_vi=eps, precision=prec))
    cols = sorted({0, K // 2, K - 1})
    x1 = {(k, m): ctx.get_values(k, m) for m in range(nI * nJ) for k in cols}
    c0, s0 = ctx.solve_staged(W, morap.Options(eps_vi=eps, precision=prec, schedule=_block(K)))
    assert s0["resident_models"] == 0 and (s1["resident_models"] > 0) == lds
    assert np.array_equal(c1, c0)
    for f in ("backups", "sweeps", "max_pair_sweeps", "floor_stops"):
        assert s1[f] == s0[f], f
    assert s1["bytes"] == pytest.approx(s0["bytes"], rel=1e-12)
    for (k, m), x in x1.items():
        assert np.array_equal(x, ctx.get_values(k, m)), (k, m)
    return s1


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("K", [1, 3, 40, 70])
def test_stages_of_small_products(ctx, morap, prec, K):
    """Up to nine stages in steps of 64: most steps span several."""
    _compare(ctx, morap, tiny_workload(7, 3, 4, width=7, height=6, kinds=("reach", "avoid"), k=7), K, prec, 1e-7, K)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("agents,tasks,K", [(5, 12, 64), (1, 3, 2)])
def test_stages_of_ordinary_products(ctx, morap, prec, agents, tasks, K):
    """Steps within one stage and across stages; many and few pairs."""
    _compare(ctx, morap, make_workload(2, n_agents=agents, n_tasks=tasks), K, prec, 1e-6)


@pytest.mark.parametrize("prec,K", [("f32", 64), ("f32", 1), ("f64", 40), ("f64", 1)])
def test_sizes_at_the_edges_of_the_classes(ctx, morap, prec, K):
    sizes = (1, 63, 64, 65, 511, 2040, 4900, 5100, 9700, 11000, 19000)
    _compare(ctx, morap, _corridor(sizes, width=80), K, prec, 1e-6)


def test_a_product_beyond_lds_takes_the_batched_sweeps(ctx, morap):
    _compare(ctx, morap, _corridor((100, 21000), width=200), 64, "f64", 1e-6, lds=False)
    _compare(ctx, morap, _corridor((100, 45000), width=200), 64, "f32", 1e-6, lds=False)


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_sweep_limit_and_long_solves(ctx, morap, prec):
    """Longer than one launch; over the limit it is NOT_CONVERGED, and the
    context goes on."""
    # (slips likelier than the move: not the grid's slots, batched sweeps)
    _compare(ctx, morap, _corridor((40,), width=41, slip=0.996), 3, prec, 1e-6, lds=False)
    wl = _corridor((5001,), width=2501, slip=0.6)
    st = _compare(ctx, morap, wl, 3, prec, 1e-6)
    assert st["max_pair_sweeps"] > 4096
    W = dirichlet_weights(np.random.default_rng(1), 3, 2)
    for limit in (7, 4100):
        with pytest.raises(morap.MorapError) as e:
            ctx.solve_staged(W, morap.Options(eps_vi=1e-6, precision=prec, max_sweeps=limit))
        assert e.value.code == morap.E_NOT_CONVERGED and f"after {limit} sweeps" in str(e.value)
    ctx.solve_staged(W, morap.Options(eps_vi=1e-6, precision=prec))
