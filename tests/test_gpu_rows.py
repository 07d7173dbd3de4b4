"""Value iteration of products given as rows of entries with the values in LDS
(the solver's own choice when every product fits a workgroup) against the
batched CSR sweep (a fixed schedule): the same bits in every value, the same
stopping sweeps, at the edges of slices, batches, rows, column groups and
launches."""
import numpy as np
import pytest

from workloads import make_workload, tiny_workload, dirichlet_weights

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


def _random_model(rng, n, max_rows, max_entries, leave=0.05, init=0, uneven=True):
    """Rows of 0 .. max_entries entries over any states, 1 .. max_rows a state
    (or exactly that many); what a row lacks of probability 1 leaves."""
    state_row, row_ptr, col, prob, rew, done = [0], [0], [], [], [], []
    for s in range(n):
        for _ in range(rng.integers(1, max_rows + 1) if uneven else max_rows):
            k = int(rng.integers(0, max_entries + 1)) if uneven else max_entries
            p = rng.dirichlet(np.ones(k)) * (1 - leave) if k else np.zeros(0)
            col.extend(rng.integers(0, n, k))
            prob.extend(p)
            row_ptr.append(len(col))
            rew.append((-rng.uniform(0.5, 2.0), rng.uniform(0, 1 - p.sum())))
            done.append(1)
        state_row.append(len(row_ptr) - 1)
    return {"state_row": np.array(state_row), "row_ptr": np.array(row_ptr), "col": np.array(col, np.int32),
            "prob": np.array(prob), "rew": np.array(rew), "to_done": np.array(done), "init": init}


def _compare(ctx, morap, models, nI, nJ, K, prec, eps=1e-6, lds=True, **kw):
    ctx.load_models(models, nI, nJ)
    W = dirichlet_weights(np.random.default_rng(K), K, nI + nJ)
    W[0] = np.eye(nI + nJ)[nI]        # a probability alone: every cost weight is 0
    c1, s1 = ctx.solve(W, morap.Options(eps_vi=eps, precision=prec, **kw))
    cols = sorted({0, K // 2, K - 1})
    x1 = {(k, m): ctx.get_values(k, m) for m in range(nI * nJ) for k in cols}
    Kp = 1
    while Kp < K:
        Kp *= 2
    v = {1: 1, 2: 2, 4: 4, 8: 7, 16: 10, 32: 13}.get(Kp, 16)
    c0, s0 = ctx.solve(W, morap.Options(eps_vi=eps, precision=prec, schedule=v, **kw))
    assert s0["resident_models"] == 0 and s0["variant"] == v
    assert (s1["resident_models"] > 0) == lds and s1["variant"] <= 18
    assert np.array_equal(c1, c0)
    for f in ("backups", "sweeps", "max_pair_sweeps", "floor_stops"):
        assert s1[f] == s0[f], f
    assert s1["bytes"] == pytest.approx(s0["bytes"], rel=1e-12)
    for (k, m), x in x1.items():
        assert np.array_equal(x, ctx.get_values(k, m)), (k, m)
    return s1


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("K", [1, 3, 40, 70])
def test_grid_products(ctx, morap, prec, K):
    wl = make_workload(2, n_agents=3, n_tasks=5)
    models = [morap.product_host(a, t, wl.letters[i][j]) for i, a in enumerate(wl.agents)
              for j, t in enumerate(wl.tasks)]
    _compare(ctx, morap, models, 3, 5, K, prec)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("rows,entries", [(1, 1), (3, 4), (5, 7)])
def test_irregular_rows_and_slices(ctx, morap, prec, rows, entries):
    """Rows without entries, states of one row beside states of many, one state
    to many slices, an initial state that is not the first."""
    rng = np.random.default_rng(rows)
    models = [_random_model(rng, n, rows, entries, init=n // 2) for n in (1, 63, 64, 65, 300, 1100)]
    _compare(ctx, morap, models, 6, 1, 20, prec)
    _compare(ctx, morap, models, 2, 3, 2, prec)


def _short_rows(rng, n, rows, leave=0.05):
    """At most `rows` rows a state of at most three entries."""
    state_row, row_ptr, col, prob, rw = [0], [0], [], [], []
    for s in range(n):
        own = np.unique(rng.integers(0, n, 5))
        for _ in range(int(rng.integers(1, rows + 1))):
            k = rng.choice(own, size=min(len(own), int(rng.integers(0, 4))), replace=False)
            p = rng.dirichlet(np.ones(len(k))) * (1 - leave) if len(k) else np.zeros(0)
            col.extend(k)
            prob.extend(p)
            row_ptr.append(len(col))
            rw.append((-rng.uniform(0.5, 2.0), rng.uniform(0, 1 - p.sum())))
        state_row.append(len(row_ptr) - 1)
    return {"state_row": np.array(state_row), "row_ptr": np.array(row_ptr), "col": np.array(col, np.int32),
            "prob": np.array(prob), "rew": np.array(rw), "to_done": np.ones(len(rw)), "init": n // 3}


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("sizes", [(1, 64, 511, 512), (513, 1024), (1025, 1536), (1537, 2048, 2049)])
@pytest.mark.parametrize("K", [1, 5, 64])
def test_short_rows(ctx, morap, prec, sizes, K):
    """At most five rows of three entries: in registers up to 2,048 (FP64:
    1,024) states, streamed above, side by side with products of six rows a
    state and of four entries a row."""
    rng = np.random.default_rng(sizes[0])
    models = [_short_rows(rng, n, 5) for n in sizes]
    models += [_short_rows(rng, 100, 6), _random_model(rng, 80, 3, 4), _short_rows(rng, 70, 1)]
    _compare(ctx, morap, models, len(models), 1, K, prec)


@pytest.mark.parametrize("prec,K", [("f32", 64), ("f64", 64), ("f32", 1), ("f64", 1)])
def test_sizes_at_the_edges_of_the_column_groups(ctx, morap, prec, K):
    rng = np.random.default_rng(5)
    models = [_random_model(rng, n, 2, 3, uneven=False) for n in (256, 257, 512, 513, 4990, 5200, 9700, 10100)]
    _compare(ctx, morap, models, 8, 1, K, prec, lds=prec == "f32")   # FP64: up to 9,664 states
    _compare(ctx, morap, models[:6], 6, 1, K, prec)


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_what_stays_with_the_batched_sweeps(ctx, morap, prec):
    """A product beyond LDS; one whose lanes' rows differ too much; models
    without states to solve for beside others."""
    rng = np.random.default_rng(6)
    small = _random_model(rng, 200, 2, 3)
    big = _random_model(rng, 21000, 1, 2)
    _compare(ctx, morap, [small, big], 2, 1, 8, prec, lds=False)
    lone = _random_model(rng, 64, 1, 1)
    wide = _random_model(rng, 1, 30, 40, uneven=False)   # a state of 30 rows among 64 of one
    for f in ("col", "prob", "rew", "to_done"):
        lone[f] = np.concatenate([lone[f], wide[f]])
    lone["state_row"] = np.concatenate([lone["state_row"], lone["state_row"][-1] + wide["state_row"][1:]])
    lone["row_ptr"] = np.concatenate([lone["row_ptr"], lone["row_ptr"][-1] + wide["row_ptr"][1:]])
    _compare(ctx, morap, [small, lone], 2, 1, 8, prec, lds=False)
    empty = {"state_row": np.zeros(1), "row_ptr": np.zeros(1), "col": np.zeros(0), "prob": np.zeros(0),
             "rew": np.zeros((0, 2)), "to_done": np.zeros(0), "init": -1}
    done = _random_model(rng, 100, 2, 3, init=-1)
    _compare(ctx, morap, [small, done, empty, small], 2, 2, 8, prec)


def test_sweep_limit_and_long_solves(ctx, morap):
    n = 6
    nxt = np.minimum(np.arange(n) + 1, n - 1)
    chain = {"state_row": np.arange(n + 1), "row_ptr": np.arange(0, 2 * n + 1, 2),
             "col": np.stack([np.arange(n), nxt], 1).ravel(), "prob": np.tile([0.9995, 0.0005], n),
             "rew": np.tile([-1.0, 0.0], (n, 1)), "to_done": np.zeros(n), "init": 0}
    chain["prob"][-1] = 0.0
    chain["to_done"][-1] = 1
    st = _compare(ctx, morap, [chain], 1, 1, 4, "f64", eps=1e-9)
    assert st["max_pair_sweeps"] > 2 * 4096
    W = dirichlet_weights(np.random.default_rng(1), 4, 2)
    for limit in (10, 5000):
        with pytest.raises(morap.MorapError) as e:
            ctx.solve(W, morap.Options(eps_vi=1e-9, precision="f64", max_sweeps=limit))
        assert e.value.code == morap.E_NOT_CONVERGED and "column" in str(e.value)
    ctx.solve(W, morap.Options(eps_vi=1e-9, precision="f64"))


def test_no_memory_for_the_layout(ctx, morap):
    """Where a memory budget leaves no room for the layout in LDS order, the
    products load and solve as before it."""
    wl = tiny_workload(3, 2, 2, width=6, height=5)
    models = [morap.product_host(a, t, wl.letters[i][j]) for i, a in enumerate(wl.agents)
              for j, t in enumerate(wl.tasks)]
    W = dirichlet_weights(np.random.default_rng(1), 8, 4)
    o = morap.Options(eps_vi=1e-7, precision="f64")
    ctx.load_models(models, 2, 2)
    c1, s1 = ctx.solve(W, o)
    assert s1["resident_models"] == 4
    held = ctx.set_memory_budget(0)
    lo, hi = 1, held
    while lo < hi:                    # the smallest budget the products load under
        mid = (lo + hi) // 2
        with morap.Context(0) as probe:
            probe.set_memory_budget(mid)
            try:
                probe.load_models(models, 2, 2)
                hi = mid
            except morap.MorapError as e:
                assert e.code == morap.E_OOM
                lo = mid + 1
    with morap.Context(0) as d:
        d.set_memory_budget(hi)
        d.load_models(models, 2, 2)
        d.set_memory_budget(0)
        c0, s0 = d.solve(W, o)
        assert s0["resident_models"] == 0 and np.array_equal(c0, c1)
