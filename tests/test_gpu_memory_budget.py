"""What fits a device memory budget beside the batched sweeps is not refused for
the layouts in LDS order, which every call can do without: they are given up
when a later allocation of a solve, an evaluation, a staged solve or the next
upload needs their memory."""
import numpy as np
import pytest

from workloads import make_workload, tiny_workload, dirichlet_weights

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def morap():
    from paper_2305_04397_amd import morap as m
    return m


def _least_budget(morap, load):
    """The smallest budget `load` passes under: no room for any layout."""
    with morap.Context(0) as c:
        load(c)
        lo, hi = 1, c.set_memory_budget(0)
    while lo < hi:
        mid = (lo + hi) // 2
        with morap.Context(0) as c:
            c.set_memory_budget(mid)
            try:
                load(c)
                hi = mid
            except morap.MorapError as e:
                assert e.code == morap.E_OOM
                lo = mid + 1
    return hi


def _loader(morap, wl, form):
    if form == "blocks":
        return lambda c: c.build_products(wl)
    models = [morap.product_host(a, t, wl.letters[i][j]) for i, a in enumerate(wl.agents) for j, t in enumerate(wl.tasks)]
    return lambda c: c.load_models(models, wl.n_agents, wl.n_tasks)


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("form", ["blocks", "rows"])
def test_solve_and_evaluation_under_a_budget_kept(morap, form, prec):
    wl = make_workload(2, n_agents=3, n_tasks=5)
    load = _loader(morap, wl, form)
    W = dirichlet_weights(np.random.default_rng(1), 16, 8)
    o = morap.Options(eps_vi=1e-7, precision=prec)
    with morap.Context(0) as free:
        load(free)
        r1, A1, c1, s1 = free.support(W, o)
        assert s1["resident_models"] == 15
    with morap.Context(0) as lean:   # what the calls hold without the layouts
        lean.set_memory_budget(_least_budget(morap, load))
        load(lean)
        lean.set_memory_budget(0)
        c, _ = lean.solve(W, o)
        after_solve = lean.set_memory_budget(0)
        for _ in range(2):   # (the second keeps the first one's evaluation beside its own)
            r0, A0, c0, s0 = lean.support(W, o)
        after_support = lean.set_memory_budget(0)
        assert s0["resident_models"] == 0
    with morap.Context(0) as tight:
        tight.set_memory_budget(after_solve)
        load(tight)
        c2, s2 = tight.solve(W, o)
        assert np.array_equal(c2, c0) and np.array_equal(c2, c1) and np.array_equal(c, c0)
    with morap.Context(0) as tight:
        tight.set_memory_budget(after_support)
        load(tight)
        r2, A2, c2, _ = tight.support(W, o)
        assert np.array_equal(A2, A0) and np.array_equal(c2, c0)
        assert np.abs(r2 - r0).max() <= 1e-6 and np.abs(r2 - r1).max() <= 1e-6
        # and again, with whatever was given up
        r3, A3, c3, _ = tight.support(W, o)
        assert np.array_equal(c3, c0) and np.abs(r3 - r0).max() <= 1e-6
        # still refused: what does not fit either way
        tight.set_memory_budget(1)
        with pytest.raises(morap.MorapError) as e:
            tight.solve(dirichlet_weights(np.random.default_rng(1), 64, 8), o)
        assert e.value.code == morap.E_OOM and "budget" in str(e.value)
        tight.set_memory_budget(0)
        assert np.array_equal(tight.solve(W, o)[0], c0)


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_staged_solve_under_a_budget_kept(morap, prec):
    """With a fixed sweep kernel a staged solve never reads its layout in LDS
    order, at least 16 bytes a state."""
    wl = make_workload(2, n_agents=3, n_tasks=5)
    W = dirichlet_weights(np.random.default_rng(2), 16, 8)
    o = morap.Options(eps_vi=1e-7, precision=prec, schedule=28)
    with morap.Context(0) as lean:
        lean.set_memory_budget(_least_budget(morap, lambda c: c.build_products(wl)))
        lean.build_products(wl)
        lean.set_memory_budget(0)
        c0, s0 = lean.solve_staged(W, o)
        held = lean.set_memory_budget(0)
        states = sum(lean.model_info(m)["n_states"] for m in range(15))
    for schedule in (28, 0):
        with morap.Context(0) as tight:
            tight.set_memory_budget(held - 16 * states)
            tight.build_products(wl)
            c, _ = tight.solve_staged(W, morap.Options(eps_vi=1e-7, precision=prec, schedule=schedule))
            assert np.array_equal(c, c0)


def test_next_upload_under_a_budget_kept(morap):
    small, large = (_loader(morap, make_workload(2, n_agents=n, n_tasks=5), "rows") for n in (1, 4))
    budget = _least_budget(morap, large)
    with morap.Context(0) as c:
        c.set_memory_budget(budget)
        small(c)
        large(c)
        c.set_memory_budget(0)
        assert c.solve(dirichlet_weights(np.random.default_rng(1), 2, 9), morap.Options())[1]["resident_models"] == 0


def test_proposer_beside_the_layouts(morap):
    """Other allocations of the context take the layouts' memory too."""
    load = _loader(morap, make_workload(2, n_agents=3, n_tasks=5), "rows")
    with morap.Context(0) as c:
        c.proposer_init(1024, 512, seed=1)
        network = c.set_memory_budget(0)
    with morap.Context(0) as c:
        c.set_memory_budget(_least_budget(morap, load) + network)
        load(c)
        c.proposer_init(1024, 512, seed=1)


def test_team_models_hold_no_layout(morap):
    """A team model's solves are batched sweeps: beyond the same model's arrays it
    holds two objectives a row, a policy and d values a state."""
    n = 3
    team = morap.team_model_mo_host(tiny_workload(42, n, n, width=3, height=2, kinds=("reach",), k=1, p_slip=0.25))
    model = {k: v for k, v in team.items() if k != "obj"}
    S, R = len(team["state_row"]) - 1, len(team["row_ptr"]) - 1
    plain = _least_budget(morap, lambda c: c.load_models([model], 1, 1))
    with morap.Context(0) as c:
        c.load_team_model(team, n, n)
        assert c.set_memory_budget(0) <= plain + 8 * R + 4 * S + 8 * 2 * n * S + 1024


def test_short_rows_hold_memory_for_their_products_alone(morap):
    """A product of short rows beside streamed ones: 344 bytes for each of its own
    states (with what the sizes need), 3,588 a batch of the others."""
    rng = np.random.default_rng(4)

    def rows(n, per_state, entries):
        R = n * per_state
        p = rng.random((R, entries)) + 0.05
        p *= 0.95 / p.sum(1, keepdims=True)
        return {"state_row": np.arange(0, R + 1, per_state), "row_ptr": np.arange(0, R * entries + 1, entries),
                "col": rng.integers(0, n, R * entries).astype(np.int32), "prob": p.ravel(),
                "rew": np.stack([-rng.uniform(0.5, 2.0, R), rng.uniform(0, 0.05, R)], 1), "to_done": np.ones(R), "init": 0}
    models = [rows(70, 2, 3), rows(4000, 2, 4), rows(3000, 2, 4)]
    batches = (63 + 47) * (2 * (2 + 4) // 4)
    load = lambda c: c.load_models(models, 3, 1)  # noqa: E731
    with morap.Context(0) as c:
        load(c)
        W = dirichlet_weights(np.random.default_rng(1), 4, 4)
        held = c.set_memory_budget(0)
        assert c.solve(W, morap.Options())[1]["resident_models"] == 3
    layouts = held - _least_budget(morap, load)
    assert layouts <= 344 * 70 + 3588 * (batches + 1) + 4096
