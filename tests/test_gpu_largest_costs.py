"""Costs so large that values can overflow keep the batched sweeps, whose maxima
pass over a NaN and start at minus infinity: solves are the fixed schedule's, bit
for bit, in every form a problem is given; the largest costs below stay in LDS."""
import dataclasses

import numpy as np
import pytest

from workloads import make_workload, dirichlet_weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,scale,lds", [("f32", 1e37, False), ("f32", 1e28, True), ("f64", 1e306, False),
                                            ("f64", 1e297, True)])
@pytest.mark.parametrize("form", ["blocks", "rows", "staged"])
def test_values_that_overflow(form, prec, scale, lds):
    from paper_2305_04397_amd import morap
    wl = make_workload(2, n_agents=3, n_tasks=4)
    wl = dataclasses.replace(wl, agents=[dataclasses.replace(a, cost=a.cost * scale) for a in wl.agents])
    W = dirichlet_weights(np.random.default_rng(1), 16, 7)
    W[0] = np.eye(7)[3]
    with morap.Context(0) as ctx:
        if form == "rows":
            ctx.load_models([morap.product_host(a, t, wl.letters[i][j]) for i, a in enumerate(wl.agents)
                             for j, t in enumerate(wl.tasks)], 3, 4)
        else:
            ctx.build_products(wl)
        solve = ctx.solve_staged if form == "staged" else ctx.solve
        runs = []
        for schedule in (0, 10 if form == "rows" else 28):
            c, st = solve(W, morap.Options(eps_vi=scale * 1e-7, precision=prec, schedule=schedule))
            runs.append((c, st, [ctx.get_values(k, m) for k in (0, 5, 15) for m in range(12)]))
        (c1, s1, x1), (c0, s0, x0) = runs
        assert s1["resident_models"] == (12 if lds else 0) and s0["resident_models"] == 0
        assert np.array_equal(c1, c0, equal_nan=True)
        assert all(np.array_equal(a, b, equal_nan=True) for a, b in zip(x1, x0))
        for f in ("backups", "sweeps", "max_pair_sweeps", "floor_stops"):
            assert s1[f] == s0[f], f
        if lds:
            assert np.isfinite(c1).all()
