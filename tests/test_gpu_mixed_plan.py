"""Solves whose products in LDS and products of the batched sweeps alternate by
size: costs that differ between states keep a product out of the larger kernels,
so such products of 2,100 to 3,300 states lie between sorted ones and small ones."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

SCRIPT = """
import dataclasses
import numpy as np
from paper_2305_04397_amd import morap
from workloads import make_workload, dirichlet_weights
from workloads.gridworld import make_agent

prec, K = sys.argv[1], int(sys.argv[2])
rng = np.random.default_rng(1)
agents, letters = [], []
for n, per_state in ((9700, 0), (300, 0), (5000, 0), (400, 1), (50, 1)) + tuple((2100 + 200 * i, 1) for i in range(7)):
    free = np.zeros((-(-(n + 1) // 80), 80), bool)
    free.ravel()[:n + 1] = True
    a = make_agent(rng, free, 0, 0.1, rng.uniform(1.0, 3.0, 5))
    if per_state:
        a = dataclasses.replace(a, cost=rng.uniform(1.0, 3.0, a.cost.size))
    lab = np.zeros(a.n_states, np.int32)
    lab[-1] = 1
    agents.append(a)
    letters.append([lab])
base = make_workload(1)
task = dataclasses.replace(base.tasks[0], kind="reach", k=1, n_locs=2, n_letters=2, q0=0,
                           delta=np.array([[0, 1], [1, 1]], np.int32), accepting=np.array([0, 1], np.uint8),
                           waypoints_uv=np.zeros((0, 2, 2)), avoid_uv=None)
wl = dataclasses.replace(base, agents=agents, tasks=[task], letters=letters)
n = len(agents)
W = dirichlet_weights(np.random.default_rng(K), K, n + 1)
with morap.Context(0) as ctx:
    ctx.build_products(wl)
    c1, s1 = ctx.solve(W, morap.Options(eps_vi=1e-6, precision=prec))
    x1 = [ctx.get_values(k, m) for m in range(n) for k in (0, K - 1)]
    c0, s0 = ctx.solve(W, morap.Options(eps_vi=1e-6, precision=prec, schedule={64: 37, 4: 22}[K]))
    assert s1["resident_models"] == 5 and s0["resident_models"] == 0
    assert np.array_equal(c1, c0)
    for f in ("backups", "sweeps", "max_pair_sweeps", "floor_stops"):
        assert s1[f] == s0[f], f
    for x, (m, k) in zip(x1, ((m, k) for m in range(n) for k in (0, K - 1))):
        assert np.array_equal(x, ctx.get_values(k, m)), (k, m)
print("same")
"""


@pytest.mark.parametrize("prec,K", [("f32", 64), ("f64", 64), ("f32", 4), ("f64", 4)])
def test_batched_products_between_products_in_lds(root, prec, K):
    """In a process of its own whose freed and fresh host memory is filled with a
    pattern: an index past the plan's models reads it and ends there."""
    env = dict(os.environ, MALLOC_PERTURB_="165")
    r = subprocess.run([sys.executable, "-c", "import sys; sys.path.insert(0, sys.argv.pop())\n" + SCRIPT, prec, str(K), root],
                       cwd=root, env=env, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "same" in r.stdout, (r.returncode, r.stdout[-500:], r.stderr[-1500:])


def _corridors(sizes):
    """One agent per size on 200-wide grids, one reach task: products of exactly
    that many states."""
    import dataclasses
    import numpy as np
    from workloads import make_workload
    from workloads.gridworld import make_agent
    rng = np.random.default_rng(len(sizes))
    agents, letters = [], []
    for n in sizes:
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
    return dataclasses.replace(base, agents=agents, tasks=[task], letters=letters)


@pytest.mark.parametrize("sizes,variant", [((45000, 3000, 3000), 40), ((45000,) + (9000,) * 11, 37)])
def test_sweep_kernel_of_the_products_beyond_lds(sizes, variant):
    """FP32 products beyond LDS take the LDS-staged sweep where they hold more than
    a third of the states, else the gather sweep; the same values either way."""
    import numpy as np
    from paper_2305_04397_amd import morap
    from workloads import dirichlet_weights
    n = len(sizes)
    W = dirichlet_weights(np.random.default_rng(3), 64, n + 1)
    with morap.Context(0) as ctx:
        ctx.build_products(_corridors(sizes))
        c1, s1 = ctx.solve(W, morap.Options(eps_vi=1e-6, precision="f32"))
        assert s1["resident_models"] == n - 1 and s1["variant"] == variant
        x1 = [ctx.get_values(k, 0) for k in (0, 63)]
        c0, s0 = ctx.solve(W, morap.Options(eps_vi=1e-6, precision="f32", schedule=37))
        assert np.array_equal(c1, c0) and s1["backups"] == s0["backups"] and s1["sweeps"] == s0["sweeps"]
        assert all(np.array_equal(x, ctx.get_values(k, 0)) for x, k in zip(x1, (0, 63)))


def test_staged_solve_takes_the_sweep_its_plain_solve_was_timed_for():
    """A staged solve after a plain one whose sweep kernel was timed on the
    products beyond LDS takes that kernel (FP64, 16 columns)."""
    import numpy as np
    from paper_2305_04397_amd import morap
    from workloads import dirichlet_weights
    W = dirichlet_weights(np.random.default_rng(3), 16, 4)
    o = morap.Options(eps_vi=1e-6, precision="f64")
    with morap.Context(0) as ctx:
        ctx.build_products(_corridors((45000, 30000, 3000)))
        c0, s0 = ctx.solve(W, o)
        assert s0["resident_models"] == 1 and 18 < s0["variant"] <= 38
        c1, s1 = ctx.solve_staged(W, o)
        assert s1["variant"] == s0["variant"]
        assert np.abs(c1 - c0).max() <= 1e-4
