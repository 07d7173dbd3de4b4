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
