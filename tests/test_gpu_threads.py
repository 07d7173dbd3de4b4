"""Contexts used from several host threads at once, each with its own streams
and host threads: every one gives what it gives alone, and a context used again
after an error goes on."""
import threading

import numpy as np
import pytest

from workloads import make_workload, dirichlet_weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 5])
def test_contexts_side_by_side(n):
    from paper_2305_04397_amd import morap
    wl = make_workload(2, n_agents=4, n_tasks=7)
    o = morap.Options(eps_vi=1e-6, precision="f32")
    W = [dirichlet_weights(np.random.default_rng(i), 17, 11) for i in range(n)]
    with morap.Context(0) as c:
        c.build_products(wl)
        alone = [c.support(w, o)[:3] for w in W]
    got, errors = [None] * n, []

    def work(i):
        try:
            with morap.Context(0) as c:
                c.build_products(wl)
                with pytest.raises(morap.MorapError):
                    c.support(W[i], morap.Options(eps_vi=1e-6, precision="f32", max_sweeps=4))
                for _ in range(3):
                    got[i] = c.support(W[i], o)[:3]
                    c.query_batch(got[i][0][:5] - 0.01, eps=0.01, max_iter=3, opts=o)
        except BaseException as e:   # noqa: BLE001 (reported by the main thread)
            errors.append(e)

    threads = [threading.Thread(target=work, args=(i,)) for i in range(n)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for i in range(n):
        for a, b in zip(alone[i], got[i]):
            assert np.array_equal(a, b), i
