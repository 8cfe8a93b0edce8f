"""Row parts per tile and the rings between two writes of the stored records
are taken only where the memory has room for them: a solve needs no more than
with one partial sum per tile and records written in every sweep.

The budgets and arenas below are the smallest of that plan, to the byte
(planes of 256 x 256 tiles, NB (NB + 1) partial sums of 256 doubles twice,
features and per-node vectors); `held` is what its solve then held.  Alpha:
1e-12 (FP64) and 1e-5 (else) of the solve without a limit, as everywhere; held
bytes: within 2 KiB (the maxima of 64 instead of 256 nodes).
"""
import numpy as np
import pytest

from paper_0810_1648_amd import gabp, inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    return _t


def close(a, b, prec):
    assert float(np.max(np.abs(a - b)) / np.max(np.abs(b))) <= (1e-12 if prec == "fp64" else 1e-5)


@pytest.mark.parametrize("n,budget,held,kw", [
    (500, 8314804, 8296072, dict(precision="fp64", edge_state="stored")),
    (1500, 29359036, 29311336, dict(precision="mixed", edge_state="stored", kstore="materialise")),
    (3001, 3909400, 4013240, dict(precision="fp32", edge_state="stateless", stateless_depth=5)),
    (3001, 4302616, 5782712, dict(precision="mixed", edge_state="stateless", stateless_depth=3, kstore="recompute")),
    (5000, 7823312, 10294428, dict(precision="mixed", schedule="grouped", sched_groups=4, edge_state="stateless",
                                   stateless_depth=3)),
    (2000, 49433048, 49371072, dict(precision="fp32", schedule="grouped", sched_groups=4, edge_state="stored",
                                    kstore="materialise"))])
def test_smallest_budgets(torch, n, budget, held, kw):
    wl = inputs.make_workload("covertype", n=n, seed=3)
    alpha = {}
    for b in (0, budget):
        s = gabp.GabpSVM(gamma=wl.gamma, C=wl.C, max_sweeps=3, hbm_budget_bytes=b, **kw)
        s.solve(wl.X, wl.y)
        alpha[b] = s.alpha()
        if b:
            assert s.plan()["device_bytes"] <= max(held + 2048, budget)
        s.close()
    # (a plan that recomputes K' under the budget may hold it without)
    close(alpha[budget], alpha[0], kw["precision"])
    s = gabp.GabpSVM(gamma=wl.gamma, C=wl.C, max_sweeps=3, hbm_budget_bytes=budget - 1, **kw)
    with pytest.raises(gabp.GabpError) as e:
        s.solve(wl.X, wl.y)
    assert e.value.status == gabp.E_NOMEM
    s.close()


@pytest.mark.parametrize("n,arena,kw", [(500, 8351232, dict(precision="fp64")),
                                        (1500, 28882176, dict(precision="mixed", edge_state="stored")),
                                        (3001, 104850176, dict(precision="fp32", schedule="grouped", sched_groups=4))])
def test_smallest_arenas(torch, n, arena, kw):
    wl = inputs.make_workload("covertype", n=n, seed=3)
    kw = dict(kw, gamma=wl.gamma, C=wl.C, max_sweeps=3)
    s = gabp.GabpSVM(kstore="materialise", **kw)
    s.solve(wl.X, wl.y)
    want = s.alpha()
    s.close()
    with gabp.GabpServer(arena_bytes=arena) as srv:
        t = srv.submit(wl.X, wl.y, **kw)
        assert srv.wait(t, 60.0)
        close(srv.result(t)[0], want, kw["precision"])
    with gabp.GabpServer(arena_bytes=arena - 256) as srv, pytest.raises(gabp.GabpError) as e:
        srv.submit(wl.X, wl.y, **kw)
    assert e.value.status == gabp.E_NOMEM
