"""Sweeps whose tiles are split into row parts (few tiles) against the FP64
oracle, at the sizes where the number of parts changes: up to 127 tiles (15
blocks) eight parts, 255 (22 blocks) four, 511 (31 blocks) two, then one.

Tolerances: 1e-12 relative (inf-norm) in FP64, whose only differences are the
rounding of sums of at most N terms; 1e-5 in FP32 and MIXED, as everywhere.
"""
import numpy as np
import pytest

from oracle import gabp_ref as R
from paper_0810_1648_amd import gabp, inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    return _t


@pytest.mark.parametrize("n", [257, 3840, 3841, 5633, 7937])
def test_row_parts_match_oracle(torch, n):
    wl = inputs.make_workload("covertype", n=n, seed=61)
    A, b = R.svm_system(wl.X, wl.y, wl.gamma, wl.C, wl.lam)
    ref = R.gabp_solve(A, b, max_sweeps=2, tol_rel=0.0, keep_trajectory=True).trajectory[2]
    # the library's groups: 256-point block I belongs to group I G / NB
    gid = np.arange(n) // 256 * 2 // ((n + 255) // 256)
    groups = [np.nonzero(gid == g)[0] for g in range(2)]
    refg = R.gabp_solve_grouped(A, b, groups, max_sweeps=2, tol_rel=0.0, keep_trajectory=True).trajectory[2]
    X, y = torch.from_numpy(wl.X).cuda(), torch.from_numpy(wl.y).cuda()
    for prec, edge, sched in (("fp64", "stored", "sync"), ("fp64", "stateless", "sync"), ("fp32", "stateless", "sync"),
                              ("mixed", "stateless", "sync"), ("mixed", "stored", "sync"),
                              ("fp64", "stored", "grouped"), ("fp32", "stateless", "grouped"),
                              ("mixed", "stateless", "grouped")):
        kw = dict(sched_groups=2) if sched == "grouped" else {}
        print(f"[case] split n={n} {prec} {edge} {sched}", flush=True)
        s = gabp.GabpSVM(gamma=wl.gamma, C=wl.C, lambda_aug=wl.lam, precision=prec, edge_state=edge, schedule=sched,
                         kstore="materialise", max_sweeps=2, tol_abs=0.0, tol_rel=0.0, stagnation_window=0, **kw)
        s.solve(X, y)
        assert s.sweeps() == 2
        want = refg if sched == "grouped" else ref
        err = float(np.max(np.abs(s.alpha() - want)) / np.max(np.abs(want)))
        assert err <= (1e-12 if prec == "fp64" else 1e-5), (n, prec, edge, sched, err)
        s.close()
