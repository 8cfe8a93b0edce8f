"""Sparse sweeps where the system is far from order one: a large augmentation
(every kept entry about lambda^2) and a large diagonal (small C).

Tolerance against the FP64 oracle's sweeps: 1e-5 (inf-norm, relative), as for
the other sparse tests; the points lie close together, so the Gram's rounding
adds nothing.
"""
import numpy as np
import pytest

from oracle import gabp_ref as R
from paper_0810_1648_amd import gabp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    return _t


# (lambda, C): lambda^2 = 2^44 passes FP32 in products of three such factors;
# 1/C = 1e200 passes FP64 in products of two (its diagonal is not FP32's)
@pytest.mark.parametrize("prec,lam,C", [("fp32", 2.0 ** 22, 1.0), ("mixed", 2.0 ** 22, 1.0), ("mixed", 0.1, 1e-200),
                                        ("fp32", 2.0 ** 29, 1.0)])
def test_systems_far_from_order_one(torch, prec, lam, C):
    rng = np.random.default_rng(7)
    n, gamma, tau = 400, 0.5, 0.3
    X = (0.05 * rng.standard_normal((n, 6))).astype(np.float32)
    X[n // 2:] += 3.0                                   # two groups that keep no pair with each other
    y = np.where(rng.random(n) < 0.5, 1.0, -1.0).astype(np.float32)
    A, b = R.sparse_svm_system(X, y, gamma, C, lam, tau)
    ref = R.gabp_solve(A, b, max_sweeps=5, tol_rel=0.0, keep_trajectory=True).trajectory
    Xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    for t in (1, 2, 3, 5):
        print(f"[case] sparse range {prec} lambda={lam} C={C} t={t}", flush=True)
        s = gabp.GabpSVM(kernel="rbf_sparse", sparse_tau=tau, gamma=gamma, C=C, lambda_aug=lam, precision=prec,
                         max_sweeps=t, tol_abs=0.0, tol_rel=0.0, stagnation_window=0)
        st = s.solve(Xd, yd)
        assert st in (gabp.OK, gabp.E_NOT_CONVERGED) and s.plan()["n_edges"] == 2 * (n // 2) * (n // 2 - 1) // 2
        want = ref[min(s.sweeps(), len(ref) - 1)]       # (1 / C = 1e200: no change after the first sweep)
        assert float(np.max(np.abs(s.alpha() - want)) / np.max(np.abs(want))) <= 1e-5
        s.close()
