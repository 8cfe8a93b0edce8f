"""Sparse sweeps by rows, at the sizes where rows meet the workgroup ranges
(256 quads of four entries): rows of one quad, of isolated points, of exactly
the range's length, and rows that cross two or three ranges.

Tolerance (inf-norm, relative) against the FP64 oracle's sweeps: 1e-5 as for
the other sparse tests, plus what the Gram's own rounding puts into K' of the
points far from the mean, which the sweeps do not touch: gamma times the
rounding of d^2 = n_i + n_j - 2 g, m + 3 operations on values up to
4 max |x|^2 at 2^-24 each.
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


# dense: points of one cluster, all pairs kept (rows of dense - 1 entries);
# alone: isolated points; pairs: couples that keep only each other
@pytest.mark.parametrize("dense,alone,pairs", [(0, 5, 0), (1025, 0, 0), (1026, 300, 3), (2300, 1, 40), (4, 1023, 1)])
@pytest.mark.parametrize("prec", ["fp32", "mixed"])
def test_rows_match_oracle(torch, prec, dense, alone, pairs):
    rng = np.random.default_rng(91)
    X = [0.05 * rng.standard_normal((dense, 6))]
    # the others on a grid of spacing 3 around it (the cut is at distance
    # 1.55), the couples nearest: their K' keeps the precision of the Gram,
    # which loses digits with the distance from the mean
    grid = 3.0 * (np.indices((5,) * 6).reshape(6, -1).T - 2)
    grid = grid[np.argsort((grid ** 2).sum(axis=1), kind="stable")][1:alone + pairs + 1]
    far = np.concatenate([grid[pairs:], grid[:pairs]])
    X.append(far[:alone])
    X.append(far[alone:])
    X.append(far[alone:] + 0.1)
    X = np.concatenate(X).astype(np.float32)
    n = len(X)
    X = X[rng.permutation(n)]
    y = np.where(rng.random(n) < 0.5, 1.0, -1.0).astype(np.float32)
    gamma, tau, C, lam = 0.5, 0.3, 10.0, 1.0 / n
    A, b = R.sparse_svm_system(X, y, gamma, C, lam, tau)
    ref = R.gabp_solve(A, b, max_sweeps=5, tol_rel=0.0, keep_trajectory=True).trajectory
    kept = np.unique(R.sparse_edges(X, gamma, tau)) if dense + pairs else np.zeros(0, int)
    r2 = float((((X - X.mean(axis=0)) ** 2).sum(axis=1))[kept].max()) if len(kept) else 0.0
    tol = 1e-5 + gamma * (6 + 3) * 4.0 * r2 * 2.0 ** -24
    Xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    for t in (1, 2, 3, 5):
        print(f"[case] sparse rows {prec} {dense}/{alone}/{pairs} t={t}", flush=True)
        s = gabp.GabpSVM(kernel="rbf_sparse", sparse_tau=tau, gamma=gamma, C=C, lambda_aug=lam, precision=prec,
                         max_sweeps=t, tol_abs=0.0, tol_rel=0.0, stagnation_window=0)
        s.solve(Xd, yd)
        assert s.plan()["n_edges"] == dense * (dense - 1) // 2 + pairs
        if s.sweeps() == t:              # (a graph without edges stops at once: no change)
            err = float(np.max(np.abs(s.alpha() - ref[t])) / np.max(np.abs(ref[t])))
            assert err <= tol, (prec, dense, alone, pairs, t, err)
        else:
            assert dense < 2 and pairs == 0 and s.sweeps() == 1
        s.close()
