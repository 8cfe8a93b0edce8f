"""The locality order of a sparsified solve (nearest of five landmarks: one
group of four and one more) at the row lengths where the number of features
held in registers changes, and beyond the longest.

Points with whole-number coordinates, so that the cut between two values of
d^2 decides every pair exactly; the kept pairs are counted in whole numbers,
and the order must not show: a permutation of the input permutes alpha.

Tolerance of that comparison (inf-norm, relative): 1e-5 for either side, as
for the other sparse tests, plus what the Gram's rounding puts into K', gamma
times m + 3 operations on values up to 4 max |x|^2 at 2^-24 each.
"""
import numpy as np
import pytest

from paper_0810_1648_amd import gabp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    return _t


@pytest.mark.parametrize("m", [3, 8, 9, 16, 17, 24, 25, 32, 33, 64, 65])
def test_order_does_not_show(torch, m):
    rng = np.random.default_rng(17)
    n = 10300
    X = rng.integers(0, 7 if m < 8 else 3, (n, m)).astype(np.float32)
    y = np.where(rng.random(n) < 0.5, 1.0, -1.0).astype(np.float32)
    g = X.astype(np.float64)
    nrm = (g ** 2).sum(axis=1)
    hist = np.zeros(int(4 * nrm.max()) + 2, dtype=np.int64)
    for i in range(0, n, 1000):
        d2 = nrm[i:i + 1000, None] + nrm[None, :] - 2.0 * (g[i:i + 1000] @ g.T)
        hist += np.bincount(d2.astype(np.int64).ravel(), minlength=len(hist))
    hist[0] -= n                              # (each point and itself)
    cum = np.cumsum(hist) // 2
    cut = int(np.searchsorted(cum, 10 * n))   # about twenty neighbours a point
    gamma = 1.0 / m
    tau = float(np.exp(-gamma * (cut + 0.5)))
    r2 = float(((g - g.mean(axis=0)) ** 2).sum(axis=1).max())
    tol = 2.0 * (1e-5 + gamma * (m + 3) * 4.0 * r2 * 2.0 ** -24)
    perm = rng.permutation(n)
    alpha = []
    for idx in (np.arange(n), perm):
        print(f"[case] sparse order m={m}", flush=True)
        s = gabp.GabpSVM(kernel="rbf_sparse", sparse_tau=tau, gamma=gamma, C=1.0, lambda_aug=1.0 / n,
                         precision="fp32", max_sweeps=4, tol_abs=0.0, tol_rel=0.0, stagnation_window=0)
        s.solve(torch.from_numpy(X[idx]).cuda(), torch.from_numpy(y[idx]).cuda())
        assert s.plan()["n_edges"] == cum[cut]
        alpha.append(np.asarray(s.alpha()))
        s.close()
    assert np.all(alpha[0] != 0.0)
    err = float(np.max(np.abs(alpha[1] - alpha[0][perm])) / np.max(np.abs(alpha[0])))
    assert err <= tol, (m, err, tol)
