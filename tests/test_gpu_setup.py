"""Setup kernels at the edges of their blocks: staged rows (64 rows and 32
columns at a time) and K' of FP64 plans (32-row bands, 16 features at a time),
through K' entries against the FP64 oracle, and wide FP32 scoring (an exact row
length per kernel) against the oracle's decision function.

Tolerances: 1e-12 for FP64 K' (one chain of m squared differences and one
exponential), 2e-6 for FP32 and three-term K' (as elsewhere), 1e-5 of sum
|alpha| for scores.
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


@pytest.mark.parametrize("m", [1, 15, 16, 17, 31, 32, 33, 64, 65, 100])
@pytest.mark.parametrize("prec,tol", [("fp64", 1e-12), ("fp32", 2e-6), ("mixed", 2e-6)])
def test_kernel_entries(torch, prec, tol, m):
    n = 289 + 64                                  # a ragged second block
    X, y = inputs.linear_teacher(n, m, 17)
    gamma = 0.5 / m
    print(f"[case] setup {prec} m={m}", flush=True)
    s = gabp.GabpSVM(gamma=gamma, C=1.0, precision=prec, max_sweeps=1)
    s.solve(torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda())
    K = R.rbf_augmented_kernel(X, gamma, 1.0 / n)
    rng = np.random.default_rng(5)
    rows = np.concatenate([np.arange(0, 288), rng.integers(0, n, 400)])
    cols = np.concatenate([np.arange(1, 289), rng.integers(0, n, 400)])
    off = rows != cols
    got = s.kernel_entries(rows[off], cols[off])
    assert np.max(np.abs(got - K[rows[off], cols[off]])) <= tol
    s.close()


@pytest.mark.parametrize("m", [63, 64, 65, 80, 96, 97, 112, 128, 129, 150])
def test_wide_scores(torch, m):
    n = 1500
    X, y, Xq, _ = inputs.linear_teacher(n, m, 19, n_test=300)
    print(f"[case] wide scores m={m}", flush=True)
    s = gabp.GabpSVM(gamma=1.0 / m, C=1.0, precision="fp32", tol_rel=1e-6)
    s.solve(torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda())
    alpha = s.alpha()
    ref = R.decision_function(X, y, alpha, Xq, 1.0 / m, 1.0 / n)
    f = s.predict(torch.from_numpy(Xq).cuda()).cpu().numpy()
    assert np.max(np.abs(f - ref)) <= 1e-5 * float(np.abs(alpha).sum())
    s.close()
