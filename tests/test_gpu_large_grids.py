"""Dense sweeps over more tiles than one launch holds threads for (1.48 M points,
K' recomputed).

With gamma -> 0 and lambda = 0 every K'_ij is 1, A_ii = 1.1 (N - 1), and the first
sweep has a closed form: P~ = A - (N - 1) / A, S_j = y_j - (sum_i y_i - y_j) / A.
Tolerance: 1e-5 relative (inf-norm) as everywhere; without the last tiles S is
off by their share of the labels' sum, 1e-2 and more.
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


@pytest.mark.parametrize("depth,schedule", [(2, "sync"), (3, "sync"), (2, "grouped")])
def test_closed_form_of_1490000_points(torch, depth, schedule):
    n, m = 1_490_000, 20
    if torch.cuda.mem_get_info()[0] < 180 << 30:
        pytest.skip("needs 180 GiB of device memory")
    rng = np.random.default_rng(depth)
    X = torch.from_numpy(rng.standard_normal((n, m), dtype=np.float32)).cuda()
    y = np.where(rng.random(n) < 0.75, 1.0, -1.0).astype(np.float32)
    s = gabp.GabpSVM(gamma=1e-12, C=1.0, lambda_aug=0.0, precision="mixed", kstore="recompute", edge_state="stateless",
                     stateless_depth=depth, schedule=schedule, sched_groups=1, max_sweeps=1, tol_abs=0.0, tol_rel=0.0,
                     stagnation_window=0)
    s.solve(X, torch.from_numpy(y).cuda())
    p = s.plan()
    assert p["n_tiles"] > 1 << 24 and s.sweeps() == 1
    A = 1.1 * (n - 1)
    assert np.max(np.abs(s.adiag() - A)) <= 1e-6 * A
    want = (y - (y.sum(dtype=np.float64) - y) / A) * y / (A - (n - 1) / A)
    assert float(np.max(np.abs(s.alpha() - want)) / np.max(np.abs(want))) <= 1e-5
    if schedule == "sync" and depth == 3:
        # (1 - A alpha in the same closed form: every tile once more)
        al = s.alpha()
        r = 1.0 - y * (A * y * al + ((y * al).sum() - y * al))
        assert abs(s.residual_bound()["residual_inf"] - np.max(np.abs(r))) <= 1e-6
    s.close()


# The sparse build over more listed tiles than one of its launches takes (2^23):
# couples of points, all others far apart, so the graph is known.
def test_sparse_build_in_several_launches(torch):
    half, m = 550_000, 20
    rng = np.random.default_rng(11)
    X = rng.standard_normal((half, m), dtype=np.float32)
    X = np.concatenate([X, X])
    X[half:, 0] += 0.05
    y = np.where(rng.random(2 * half) < 0.5, 1.0, -1.0).astype(np.float32)
    s = gabp.GabpSVM(kernel="rbf_sparse", sparse_tau=0.9, gamma=1.0, C=1.0, precision="mixed", max_sweeps=2)
    s.solve(torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda())
    assert s.plan()["n_tiles"] > 1 << 23
    k = np.arange(half)
    assert np.array_equal(s.edges(), np.stack([k, k + half], axis=1))
    s.close()
