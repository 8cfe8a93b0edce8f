"""Series sweeps summed over powers of K' (one, two and three levels) where
the powers beyond the second matter: their terms in the message sums.

The message sums A_ii - P~_i of systems of about 300 points, whose
contraction is the largest that three levels of form 3 take (1.25 rho just
below 2^-8): a third and a fourth power of K' enter them with rho^2, 9e-6.
Tolerance (relative) against the FP64 oracle: 16 x 2^-24 = 9.5e-7; at most 8
roundings of one message in FP32 (K' and its power, the factors and their
products) and 8 = sqrt(64) for sums of 64 messages.  alpha: 1e-5 (inf-norm,
relative) as everywhere.
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


def labels(rng, n):
    return np.where(rng.random(n) < 0.5, 1.0, -1.0).astype(np.float32)


def check_messages(s, K, y, sweeps):
    adiag = s.adiag()
    A = (y[:, None] * y[None, :]).astype(np.float64) * K
    np.fill_diagonal(A, adiag)
    ref = R.gabp_solve(A, np.ones(len(y)), max_sweeps=sweeps, tol_rel=0.0)
    want = adiag - ref.ptilde
    err = float(np.max(np.abs((adiag - s.ptilde()) / want - 1.0)))
    ea = float(np.max(np.abs(s.alpha() - ref.alpha)) / np.max(np.abs(ref.alpha)))
    print(f"[case] message sums {err:.2e}, alpha {ea:.2e}", flush=True)
    assert err <= 16 * 2.0 ** -24 and ea <= 1e-5, (err, ea)


FIXED = dict(precision="mixed", edge_state="stateless", stateless_depth=3, tol_abs=0.0, tol_rel=0.0,
             stagnation_window=0)


@pytest.mark.parametrize("n", [300, 513])
@pytest.mark.parametrize("chunk", [1, 2])
@pytest.mark.parametrize("sweeps", [1, 2, 3, 6])
def test_fourth_power_over_the_plane(torch, n, chunk, sweeps):
    rng = np.random.default_rng(n)
    K = 1.0 + 0.01 * rng.random((n, n))
    K = ((K + K.T) / 2).astype(np.float32).astype(np.float64)      # exact in the plane
    y = labels(rng, n)
    s = gabp.GabpSVM(kernel="precomputed", C=1.0, tile_chunk=chunk, max_sweeps=sweeps, **FIXED)
    s.solve_kernel(torch.from_numpy(K).cuda(), torch.from_numpy(y).cuda())
    p = s.plan()
    assert p["series_reciprocal"] == 3 and p["tile_chunk"] == chunk and 1.25 * p["stateless_rho"] < 2.0 ** -8
    check_messages(s, K, y, sweeps)
    s.close()


# 300 points: tiles in eight parts (through the LDS band); 6,000: two parts,
# from the MFMA output (against the same system over the plane)
@pytest.mark.parametrize("m", [20, 62])
def test_fourth_power_recomputed(torch, m):
    rng = np.random.default_rng(m)
    gamma, n = 0.05, 300
    X = (0.05 * rng.standard_normal((n, m))).astype(np.float32)
    y = labels(rng, n)
    d = X.astype(np.float64)
    K = np.exp(-gamma * ((d[:, None, :] - d[None, :, :]) ** 2).sum(axis=2)) + (1.0 / n) ** 2
    s = gabp.GabpSVM(gamma=gamma, C=1.0, kstore="recompute", max_sweeps=4, **FIXED)
    s.solve(torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda())
    p = s.plan()
    assert p["series_reciprocal"] == 3 and p["recompute_aug"] == 1 and 1.25 * p["stateless_rho"] < 2.0 ** -8
    check_messages(s, K, y, 4)
    s.close()


# The recomputed form adds a row's 256 columns of a tile in FP64 (a lane's eight
# in FP32), the plane four strips of 64 added in FP32: its message sums must be
# the closer ones to FP64 (rms over the nodes; the longer FP32 sums make up
# about half of the plane's error here, so by 5% at least).
def test_recomputed_row_sums_in_64_bits(torch):
    from paper_0810_1648_amd import inputs
    X, y = inputs.cluster_mixture(6000, 20, 71)
    Xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    m = {}
    for name, kw in (("fp64", dict(precision="fp64", edge_state="stored", kstore="materialise")),
                     ("plane", dict(FIXED, kstore="materialise")), ("recompute", dict(FIXED, kstore="recompute"))):
        base = dict(tol_abs=0.0, tol_rel=0.0, stagnation_window=0)
        s = gabp.GabpSVM(gamma=0.0005, C=1.0, max_sweeps=6, **dict(base, **kw))
        s.solve(Xd, yd)
        if name != "fp64":
            assert s.plan()["series_reciprocal"] == 3
        m[name] = s.adiag() - s.ptilde()
        s.close()
    rms = {k: float(np.std(m[k] / m["fp64"])) for k in ("plane", "recompute")}
    print(f"[case] message sums rms {rms}", flush=True)
    assert rms["recompute"] <= 0.95 * rms["plane"], rms


# A system times a power of two is the same system: the same rho, depth and
# form, alpha over the scale.  Beyond 2^30 (or P~ below 2^-16) the fourth power
# of K' leaves the range of FP32, and the sweep runs level by level.
# Tolerance: the rounding of the two ways, 16 x 2^-24 each.
@pytest.mark.parametrize("exponent", [-53, -43, -20, 30, 33, 43, 53])
@pytest.mark.parametrize("prec,depth", [("fp32", 2), ("fp32", 3), ("mixed", 2), ("mixed", 3)])
@pytest.mark.parametrize("chunk", [1, 2])
def test_given_matrix_of_any_scale(torch, exponent, prec, depth, chunk):
    n, scale = 513, 2.0 ** exponent
    rng = np.random.default_rng(n)
    K = 1.0 + 0.01 * rng.random((n, n))
    K = ((K + K.T) / 2).astype(np.float32).astype(np.float64)
    y = labels(rng, n)
    yd = torch.from_numpy(y).cuda()
    got = {}
    for f in (1.0, scale):
        s = gabp.GabpSVM(kernel="precomputed", C=1e30, tile_chunk=chunk, max_sweeps=6,
                         **dict(FIXED, precision=prec, stateless_depth=depth))
        assert s.solve_kernel(torch.from_numpy(K * f).cuda(), yd) == gabp.E_NOT_CONVERGED     # (sweeps as asked)
        p = s.plan()
        assert p["series_reciprocal"] == (3 if depth == 3 else 1) and p["tile_chunk"] == chunk
        got[f] = s.alpha() * f
        if prec == "mixed":
            check_messages(s, K * f, y, 6)
        s.close()
    err = float(np.max(np.abs(got[scale] - got[1.0])) / np.max(np.abs(got[1.0])))
    assert err <= 32 * 2.0 ** -24, err


# the augmentation lambda^2 = 2^44 makes every entry of an RBF system that large:
# the plane, K' recomputed (through the band; 6,000 points: the plans that take
# the MFMA output otherwise) and a served request, against FP64
@pytest.mark.parametrize("n", [513, 6000])
def test_large_augmentation(torch, n):
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, 20)).astype(np.float32)
    y = labels(rng, n)
    Xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    common = dict(gamma=0.05, C=1.0, lambda_aug=2.0 ** 22, max_sweeps=5, tol_abs=0.0, tol_rel=0.0, stagnation_window=0)
    s = gabp.GabpSVM(precision="fp64", edge_state="stored", kstore="materialise", **common)
    s.solve(Xd, yd)
    ref = s.alpha()
    s.close()
    for prec, depth, kstore in (("mixed", 3, "materialise"), ("mixed", 3, "recompute"), ("fp32", 2, "materialise"),
                                ("fp32", 2, "recompute")):
        print(f"[case] lambda 2^22 n={n} {prec} {depth} {kstore}", flush=True)
        kw = dict(common, precision=prec, stateless_depth=depth, edge_state="stateless", kstore=kstore)
        s = gabp.GabpSVM(**kw)
        assert s.solve(Xd, yd) == gabp.E_NOT_CONVERGED
        assert s.plan()["series_reciprocal"] == (3 if depth == 3 else 1)
        a = s.alpha()
        s.close()
        assert float(np.max(np.abs(a - ref)) / np.max(np.abs(ref))) <= 1e-5
        if kstore == "materialise" and n == 513:
            with gabp.GabpServer() as srv:
                t = srv.submit(X, y, **kw)
                assert srv.wait(t, 60.0)
                served, _ = srv.result(t)
            assert np.array_equal(served, a)
