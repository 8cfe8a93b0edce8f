"""Sweeps over K' recomputed from augmented rows, formed in the MFMA's layout,
against the same sweeps over the materialised K', where tiles are split in two
(6,000 points) and whole (8,200), with 32 and 64 padded features and every
split of the features.

Tolerances (relative, inf-norm): K' of the two plans differs by the Gram's
rounding, as in the other tests of the two plans: 1e-6 for the three-term
split, 1e-4 for two terms, 1e-2 for one.
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


@pytest.mark.parametrize("n", [6000, 8200])
@pytest.mark.parametrize("m,gamma", [(20, 0.01), (54, 0.05), (62, 0.01), (30, 0.01)])
@pytest.mark.parametrize("gram,tol", [("bf16x6", 1e-6), ("bf16x3", 1e-4), ("bf16", 1e-2)])
def test_recomputed_sweeps_match_the_plane(torch, n, m, gamma, gram, tol):
    if m == 54:
        X, y = inputs.covertype_like(n, m, 71)
    else:
        X, y = inputs.cluster_mixture(n, m, 71)
    Xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    for t in (1, 2, 6):
        a = {}
        for ks in ("materialise", "recompute"):
            print(f"[case] recompute n={n} m={m} {gram} {ks} t={t}", flush=True)
            s = gabp.GabpSVM(gamma=gamma, C=1.0, precision="mixed", gram=gram, kstore=ks, edge_state="stateless",
                             stateless_depth=3, max_sweeps=t, tol_abs=0.0, tol_rel=0.0, stagnation_window=0)
            s.solve(Xd, yd)
            p = s.plan()
            assert p["series_reciprocal"] == 3 and p["recompute_aug"] == (1 if ks == "recompute" else 0)
            a[ks] = s.alpha()
            s.close()
        err = float(np.max(np.abs(a["recompute"] - a["materialise"])) / np.max(np.abs(a["materialise"])))
        assert err <= tol, (n, m, gram, t, err)
