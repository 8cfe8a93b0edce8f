"""Decision function of few queries (queries augmented and weights formed in
the kernel) against the FP64 oracle and against the bulk form, on both sides
of the rule that chooses between them (queries x padded points <= 45 million,
or at most 32 queries).

Tolerances of sum |alpha| (K' <= 1 + lambda^2), as for the other forms: 1e-5
for FP32 features and the three-term split, 1e-4 for two terms, 1e-2 for one;
twice that between the two forms.
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


@pytest.mark.parametrize("prec,gram,m,tol", [("mixed", "auto", 54, 1e-5), ("mixed", "auto", 20, 1e-5),
                                             ("mixed", "auto", 62, 1e-5), ("mixed", "bf16x3", 30, 1e-4),
                                             ("mixed", "bf16", 31, 1e-2), ("fp32", "auto", 30, 1e-5)])
def test_few_queries(torch, prec, gram, m, tol):
    n = 3001                                   # 94 blocks of 32 rows, 3,072 padded
    last = 45000000 // 3072                    # the largest call of the few-query form
    X, y, Xq, _ = inputs.linear_teacher(n, m, 81, n_test=last + 1)
    print(f"[case] few queries {prec}/{gram} m={m}", flush=True)
    s = gabp.GabpSVM(gamma=1.0 / m, C=1.0, precision=prec, gram=gram, tol_rel=1e-6)
    s.solve(torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda())
    alpha = s.alpha()
    scale = float(np.abs(alpha).sum())
    ref = R.decision_function(X, y, alpha, Xq[:65], 1.0 / m, 1.0 / n)
    bulk = s.predict(torch.from_numpy(Xq).cuda()).cpu().numpy()
    edge = s.predict(torch.from_numpy(Xq[:last]).cuda()).cpu().numpy()
    assert np.max(np.abs(bulk[:last] - edge)) <= 2 * tol * scale
    for nq in (1, 31, 32, 33, 65):
        f = s.predict(torch.from_numpy(Xq[:nq]).cuda()).cpu().numpy()
        assert f.shape == (nq,)
        assert np.max(np.abs(f - ref[:nq])) <= tol * scale, (prec, gram, m, nq)
    s.close()
