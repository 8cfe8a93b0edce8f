"""Augmented rows of the decision function and of the recomputed K': the last
column, -c/2 |x|^2, is the split of the product itself.

Tolerance: each BF16 term leaves at most 2^-9 of what it splits, three of them
2^-27 of the value; doubled, 2^-26.  The product rounded to FP32 would err by
2^-24 of values just above a power of two.
"""
import ctypes as ct

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


@pytest.mark.parametrize("n,m,mp", [(1, 1, 32), (257, 30, 32), (1000, 62, 64)])
def test_norm_column_is_the_product(torch, n, m, mp):
    vp = ct.c_void_p
    f = gabp.lib()._ZN4gabp16launch_stage_augEPKfPKdllliiifPtP12ihipStream_t
    f.argtypes = [vp, vp, ct.c_int64, ct.c_int64, ct.c_int64, ct.c_int, ct.c_int, ct.c_int, ct.c_float, vp, vp]
    rng = np.random.default_rng(n)
    npad, three_terms = (n + 255) // 256 * 256, 4
    X = torch.from_numpy(rng.standard_normal((n, m)).astype(np.float32)).cuda()
    mean = torch.zeros(m, dtype=torch.float64, device="cuda")
    c = np.float32(2.0 * 0.05 * 1.4426950408889634)
    rows = []
    for side in (0, 1):
        o = torch.zeros(3 * npad * mp, dtype=torch.bfloat16, device="cuda")
        assert f(X.data_ptr(), mean.data_ptr(), n, m, npad, mp, three_terms, side, ct.c_float(c), o.data_ptr(),
                 torch.cuda.current_stream().cuda_stream) == 0
        rows.append(o.view(3, npad, mp).double().sum(dim=0).cpu().numpy())
    norm = rows[0][:n, m].astype(np.float32).astype(np.float64)      # FP32, three terms hold it
    want = -0.5 * float(c) * norm
    assert np.all(np.abs(rows[1][:n, m + 1] - want) <= 2.0 ** -26 * np.abs(want))
    assert np.all(rows[1][n:] == 0) and np.all(rows[0][n:] == 0)
