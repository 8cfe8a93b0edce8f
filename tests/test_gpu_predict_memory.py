"""Host-buffer calls of the decision function keep their device buffers in the
handle: repeated calls take no more memory.

Bound: 16 MiB of drift of the device's free memory, against 6 MiB a call.
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


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_repeated_host_calls_hold_one_batch(torch, prec):
    wl = inputs.make_workload("tiny", n=300, seed=3)
    Xq = np.random.default_rng(0).standard_normal((1 << 17, wl.m)).astype(np.float32)
    s = gabp.GabpSVM(gamma=wl.gamma, C=wl.C, precision=prec)
    s.solve(wl.X, wl.y)
    f = s.predict(Xq)
    free = torch.cuda.mem_get_info()[0]
    for _ in range(10):
        assert np.array_equal(s.predict(Xq), f)
    assert free - torch.cuda.mem_get_info()[0] <= 16 << 20
    assert np.array_equal(s.predict(Xq[:77]), s.predict(torch.from_numpy(Xq[:77]).cuda()).cpu().numpy())
    s.close()
