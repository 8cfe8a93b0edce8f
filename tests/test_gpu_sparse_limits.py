"""The sparse graph build beyond 32 bits: its scan by itself, and a graph whose
rows hold more than 2^31 entries.

Tolerances: whole numbers are equal; alpha 1e-5 (inf-norm, relative), as for
the other sparse tests.
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


def _entry(name, *argtypes):
    f = getattr(gabp.lib(), name)
    f.argtypes, f.restype = argtypes, ct.c_int
    return f


# row lengths whose sums pass 2^31 (at 2^30 kept pairs) and 2^32
@pytest.mark.parametrize("n,length", [(3, 2 ** 30 + 4), (1 << 16, 1 << 16), (100_003, 65_540)])
def test_row_offsets_beyond_32_bits(torch, n, length):
    vp = ct.c_void_p
    scan = _entry("_ZN4gabp7sp_scanEPvPmPKlPllP12ihipStream_t", vp, ct.POINTER(ct.c_size_t), vp, vp, ct.c_int64, vp)
    x = torch.full((n + 1,), length, dtype=torch.int64, device="cuda")
    out = torch.zeros_like(x)
    s = torch.cuda.current_stream().cuda_stream
    nb = ct.c_size_t(0)
    assert scan(None, ct.byref(nb), x.data_ptr(), out.data_ptr(), n + 1, s) == 0
    tmp = torch.empty(max(nb.value, 16), dtype=torch.uint8, device="cuda")
    assert scan(tmp.data_ptr(), ct.byref(nb), x.data_ptr(), out.data_ptr(), n + 1, s) == 0
    assert torch.equal(out, length * torch.arange(n + 1, dtype=torch.int64, device="cuda"))
    assert int(out[-1]) > 2 ** 31


# every pair of 47,000 points kept: 1.1e9 pairs, 2.2e9 directed edges, the same
# system as the dense solve over stored records
def test_graph_of_more_than_2_30_pairs(torch):
    n = 47_000
    if torch.cuda.mem_get_info()[0] < 160 << 30:
        pytest.skip("needs 160 GiB of device memory")
    rng = np.random.default_rng(5)
    X = torch.from_numpy((0.3 * rng.standard_normal((n, 6))).astype(np.float32)).cuda()
    y = torch.from_numpy(np.where(rng.random(n) < 0.5, 1.0, -1.0).astype(np.float32)).cuda()
    kw = dict(gamma=0.5, C=10.0, lambda_aug=1.0 / n, precision="mixed", max_sweeps=5, tol_abs=0.0, tol_rel=0.0,
              stagnation_window=0)
    a = {}
    for kernel, how in (("rbf", dict(edge_state="stored", kstore="materialise")), ("rbf_sparse", dict(sparse_tau=1e-12))):
        s = gabp.GabpSVM(kernel=kernel, **kw, **how)
        s.solve(X, y)
        if kernel == "rbf_sparse":
            assert s.plan()["n_edges"] == n * (n - 1) // 2
        a[kernel] = s.alpha()
        s.close()
    assert float(np.max(np.abs(a["rbf_sparse"] - a["rbf"])) / np.max(np.abs(a["rbf"]))) <= 1e-5


# augmented rows of more values than one launch holds threads
def test_augmented_rows_of_more_than_2_32_values(torch):
    vp, n, mp = ct.c_void_p, 65_792, 65_536
    m = mp - 2
    aug = _entry("_ZN4gabp17launch_sp_augmentElliiPKfPfPtS3_S3_S2_S3_S3_S3_P12ihipStream_t", ct.c_int64, ct.c_int64,
                 ct.c_int, ct.c_int, vp, vp, vp, vp, vp, vp, vp, vp, vp, vp)
    a = torch.ones((n, mp), dtype=torch.bfloat16, device="cuda")
    b = torch.zeros_like(a)
    nrm = 2.0 ** (torch.arange(n, device="cuda") % 8).float()      # exact in BF16
    one_term = 1                                                    # the kind whose rows are one BF16 plane
    assert a.numel() > 2 ** 32
    assert aug(n, m, mp, one_term, nrm.data_ptr(), None, a.data_ptr(), None, None, None, b.data_ptr(), None, None,
               torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert bool((b[:, :m] == 1).all()) and bool((a[:, :m] == 1).all())
    assert torch.equal(a[:, m].float(), nrm) and bool((a[:, m + 1] == 1).all())
    assert bool((b[:, m] == -0.5).all()) and torch.equal(b[:, m + 1].float(), -0.5 * nrm)


# 80 bytes per kept pair hold the build (with an edge list 1.5 times the graph)
# and, after it, the sweep: 2e8 pairs in 16 GiB, the same to the bit
def test_records_take_the_place_of_the_sort(torch):
    n = 20_000
    free = torch.cuda.mem_get_info()[0]
    if free < 60 << 30:
        pytest.skip("needs 60 GiB of device memory")
    rng = np.random.default_rng(6)
    X = torch.from_numpy((0.3 * rng.standard_normal((n, 6))).astype(np.float32)).cuda()
    y = torch.from_numpy(np.where(rng.random(n) < 0.5, 1.0, -1.0).astype(np.float32)).cuda()
    kw = dict(kernel="rbf_sparse", sparse_tau=1e-12, gamma=0.5, C=10.0, precision="mixed", max_sweeps=3, tol_abs=0.0,
              tol_rel=0.0, stagnation_window=0)
    alpha = []
    for left in (None, 16 << 30):
        torch.cuda.empty_cache()
        rest = torch.empty(torch.cuda.mem_get_info()[0] - left, dtype=torch.uint8, device="cuda") if left else None
        s = gabp.GabpSVM(**kw)
        for _ in range(2 if left else 1):          # (again on a handle that holds what it needs)
            s.solve(X, y)
            assert s.plan()["n_edges"] == n * (n - 1) // 2
            alpha.append(s.alpha())
        s.close()
        del rest
    torch.cuda.empty_cache()
    assert np.array_equal(alpha[0], alpha[1]) and np.array_equal(alpha[0], alpha[2])


# Points without edges cost the build no more than the same points with edges
# to their neighbours (a chain of stores by one lane took ten times as long;
# 1 ms for the timing's own spread).
def test_isolated_points_in_parallel(torch):
    side = 700
    X = np.ascontiguousarray(np.indices((side, side)).reshape(2, -1).T.astype(np.float32) - side // 2)
    y = np.where(np.random.default_rng(1).random(len(X)) < 0.5, 1.0, -1.0).astype(np.float32)
    Xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    ms = {}
    for tau, edges in ((0.5, 0), (0.04, 2 * side * (side - 1))):       # K of neighbours: 1 / 16
        s = gabp.GabpSVM(kernel="rbf_sparse", sparse_tau=tau, gamma=4.0 * np.log(2.0), C=1.0, precision="mixed",
                         max_sweeps=2)
        t = []
        for _ in range(4):
            s.solve(Xd, yd)
            assert s.plan()["n_edges"] == edges
            t.append(s.timings()["kbuild_ms"])
        ms[edges] = min(t)
        s.close()
    print(f"[case] build of isolated points and of a grid: {ms} ms", flush=True)
    assert ms[0] <= ms[2 * side * (side - 1)] + 1.0, ms


# a solve that only succeeds after it has given up what the handle held from the
# solve before: no error message is left of its first attempt
def test_no_message_after_a_second_attempt(torch):
    n = 20_000
    if torch.cuda.mem_get_info()[0] < 60 << 30:
        pytest.skip("needs 60 GiB of device memory")
    rng = np.random.default_rng(6)
    X = torch.from_numpy((0.3 * rng.standard_normal((n, 6))).astype(np.float32)).cuda()
    y = torch.from_numpy(np.where(rng.random(n) < 0.5, 1.0, -1.0).astype(np.float32)).cuda()
    torch.cuda.empty_cache()
    rest = torch.empty(torch.cuda.mem_get_info()[0] - (16 << 30), dtype=torch.uint8, device="cuda")
    s = gabp.GabpSVM(kernel="rbf_sparse", sparse_tau=1e-12, gamma=0.5, C=10.0, precision="mixed", tol_abs=1e30)
    for _ in range(2):
        assert s.solve(X, y) == gabp.OK
        assert gabp.lib().gabp_svm_last_error(s._h) == b""
    s.close()
    del rest
    torch.cuda.empty_cache()
