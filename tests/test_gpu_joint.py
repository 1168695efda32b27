"""The joint exponent scan and deconstruction of both operands, and the
separate launches beyond their limit, against the oracle bit for bit: rows of
A on either side of the wavefront-per-row length (1024), odd starts, slabs of
64 and 256 rows of B, partial slabs, and the slab limit itself."""
import numpy as np
import pytest

import oracle
import paper_2609_09095_amd as oz
import workloads
from gpu_util import assert_bits_equal, log, require_gpu
from routes import route, rules

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    require_gpu()


def _dev(M, pad):
    import torch
    full = torch.full((M.shape[0], M.shape[1] + pad), float("nan"), dtype=torch.float64, device="cuda")
    view = full[:, :M.shape[1]]
    view.copy_(torch.from_numpy(M))
    return view


# slabs: the partial maxima per column that the joint scan leaves, 0: separate
@pytest.mark.parametrize("m, n, k, pad, slabs", [
    (301, 201, 1023, 1, 16), (301, 130, 1024, 0, 16), (299, 257, 1025, 1, 17), (65, 300, 2000, 2, 32),
    (2000, 70, 1025, 1, 17), (5, 300, 65537, 1, 257), (3, 5, 524288, 0, 2048), (3, 5, 524289, 1, 0), (1, 1, 600001, 0, 0)])
def test_joint_and_separate_launches(m, n, k, pad, slabs):
    import torch
    assert route(m, n, k, k + pad, n + pad) != "one"
    kp = -(-k // 128) * 128
    room = 15 * n * kp if m >= 1024 and n <= 128 else 15 * (m + n) * kp  # what the published set's workspace leaves
    assert rules().rule_both_at_once(m, n, k, kp, room) == (slabs > 0)
    assert slabs == 0 or rules().rule_scan_both_slabs(n, k) == slabs
    A = workloads.random_matrix(m, k, 1.0, 510 + n)
    B = workloads.random_matrix(k, n, 1.0, 511 + m)
    # the largest magnitude of a row and a column at the end of k, and a
    # non-finite one there
    A[0, k - 1], B[k - 1, 0] = 3.0e40, -2.0e50
    if m > 2 and n > 2:
        A[2, k - 1], B[k - 1, 2] = np.inf, np.nan
    log(f"joint m={m} n={n} k={k} pad={pad} slabs={slabs}")
    C = torch.full((m, n), 7.0, dtype=torch.float64, device="cuda")
    oz.ozaki25_dgemm_ex(_dev(A, pad), _dev(B, pad), C, set=oz.S12)
    torch.cuda.synchronize()
    rows = np.unique(np.r_[0, min(2, m - 1), np.linspace(0, m - 1, min(m, 24)).astype(int)])
    want = oracle.dgemm(A, B, rows=rows, set=oz.S12, want_planes=False).C
    assert_bits_equal(C.cpu().numpy()[rows], want, "C (sampled rows)")
