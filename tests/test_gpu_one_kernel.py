"""Small products, which run as one kernel: tile edges (32 x 32), chunk edges
(64 k), single rows and columns, padded leading dimensions, every residue
route (t up to 51, 52 and beyond), both quantisers, C -= AB, non-finite rows
and columns, and the leading dimensions on either side of the kernel's limit
-- against the oracle, bit for bit."""
import numpy as np
import pytest

import oracle
import paper_2609_09095_amd as oz
import workloads
from gpu_util import assert_bits_equal, log, require_gpu

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


def _run(A, B, C0, set, quant, pad):
    import torch
    Ad, Bd = _dev(A, pad), _dev(B, pad)
    Cd = _dev(C0 if C0 is not None else np.zeros((A.shape[0], B.shape[1])), pad)
    oz.ozaki25_dgemm_ex(Ad, Bd, Cd, subtract=C0 is not None, set=set, quantiser=quant)
    torch.cuda.synchronize()
    return Cd.cpu().numpy()


@pytest.mark.parametrize("set", [oz.S12, oz.A15])
@pytest.mark.parametrize("m, n, k, pad", [(1, 1, 1, 0), (32, 32, 64, 0), (31, 33, 63, 1), (33, 31, 65, 3), (1, 70, 128, 0),
                                          (97, 1, 129, 1), (64, 96, 255, 2), (65, 34, 511, 1), (40, 24, 640, 0),
                                          (300, 200, 20, 5)])
def test_one_kernel_matches_oracle(m, n, k, pad, set):
    A = workloads.random_matrix(m, k, 2.0, 900 + m)
    B = workloads.random_matrix(k, n, 2.0, 901 + n)
    C0 = workloads.random_matrix(m, n, 1.0, 902 + k)
    for quant in (oz.RN, oz.TZ):
        for c in (None, C0):
            log(f"one kernel set={set} quant={quant} m={m} n={n} k={k} pad={pad} subtract={c is not None}")
            want = oracle.dgemm(A, B, C_in=c, set=set, quant=quant, want_planes=False).C
            assert_bits_equal(_run(A, B, c, set, quant, pad), want, "C")


@pytest.mark.parametrize("set", [oz.S12, oz.A15])
def test_one_kernel_edge_values(set):
    m, n, k = 50, 45, 150
    A = workloads.random_matrix(m, k, 1.0, 910)
    B = workloads.random_matrix(k, n, 1.0, 911)
    A[3] = 0.0
    A[5] *= 1e-310
    A[7, 2], A[9, 149], A[34, 64] = np.inf, np.nan, -np.inf
    B[:, 4] = 0.0
    B[11, 40], B[149, 33] = np.nan, np.inf
    B[:, 8] *= 1e300
    C0 = workloads.random_matrix(m, n, 1.0, 912)
    for c in (None, C0):
        log(f"one kernel set={set} zero, subnormal, huge and non-finite vectors subtract={c is not None}")
        want = oracle.dgemm(A, B, C_in=c, set=set, want_planes=False).C
        assert_bits_equal(_run(A, B, c, set, oz.RN, 1), want, "C")


@pytest.mark.parametrize("ldb", [1 << 21, (1 << 21) + 1])
def test_one_kernel_leading_dimension_limit(ldb):
    import torch
    m, n, k = 33, 40, 70
    A = workloads.random_matrix(m, k, 1.0, 920)
    B = workloads.random_matrix(k, n, 1.0, 921)
    log(f"one kernel ldb={ldb}")
    full = torch.zeros((k, ldb), dtype=torch.float64, device="cuda")
    Bd = full[:, :n]
    Bd.copy_(torch.from_numpy(B))
    Cd = torch.empty((m, n), dtype=torch.float64, device="cuda")
    oz.ozaki25_dgemm_ex(torch.from_numpy(A).cuda(), Bd, Cd)
    torch.cuda.synchronize()
    assert_bits_equal(Cd.cpu().numpy(), oracle.dgemm(A, B, want_planes=False).C, "C")
