"""Small products, which run as one kernel: tile edges (32 x 32), chunk edges
(64 k), single rows and columns, padded leading dimensions, every residue
route (t up to 51, 52 and beyond), both quantisers, C -= AB, non-finite rows
and columns, grids of several rounds of CUs, tall products, and the leading
dimensions on either side of the kernel's limit -- against the oracle, bit for
bit."""
import numpy as np
import pytest

import oracle
import paper_2609_09095_amd as oz
import workloads
from gpu_util import assert_bits_equal, log, require_gpu, sample_indices
from routes import route

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
    assert route(m, n, k, k + pad, n + pad) == "one"
    A = workloads.random_matrix(m, k, 2.0, 900 + m)
    B = workloads.random_matrix(k, n, 2.0, 901 + n)
    C0 = workloads.random_matrix(m, n, 1.0, 902 + k)
    for quant in (oz.RN, oz.TZ):
        for c in (None, C0):
            log(f"one kernel set={set} quant={quant} m={m} n={n} k={k} pad={pad} subtract={c is not None}")
            want = oracle.dgemm(A, B, C_in=c, set=set, quant=quant, want_planes=False).C
            assert_bits_equal(_run(A, B, c, set, quant, pad), want, "C")


@pytest.mark.parametrize("m, n, k", [(512, 512, 768), (256, 256, 1024), (1024, 1024, 64), (2048, 2048, 64),
                                     (4096, 128, 320), (4096, 128, 321)])
def test_rule_is_what_runs(m, n, k):
    """The one launch leaves a caller's workspace alone, the other routes
    write their planes and exponents there: on both sides of the rule."""
    import torch
    A = torch.zeros((m, k), dtype=torch.float64, device="cuda")
    B = torch.zeros((k, n), dtype=torch.float64, device="cuda")
    C = torch.empty((m, n), dtype=torch.float64, device="cuda")
    ws = torch.full((oz.ozaki25_dgemm_workspace_size(m, n, k),), 0xA5, dtype=torch.uint8, device="cuda")
    oz.ozaki25_dgemm_ex(A, B, C, workspace=ws)
    torch.cuda.synchronize()
    assert bool((ws == 0xA5).all()) == (route(m, n, k) == "one")


# more than one round of 256 tiles, and rows enough for storage mode F
@pytest.mark.parametrize("set", [oz.S12, oz.A15])
@pytest.mark.parametrize("m, n, k, pad", [(700, 600, 64, 1), (513, 545, 130, 0), (1024, 128, 64, 0), (1100, 90, 300, 1),
                                          (1040, 24, 600, 0), (2049, 1, 257, 3), (1030, 128, 8, 0), (1024, 3, 575, 0),
                                          (9000, 20, 250, 1), (16384, 64, 64, 0), (40001, 33, 100, 2)])
def test_one_kernel_many_tiles_match_oracle(m, n, k, pad, set):
    assert route(m, n, k, k + pad, n + pad) == "one"
    A = workloads.random_matrix(m, k, 2.0, 930 + n)
    B = workloads.random_matrix(k, n, 2.0, 931 + m)
    C0 = workloads.random_matrix(m, n, 1.0, 932 + k)
    A[m - 3, k - 1] = np.inf
    rows = np.unique(np.r_[m - 3, sample_indices(m, 200, 933)])
    for quant, c in ((oz.RN, None), (oz.TZ, C0)):
        log(f"one kernel set={set} quant={quant} m={m} n={n} k={k} pad={pad} subtract={c is not None}")
        want = oracle.dgemm(A, B, C_in=c, rows=rows, set=set, quant=quant, want_planes=False).C
        assert_bits_equal(_run(A, B, c, set, quant, pad)[rows], want, "C (sampled rows)")


@pytest.mark.parametrize("set", [oz.S12, oz.A15])
def test_one_kernel_edge_values(set):
    m, n, k = 50, 45, 150
    assert route(m, n, k, k + 1, n + 1) == "one"
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
    assert route(m, n, k, k, ldb) == ("one" if ldb <= 1 << 21 else "staged")
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
