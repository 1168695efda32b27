"""Storage mode F for A (at most 128 columns, at least 1024 rows, both
modulus sets): ozaki25_dgemm_ex converts A inside the product kernel instead
of storing its planes.  Outputs are compared with the oracle bit for bit
(any NaN matching any NaN), all of them or on sampled rows that include both
ends: ragged rows, columns and k, one column, k past the 65536 after which
the int32 sums are reduced, C -= AB, the truncating quantiser, rows and
columns with non-finite values (native re-issue), a wide exponent range, and
zero, subnormal, huge and tie rows.  Every size asserts that it reaches the
kernel -- smaller products run as one launch -- and which of its forms, with
three or five moduli per block."""
import numpy as np
import pytest

import oracle
import paper_2609_09095_amd as oz
import workloads
from gpu_util import assert_bits_equal, log, require_gpu, sample_indices, to_dev
from routes import route, rules

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    require_gpu()


SETS = [pytest.param(oz.S12, id="S12"), pytest.param(oz.A15, id="A15")]
# rows that take three and five moduli per block
FORMS = [pytest.param(5000, 3, id="G3"), pytest.param(6600, 5, id="G5")]


def _reaches(m, n, k, moduli):
    assert route(m, n, k) == "fused", (m, n, k)
    assert rules().rule_fused_moduli(m) == moduli, m


def _run(A, B, set, C0=None, quant=oz.RN):
    import torch
    m, k = A.shape
    n = B.shape[1]
    ws = torch.empty(oz.ozaki25_dgemm_workspace_size(m, n, k, set), dtype=torch.uint8, device="cuda")
    C = to_dev(C0) if C0 is not None else torch.empty((m, n), dtype=torch.float64, device="cuda")
    oz.ozaki25_dgemm_ex(to_dev(A), to_dev(B), C, subtract=C0 is not None, workspace=ws, set=set,
                        quantiser=quant)
    torch.cuda.synchronize()
    return C.cpu().numpy()


def _want(A, B, set, rows, C0=None, quant=oz.RN):
    return oracle.dgemm(A, B, C_in=C0, rows=rows, set=set, want_planes=False,
                        quant=oracle.TZ if quant == oz.TZ else oracle.RN).C


# k 8 and 64 on the published set, and 300, 2000 and 8192 on the all-byte one,
# take each residue route (t up to 51, 52, beyond)
@pytest.mark.parametrize("set", SETS)
@pytest.mark.parametrize("m,n,k,s,moduli", [(1300, 70, 1000, 1.0, 3), (2049, 1, 1500, 2.0, 3), (4096, 128, 4096, 1.0, 3),
                                            (5100, 100, 200, 4.0, 3), (11000, 33, 600, 1.0, 3), (1100, 20, 8192, 1.0, 3),
                                            (6600, 70, 2000, 1.0, 5), (6145, 9, 8192, 0.5, 5), (18500, 128, 8, 0.5, 5),
                                            (18500, 127, 64, 1.0, 5), (13001, 101, 300, 2.0, 5)])
def test_fused_matches_oracle(set, m, n, k, s, moduli):
    _reaches(m, n, k, moduli)
    A = workloads.random_matrix(m, k, s, m)
    B = workloads.random_matrix(k, n, s, n + 100)
    rows = sample_indices(m, 400 if k <= 2000 else 100, 7)
    for quant in (oz.RN, oz.TZ):
        log(f"fused set={set} quant={quant} m={m} n={n} k={k} s={s}")
        assert_bits_equal(_run(A, B, set, quant=quant)[rows], _want(A, B, set, rows, quant=quant), "C (sampled rows)")


@pytest.mark.parametrize("set", SETS)
@pytest.mark.parametrize("m, moduli", FORMS)
def test_fused_k_sweep(set, m, moduli):
    """k around the points where the kernel's main loop (both look-ahead
    stages whole) hands over to its guarded steps, and where the last stage
    turns partial or lies past k: each multiple of 64 from 256 to 576 and its
    two neighbours."""
    n = 100
    rows = sample_indices(m, 64, 8)
    ks = sorted({kk + d for kk in range(256, 577, 64) for d in (-1, 0, 1)})
    for i, k in enumerate(ks):
        _reaches(m, n, k, moduli)
        A = workloads.random_matrix(m, k, 1.0, 300 + i)
        B = workloads.random_matrix(k, n, 1.0, 400 + i)
        log(f"fused set={set} m={m} k={k}")
        assert_bits_equal(_run(A, B, set)[rows], _want(A, B, set, rows), f"C (sampled rows, k={k})")


@pytest.mark.parametrize("set", SETS)
@pytest.mark.parametrize("m, moduli", FORMS)
def test_fused_subtract_tz_and_nonfinite(set, m, moduli):
    n, k = 100, 300
    _reaches(m, n, k, moduli)
    A = workloads.random_matrix(m, k, 1.0, 11)
    B = workloads.random_matrix(k, n, 1.0, 12)
    C0 = workloads.random_matrix(m, n, 1.0, 13)
    A[5, 7] = np.nan
    A[m - 10, 0] = -np.inf
    B[3, 40] = np.inf
    rows = np.unique(np.r_[np.arange(130), m - 10, sample_indices(m, 300, 14)])
    log(f"fused set={set} m={m} C -= AB with non-finite rows and columns")
    assert_bits_equal(_run(A, B, set, C0)[rows], _want(A, B, set, rows, C0), "C -= AB (sampled rows)")
    log(f"fused set={set} m={m} truncating quantiser")
    A[5, 7], A[m - 10, 0], B[3, 40] = 1.0, 2.0, 3.0
    assert_bits_equal(_run(A, B, set, C0, quant=oz.TZ)[rows], _want(A, B, set, rows, C0, quant=oz.TZ),
                      "C -= AB (TZ, sampled rows)")


@pytest.mark.parametrize("set", SETS)
@pytest.mark.parametrize("m, moduli", [pytest.param(1024, 3, id="G3"), pytest.param(6200, 5, id="G5")])
def test_fused_long_k_segments(set, m, moduli):
    """k = 70000 crosses the 65536 after which the int32 sums are reduced mod
    m.  64 different rows of A, repeated on the device."""
    import torch
    n, k = 3, 70000
    _reaches(m, n, k, moduli)
    A = workloads.random_matrix(64, k, 1.0, 21)
    B = workloads.random_matrix(k, n, 1.0, 22)
    log(f"fused set={set} m={m} k={k}")
    Ad = to_dev(A).repeat(-(-m // 64), 1)[:m].contiguous()
    C = torch.full((m, n), 7.0, dtype=torch.float64, device="cuda")
    oz.ozaki25_dgemm_ex(Ad, to_dev(B), C, set=set)
    torch.cuda.synchronize()
    want = np.tile(oracle.dgemm(A, B, set=set, want_planes=False).C, (-(-m // 64), 1))[:m]
    assert_bits_equal(C.cpu().numpy(), want, "C")


@pytest.mark.parametrize("set", SETS)
@pytest.mark.parametrize("quant", [pytest.param(oz.RN, id="RN"), pytest.param(oz.TZ, id="TZ")])
@pytest.mark.parametrize("m, moduli", FORMS)
def test_fused_edge_rows(set, quant, m, moduli):
    """Zero, subnormal, huge, tie, boundary and non-finite rows of A and
    columns of B, converted inside the product kernel with their own row
    scales (k = 600: whole stages, then a partial one)."""
    n, k = 100, 600
    _reaches(m, n, k, moduli)
    A = workloads.edge_rows(workloads.random_matrix(m, k, 1.0, 61), 62)
    B = np.ascontiguousarray(workloads.edge_rows(workloads.random_matrix(n, k, 1.0, 63), 64).T)
    rows = np.unique(np.r_[np.arange(200), sample_indices(m, 200, 65)])
    log(f"fused set={set} m={m} edge rows and columns, quantiser {quant}")
    want = _want(A, B, set, rows, quant=quant)
    got = _run(A, B, set, quant=quant)
    assert_bits_equal(got[rows], want, "C (sampled rows)")
    # row 3 of A and column 3 of B hold a NaN: re-issued natively
    assert np.all(np.isnan(got[3])) and np.all(np.isnan(got[:, 3]))


@pytest.mark.parametrize("set", SETS)
@pytest.mark.parametrize("m, moduli", [pytest.param(1024, 3, id="G3"), pytest.param(6600, 5, id="G5")])
def test_fused_constant_vectors(set, m, moduli):
    """Constant rows of A and columns of B, so that every term of a sum has
    the same residue product and the int32 sums grow without cancellation
    (their largest magnitudes for those residues), beside random rows and
    columns."""
    n, k = 8, 2048
    _reaches(m, n, k, moduli)
    A = workloads.random_matrix(m, k, 1.0, 32)
    B = workloads.random_matrix(k, n, 1.0, 33)
    A[:16, :] = np.ldexp(1.0, -3) * (1 - 2.0 ** -40)
    A[16:32, :] = -1.0
    A[32:48, :] = 3.0 * (1 + 2.0 ** -30)
    B[:, :2] = 7.0 * (1 - 2.0 ** -45)
    B[:, 2] = -3.0
    rows = np.unique(np.r_[np.arange(64), sample_indices(m, 200, 34)])
    log(f"fused set={set} m={m} constant rows and columns")
    assert_bits_equal(_run(A, B, set)[rows], _want(A, B, set, rows), "C (sampled rows)")


@pytest.mark.parametrize("set", SETS)
@pytest.mark.parametrize("lda", [(1 << 20) - 1, 1 << 20, (1 << 20) + 1, (1 << 21) - 1])
def test_fused_leading_dimension_limit(set, lda):
    """Leading dimensions of A on either side of 2^20, up to which the kernel
    takes 24-bit row offsets (8 lda must not reach the sign bit, 2^23), and
    at 2^21 - 1, where such an offset wraps to a small negative one.  NaN
    beyond the k columns: no output may see it."""
    import torch
    m, n, k = 1030, 5, 1000
    assert route(m, n, k, lda) == "fused"
    A = workloads.random_matrix(m, k, 1.0, 81)
    B = workloads.random_matrix(k, n, 1.0, 82)
    log(f"fused set={set} lda={lda}")
    flat = torch.empty((m - 1) * lda + k, dtype=torch.float64, device="cuda")
    flat.fill_(float("nan"))
    Ad = flat.as_strided((m, k), (lda, 1))
    Ad.copy_(torch.from_numpy(A))
    C = torch.full((m, n), 7.0, dtype=torch.float64, device="cuda")
    oz.ozaki25_dgemm_ex(Ad, to_dev(B), C, set=set)
    torch.cuda.synchronize()
    assert_bits_equal(C.cpu().numpy(), oracle.dgemm(A, B, set=set, want_planes=False).C, "C")
