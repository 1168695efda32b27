"""The byte moduli's reconstruction in runs of 1024 outputs: rows shorter than,
equal to and longer than a run, single rows and columns, a partial last run,
residue planes on and off a dword boundary, C -= AB and flagged rows and
columns -- and in strips of 256 columns, whole and partial, which small and
wide outputs take: through stored planes, against the oracle, bit for bit."""
import numpy as np
import pytest

import oracle
import paper_2609_09095_amd as oz
import workloads
from gpu_util import assert_bits_equal, log, require_gpu, to_dev
from routes import rules

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    require_gpu()


RUNS = [(32, 24, 0), (8, 63, 1), (1366, 24, 0), (257, 1023, 0), (301, 1028, 1), (259, 1025, 3), (2049, 129, 0), (5000, 53, 1), (3, 7, 0), (4, 63, 2),
        (1, 1048579, 0), (262147, 1, 2), (513, 513, 1), (2049, 1024, 0)]
STRIPS = [(4, 64, 0), (33, 24, 1), (9, 57, 0), (1040, 31, 2), (520, 63, 0), (300, 1024, 1), (1, 262147, 0),
          (255, 1028, 2), (9, 93106, 1), (2050, 512, 0), (2, 100, 3)]


@pytest.mark.parametrize("m, n, pad, strips", [(*c, False) for c in RUNS] + [(*c, True) for c in STRIPS])
def test_runs_and_strips_match_oracle(m, n, pad, strips):
    import torch
    assert bool(rules().rule_reconstruct_strips(m, n)) == strips
    k = 3
    A = workloads.random_matrix(m, k, 1.0, 700 + n % 97)
    B = workloads.random_matrix(k, n, 1.0, 701 + m % 89)
    if m > 2 and n > 2:
        A[m - 1, 1] = np.inf
        B[2, n // 2] = np.nan
    C0 = workloads.random_matrix(m, n, 1.0, 702)
    pA, eA = oz.ozaki25_deconstruct(0, to_dev(A), set=oz.A15)
    pB, eB = oz.ozaki25_deconstruct(1, to_dev(B), set=oz.A15)
    for c in (None, C0):
        log(f"runs m={m} n={n} pad={pad} subtract={c is not None}")
        full = torch.full((m, n + pad), 5.0, dtype=torch.float64, device="cuda")
        C = full[:, :n]
        if c is not None:
            C.copy_(torch.from_numpy(c))
        oz.ozaki25_dgemm_planes(k, pA, eA, pB, eB, C, subtract=c is not None, set=oz.A15)
        torch.cuda.synchronize()
        want = oracle.dgemm(A, B, C_in=c, set=1, want_planes=False, fallback=False).C
        assert_bits_equal(C.cpu().numpy(), want, "C")
        assert bool((full[:, n:] == 5.0).all())


# results across the whole subnormal range, and exact ones with ties: one
# launch, runs (re-issue inside and apart), storage mode F
@pytest.mark.parametrize("scale", [2.0 ** -515, 2.0 ** -530, 1.0])
@pytest.mark.parametrize("m, n, k", [(300, 200, 20), (700, 650, 300), (2100, 2050, 40), (1500, 100, 500)])
def test_subnormal_and_exact_results_match_oracle(m, n, k, scale):
    import torch
    rng = np.random.default_rng(m + n)
    rows = np.unique(rng.integers(0, m, 60))
    A = workloads.random_matrix(m, k, 3.0, 750)
    B = workloads.random_matrix(k, n, 3.0, 751)
    if scale == 1.0:  # products of FP32 values: ties in the last bits
        A, B = A.astype(np.float32).astype(np.float64), B.astype(np.float32).astype(np.float64)
        A[:, 2:] = 0.0
        A[1] = 0.0
        A[1, 0] = 1.0
    A, B = A * scale, B * scale
    log(f"subnormal results m={m} n={n} k={k} scale={scale}")
    C = torch.empty((m, n), dtype=torch.float64, device="cuda")
    oz.ozaki25_dgemm_ex(to_dev(A), to_dev(B), C)
    torch.cuda.synchronize()
    want = oracle.dgemm(A, B, rows=rows, want_planes=False).C
    assert_bits_equal(C.cpu().numpy()[rows], want, "C (sampled rows)")
