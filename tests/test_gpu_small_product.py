"""Products of a few tiles with k <= 128 (256 up to eight slices), which one kernel splits and multiplies: plain, double-double and BLAS-style, every
storage order, edges of its 32 x 32 tiles, its words of four and its steps of 64 positions, and adversarial values, against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2306_11975_amd import ozimmu
from paper_2306_11975_amd import workloads as wl

pytestmark = pytest.mark.gpu


def bits(x):
    return np.ascontiguousarray(x).view(np.uint64)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def run(A, B, s, extra=0):
    """C of the call with leading dimensions `extra` beyond the rows; what lies between the rows stays as it was."""
    m, k = A.shape
    n = B.shape[1]

    def wide(x):
        y = torch.full((x.shape[0], x.shape[1] + extra), float("nan"), dtype=torch.float64, device="cuda")
        y[:, : x.shape[1]] = dev(x)
        return y[:, : x.shape[1]]

    C = torch.full((m, n + extra), float("nan"), dtype=torch.float64, device="cuda")
    ozimmu.dgemm(wide(A), wide(B), C[:, :n], s, ozimmu.alloc_workspace(m, n, k, s))
    got = C.cpu().numpy()
    assert np.isnan(got[:, n:]).all()
    return got[:, :n]


# tiles times steps: 1024 is the largest, those behind them are just beyond it (the general path); k = 129: four steps up to eight slices
SHAPES = [(1, 1, 1), (32, 32, 64), (33, 31, 63), (64, 64, 64), (31, 65, 65), (70, 40, 128), (5, 200, 3), (17, 1, 100), (33, 40, 129), (40, 33, 256),
          (1024, 1024, 2), (1025, 1023, 3), (511, 1024, 66), (513, 1024, 66), (500, 512, 130), (520, 512, 130)]


@pytest.mark.parametrize("s", range(1, 17))
@pytest.mark.parametrize("m,n,k", SHAPES)
def test_plain(m, n, k, s):
    A, B = wl.phi_pair(m, n, k, 1.0, seed=m + k + s)
    assert np.array_equal(bits(run(A, B, s, extra=s % 3)), bits(oracle.dgemm(A, B, s)))


@pytest.mark.parametrize("s", range(1, 17))
@pytest.mark.parametrize("m,n,k", [(33, 31, 63), (40, 70, 128), (20, 33, 200)])
def test_double_double(m, n, k, s):
    A, B = wl.phi_pair(m, n, k, 0.5, seed=m + k + s)
    hi = torch.full((m, n), float("nan"), dtype=torch.float64, device="cuda")
    lo = torch.full_like(hi, float("nan"))
    ozimmu.dgemm_dd(dev(A), dev(B), hi, lo, s, ozimmu.alloc_workspace(m, n, k, s))
    hi_want, lo_want = oracle.dgemm_dd(A, B, s)
    assert np.array_equal(bits(hi.cpu().numpy()), bits(hi_want)) and np.array_equal(bits(lo.cpu().numpy()), bits(lo_want))


@pytest.mark.parametrize("s", [3, 8, 9, 10, 16])
def test_adversarial_values(s):
    rng = np.random.default_rng(s)
    m, n, k = 40, 50, 90 if s != 8 else 200
    A = np.ldexp(rng.standard_normal((m, k)), rng.integers(-60, 60, (m, k)))
    B = np.ldexp(rng.standard_normal((k, n)), rng.integers(-60, 60, (k, n)))
    A[3] = 0.0                                   # a row and a column of zeros, signed ones among them
    A[4] = -0.0
    B[:, 7] = 0.0
    A[5] = np.ldexp(rng.standard_normal(k), -1060)        # subnormal rows and columns
    A[6] = 0.0
    A[6, 11] = 5e-324
    B[:, 9] = np.ldexp(rng.standard_normal(k), -1050)
    A[8] = np.finfo(np.float64).max              # the largest exponent; exact powers of two; the largest slices
    A[9] = 2.0 ** 40
    A[10] = 1.0 - 2.0 ** -53
    B[:, 12] = -(1.0 - 2.0 ** -53)
    B[:, 13] = np.ldexp(B[:, 13], -900)
    assert np.array_equal(bits(run(A, B, s)), bits(oracle.dgemm(A, B, s)))


@pytest.mark.parametrize("transa", "NT")
@pytest.mark.parametrize("transb", "NT")
@pytest.mark.parametrize("alpha,beta", [(1.0, 0.0), (0.5, 1.0), (-1.25, -0.75)])
@pytest.mark.parametrize("m,n,k,s", [(45, 70, 37, 6), (33, 20, 128, 11), (20, 33, 150, 7)])
def test_blas_form(transa, transb, alpha, beta, m, n, k, s):
    ta, tb = transa == "T", transb == "T"
    A, B = wl.phi_pair(m, n, k, 1.0, seed=m + s)   # op(A), op(B)
    C = wl.phi_matrix(m, n, 1.0, 5)
    pad = 3

    def column_major(x):   # as a wider row-major array of its transpose
        y = np.full((x.shape[1], x.shape[0] + pad), np.nan)
        y[:, : x.shape[0]] = x.T
        return dev(y), x.shape[0] + pad

    (dA, lda), (dB, ldb) = column_major(A.T if ta else A), column_major(B.T if tb else B)
    dC, ldc = column_major(C if beta else np.full_like(C, np.nan))
    ozimmu.dgemm_blas(transa, transb, m, n, k, alpha, dA, lda, dB, ldb, beta, dC, ldc, s, ozimmu.alloc_workspace(n, m, k, s))
    got = dC.cpu().numpy()
    want = oracle.dgemm_blas(ta, tb, alpha, A.T if ta else A, B.T if tb else B, beta, C, s)
    assert np.array_equal(bits(got[:, :m].T), bits(want)) and np.isnan(got[:, m:]).all()


# complex: up to 256 tiles; (1, 64, 64): a small register's gate; k = 65: two steps up to eight slices, the other kernels beyond
@pytest.mark.parametrize("s", range(1, 17))
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (32, 32, 64), (33, 31, 63), (1024, 64, 64), (5, 40, 3), (40, 70, 65), (33, 20, 128), (512, 512, 5), (515, 512, 5),
                                   (500, 510, 70)])
def test_complex(m, n, k, s):
    rng = np.random.default_rng(m + k + s)
    A = rng.standard_normal((m, k)) + 1j * rng.standard_normal((m, k))
    B = rng.standard_normal((k, n)) + 1j * rng.standard_normal((k, n))
    A[m // 2] = 0.0
    A[m - 1, k - 1] = 3e-310 - 5e-324j
    B[:, 0] = B[:, 0].real
    pad = s % 3
    dA, dC = torch.zeros((m, k + pad), dtype=torch.complex128, device="cuda"), torch.full((m, n + pad), float("nan"), dtype=torch.complex128, device="cuda")
    dA[:, :k] = dev(A)
    ozimmu.zgemm(dA[:, :k], dev(B), dC[:, :n], s, ozimmu.alloc_workspace(m, n, k, s, True))
    got = dC.cpu().numpy()
    assert np.array_equal(bits(got[:, :n]), bits(oracle.zgemm(A, B, s))) and np.isnan(got[:, n:]).all()


# the choice checked from the counts per tile: right, wrong and extreme guesses, several tiles of rows and of columns
@pytest.mark.parametrize("cplx,m,n,k", [(False, 100, 70, 50), (False, 33, 300, 128), (False, 40, 33, 200), (False, 1, 1, 1), (True, 100, 70, 50), (True, 1024, 64, 64),
                                        (True, 40, 33, 100), (True, 3, 2, 1)])
def test_guess_is_checked_from_the_counts_of_the_tiles(cplx, m, n, k):
    A, B = (wl.gaussian_complex(m, k, 5), wl.gaussian_complex(k, n, 6)) if cplx else wl.phi_pair(m, n, k, 1.0, seed=4)
    A[m // 2] = 0.0
    dA, dB = dev(A), dev(B)
    auto, product = (ozimmu.zgemm_auto, oracle.zgemm) if cplx else (ozimmu.dgemm_auto, oracle.dgemm)
    for T in (0.0, 1.0, 3.0):
        right, _ = oracle.auto_num_slices(A, B, T)
        want = product(A, B, right)
        for guess in {max(1, right - 1), right, min(16, right + 1), 1, 16}:
            C = torch.full((m, n), float("nan"), dtype=dA.dtype, device="cuda")
            got, confirmed = auto(dA, dB, C, T, guess=guess)
            assert got == right and confirmed == (guess == right), (T, guess)
            assert np.array_equal(bits(C.cpu().numpy()), bits(want))


# the complex BLAS-style call of plain operands, with scalars (held beside C, then combined) and without
@pytest.mark.parametrize("alpha,beta", [(1.0, 0.0), (0.5 - 2.0j, 0.0), (1.5j, -0.75 + 1.0j)])
@pytest.mark.parametrize("m,n,k,s", [(20, 45, 33, 8), (40, 33, 100, 5), (33, 70, 64, 11)])
def test_complex_blas_form(m, n, k, s, alpha, beta):
    A, B, C = wl.gaussian_complex(m, k, 1), wl.gaussian_complex(k, n, 2), wl.gaussian_complex(m, n, 3)
    dA, dB, dC = dev(A.T), dev(B.T), dev(C.T if beta else np.full((n, m), np.nan + 0j))   # column-major as row-major transposes
    ws = torch.empty(ozimmu.zgemm_blas_workspace_bytes(m, n, k, s, beta == 0), dtype=torch.uint8, device="cuda")
    ozimmu.zgemm_blas("N", "N", m, n, k, alpha, dA, m, dB, k, beta, dC, m, s, ws)
    want = oracle.zgemm_blas("N", "N", alpha, A, B, beta, C, s)
    assert np.array_equal(bits(dC.cpu().numpy().T), bits(want))
