"""The launch that splits both operands of a product (short vectors): every way the operands can be stored, at the edges of the
register tiling and beyond them, against the oracle bit for bit; the counts it takes on the way for the slice-count check. (Products of few tiles
with short vectors are one kernel's, test_gpu_small_product.py: with the smallest shapes here that one runs.)"""
import numpy as np
import pytest
import torch

import oracle
from paper_2306_11975_amd import ozimmu
from paper_2306_11975_amd import workloads as wl

pytestmark = pytest.mark.gpu


def bits(x):
    return np.ascontiguousarray(x).view(np.uint64)


def stored(M, pad, odd):
    """M as the left part of a wider device array (leading dimension odd or even), base 16-byte aligned or 8 bytes off."""
    r, c = M.shape
    buf = torch.full((r, c + pad + odd), float("nan"), dtype=torch.complex128 if np.iscomplexobj(M) else torch.float64, device="cuda")
    view = buf[:, odd:odd + c]
    view.copy_(torch.from_numpy(np.ascontiguousarray(M)))
    return view


@pytest.mark.parametrize("ta", [False, True])
@pytest.mark.parametrize("tb", [False, True])
@pytest.mark.parametrize("m,n,k,s", [(5, 17, 1, 3), (16, 33, 64, 9), (130, 70, 65, 10), (40, 20, 1024, 8), (40, 20, 1025, 12), (20, 50, 2048, 7),
                                     (20, 50, 2049, 7), (9, 4100, 40, 6), (300, 150, 130, 5)])
def test_real_operands_bit_exact(ta, tb, m, n, k, s):
    A, B = wl.phi_pair(m, n, k, 1.0, seed=k)
    A[0, :] = 0.0
    A[m - 1, k - 1] = 3.0e-310          # a subnormal maximum or element
    for pad, odd in ((0, 0), (3, 1)):
        dA, dB = stored(A if ta else A.T, pad, odd), stored(B if tb else B.T, pad, odd)   # column-major op() as row-major arrays
        C = torch.empty((n, m), dtype=torch.float64, device="cuda")
        ozimmu.dgemm_blas("T" if ta else "N", "T" if tb else "N", m, n, k, 1.0, dA, dA.stride(0) if dA.shape[0] > 1 else max(dA.shape[1], 1),
                          dB, dB.stride(0) if dB.shape[0] > 1 else max(dB.shape[1], 1), 0.0, C, m, s, ozimmu.alloc_workspace(n, m, k, s))
        torch.cuda.synchronize()
        assert np.array_equal(bits(C.cpu().numpy().T), bits(oracle.dgemm(A, B, s))), (pad, odd)


# the shortest vectors, with more tiles than the kernel for small products takes
@pytest.mark.parametrize("ta", [False, True])
@pytest.mark.parametrize("tb", [False, True])
@pytest.mark.parametrize("m,n,k,s", [(1030, 1060, 1, 3), (1060, 1030, 33, 7), (1030, 1060, 64, 9), (1030, 1060, 65, 10), (9, 33000, 40, 6), (520, 1040, 130, 5)])
def test_short_vectors_of_many_tiles(ta, tb, m, n, k, s):
    A, B = wl.phi_pair(m, n, k, 1.0, seed=k)
    A[0, :] = 0.0
    A[m - 1, k - 1] = 3.0e-310
    rows = np.r_[0:9] if m < 20 else np.r_[0:9, m // 2 - 2:m // 2 + 3, m - 9:m]
    want = oracle.dgemm(A[rows], B, s)
    for pad, odd in ((0, 0), (3, 1)):
        dA, dB = stored(A if ta else A.T, pad, odd), stored(B if tb else B.T, pad, odd)
        C = torch.full((n, m), float("nan"), dtype=torch.float64, device="cuda")
        ozimmu.dgemm_blas("T" if ta else "N", "T" if tb else "N", m, n, k, 1.0, dA, dA.stride(0) if dA.shape[0] > 1 else dA.shape[1],
                          dB, dB.stride(0) if dB.shape[0] > 1 else dB.shape[1], 0.0, C, m, s, ozimmu.alloc_workspace(n, m, k, s))
        torch.cuda.synchronize()
        got = C.cpu().numpy().T
        assert np.array_equal(bits(got[rows]), bits(want)) and not np.isnan(got).any(), (pad, odd)


@pytest.mark.parametrize("m,n,k", [(1030, 1060, 33), (520, 700, 200), (1060, 1030, 1)])
def test_guess_is_checked_from_the_counts_of_many_tiles(m, n, k):
    A, B = wl.phi_pair(m, n, k, 1.0, seed=4)
    A[3] = 0.0
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    rows = np.r_[0:9, m - 9:m]
    for T in (0.0, 1.0):
        right, _ = oracle.auto_num_slices(A, B, T)
        want = oracle.dgemm(A[rows], B, right)
        for guess in (right - 1, right, min(16, right + 1), 16):
            C = torch.empty((m, n), dtype=torch.float64, device="cuda")
            got, confirmed = ozimmu.dgemm_auto(dA, dB, C, T, guess=guess)
            torch.cuda.synchronize()
            assert got == right and confirmed == (guess == right)
            assert np.array_equal(bits(C.cpu().numpy()[rows]), bits(want))


@pytest.mark.parametrize("ta", ["N", "C"])
@pytest.mark.parametrize("tb", ["N", "T"])
@pytest.mark.parametrize("m,n,k,s", [(20, 300, 33, 8), (300, 260, 64, 11), (24, 40, 1024, 5), (24, 40, 1025, 5)])
def test_complex_operands_bit_exact(ta, tb, m, n, k, s):
    A, B = wl.gaussian_complex(m, k, 1), wl.gaussian_complex(k, n, 2)
    SA, SB = (A.conj() if ta == "C" else A.T), (B if tb == "T" else B.T)
    dA, dB = stored(SA, 2, 0), stored(SB, 1, 0)
    C = torch.empty((n, m), dtype=torch.complex128, device="cuda")
    ws = torch.empty(ozimmu.zgemm_blas_workspace_bytes(m, n, k, s, True), dtype=torch.uint8, device="cuda")
    ozimmu.zgemm_blas(ta, tb, m, n, k, 1.0, dA, dA.stride(0), dB, dB.stride(0), 0.0, C, m, s, ws)
    torch.cuda.synchronize()
    assert np.array_equal(bits(C.cpu().numpy().T.copy().view(np.float64)), bits(oracle.zgemm(A, B, s).view(np.float64)))


@pytest.mark.parametrize("cplx", [False, True])
@pytest.mark.parametrize("m,n,k", [(5, 7, 33), (300, 40, 200), (30, 500, 1024), (16, 16, 1100)])
def test_guess_is_checked_from_the_counts(cplx, m, n, k):
    A, B = (wl.gaussian_complex(m, k, 5), wl.gaussian_complex(k, n, 6)) if cplx else wl.phi_pair(m, n, k, 1.0, seed=4)
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    auto, product = (ozimmu.zgemm_auto, oracle.zgemm) if cplx else (ozimmu.dgemm_auto, oracle.dgemm)
    for T in (0.0, 1.0):
        right, _ = oracle.auto_num_slices(A, B, T)
        want = product(A, B, right)
        for guess in (right - 1, right, right + 1, 1, 16):
            C = torch.empty((m, n), dtype=dA.dtype, device="cuda")
            got, confirmed = auto(dA, dB, C, T, guess=guess)
            torch.cuda.synchronize()
            assert got == right and confirmed == (guess == right)
            assert np.array_equal(bits(C.cpu().numpy().view(np.float64)), bits(want.view(np.float64)))


# rows of 2^20 elements and more are read four words to a thread: beside columns by workgroups of sixteen rows (k up to 1024) and of eight,
# beside rows by one to eight wavefronts; rows aligned and not, numbers of rows that leave groups empty
@pytest.mark.parametrize("rows_too", [False, True])
@pytest.mark.parametrize("m,n,k,s", [(4097, 20, 257, 9), (4100, 40, 256, 3), (1300, 33, 1000, 10), (1025, 17, 1024, 4), (1030, 20, 1025, 5), (515, 50, 2047, 12)])
def test_long_rows_bit_exact(m, n, k, s, rows_too):
    A, B = wl.phi_pair(m, n, k, 1.0, seed=k)
    A[m // 2, :] = 0.0
    rows = np.r_[0:9, m // 2 - 2:m // 2 + 3, m - 9:m]
    want = oracle.dgemm(A[rows], B, s)
    for pad, odd in ((0, 0), (3, 1)):
        dA, dB = stored(A, pad, odd), stored(B.T if rows_too else B, pad, odd)
        C = torch.empty((n, m), dtype=torch.float64, device="cuda")
        ozimmu.dgemm_blas("T", "N" if rows_too else "T", m, n, k, 1.0, dA, dA.stride(0), dB, dB.stride(0), 0.0, C, m, s, ozimmu.alloc_workspace(n, m, k, s))
        torch.cuda.synchronize()
        assert np.array_equal(bits(C.cpu().numpy().T[rows]), bits(want)), (pad, odd)


# complex: four words up to nine slices, kernels of their own beyond
@pytest.mark.parametrize("m,n,k,s", [(5130, 140, 256, 8), (2050, 150, 700, 9), (1300, 200, 1024, 3), (2050, 150, 700, 10)])
def test_long_complex_rows_bit_exact(m, n, k, s):
    A, B = wl.gaussian_complex(m, k, 1), wl.gaussian_complex(k, n, 2)
    rows = np.r_[0:9, m - 9:m]
    C = torch.empty((m, n), dtype=torch.complex128, device="cuda")
    dA, dB = stored(A, 1, 0), stored(B, 2, 0)
    ozimmu.zgemm(dA, dB, C, s, ozimmu.alloc_workspace(m, n, k, s, True))
    torch.cuda.synchronize()
    assert np.array_equal(bits(C.cpu().numpy()[rows].view(np.float64)), bits(oracle.zgemm(A[rows], B, s).view(np.float64)))


@pytest.mark.parametrize("cplx,m,n,k", [(False, 4097, 20, 257), (False, 600, 30, 2000), (True, 1300, 150, 1024)])
def test_guess_is_checked_from_the_counts_of_long_rows(cplx, m, n, k):
    A, B = (wl.gaussian_complex(m, k, 5), wl.gaussian_complex(k, n, 6)) if cplx else wl.phi_pair(m, n, k, 1.0, seed=4)
    dA, dB = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    rows = np.r_[0:9, m - 9:m]
    right, _ = oracle.auto_num_slices(A, B, 1.0)
    want = (oracle.zgemm if cplx else oracle.dgemm)(A[rows], B, right)
    for guess in (right - 1, right, right + 1, 16):
        C = torch.empty((m, n), dtype=dA.dtype, device="cuda")
        got, confirmed = (ozimmu.zgemm_auto if cplx else ozimmu.dgemm_auto)(dA, dB, C, 1.0, guess=guess)
        torch.cuda.synchronize()
        assert got == right and confirmed == (guess == right)
        assert np.array_equal(bits(C.cpu().numpy()[rows].view(np.float64)), bits(want.view(np.float64)))
