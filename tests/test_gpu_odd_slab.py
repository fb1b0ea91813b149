"""Products whose k is an odd number of slabs of 32 positions, with nine slices and more: the kernel that takes the last slab
ahead of its steps, two pairs of a diagonal to an MFMA (nine slices: with more small tiles than compute units). Every such slice
count, one slab and more, ragged edges of k and of the
tiles, in every form of the product, against the oracle bit for bit. Products of up to 1024 tiles of 32 x 32 with so short a k are one kernel's
(test_gpu_small_product.py); the smaller shapes here run that one, the larger ones the kernel described."""
import numpy as np
import pytest
import torch

import oracle
from paper_2306_11975_amd import ozimmu
from paper_2306_11975_amd import workloads as wl

pytestmark = pytest.mark.gpu
SLICES = range(9, 17)


def bits(x):
    return np.ascontiguousarray(x).view(np.uint64)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def nan(m, n, dtype=torch.float64):
    return torch.full((m, n), float("nan"), dtype=dtype, device="cuda")


# one slab (no step at all), three, five, and 33 with enough tiles that no walk is shared
@pytest.mark.parametrize("s", SLICES)
@pytest.mark.parametrize("m,n,k", [(70, 140, 1), (130, 70, 32), (70, 140, 65), (64, 128, 96), (129, 257, 131), (1100, 1000, 30), (1060, 1030, 90), (1100, 1000, 1027), (1100, 2100, 1056)])
def test_dgemm(m, n, k, s):
    A, B = wl.phi_pair(m, n, k, 1.0, seed=k + s)
    C = nan(m, n + 3)
    ozimmu.dgemm(dev(A), dev(B), C[:, :n], s, ozimmu.alloc_workspace(m, n, k, s))
    torch.cuda.synchronize()
    out = C.cpu().numpy()
    rows = np.arange(m) if m < 200 else np.r_[0:20, 500:520, m - 20:m]
    assert np.array_equal(bits(out[rows, :n]), bits(oracle.dgemm(A[rows], B, s)))
    assert np.isnan(out[:, n:]).all()


@pytest.mark.parametrize("s", SLICES)
@pytest.mark.parametrize("k", [20, 96])
def test_saturating_slices(s, k):
    # every slice at +-127: each pair counted once, no more and no less
    A, B = wl.saturating_matrix(40, k), wl.saturating_matrix(k, 50)
    C = nan(40, 50)
    ozimmu.dgemm(dev(A), dev(B), C, s, ozimmu.alloc_workspace(40, 50, k, s))
    torch.cuda.synchronize()
    assert np.array_equal(bits(C.cpu().numpy()), bits(oracle.dgemm(A, B, s)))


# more tiles than the kernel for small products takes: every pair of the head counted once, rows of one tile and of the last
@pytest.mark.parametrize("s", SLICES)
@pytest.mark.parametrize("k", [20, 96])
def test_saturating_slices_of_many_tiles(s, k):
    m, n = 1030, 1040
    A, B = wl.saturating_matrix(m, k), wl.saturating_matrix(k, n)
    C = nan(m, n)
    ozimmu.dgemm(dev(A), dev(B), C, s, ozimmu.alloc_workspace(m, n, k, s))
    torch.cuda.synchronize()
    rows = np.r_[0:4, 62:66, m - 4:m]
    out = C.cpu().numpy()
    assert np.array_equal(bits(out[rows]), bits(oracle.dgemm(A[rows], B, s))) and not np.isnan(out).any()


@pytest.mark.parametrize("s", SLICES)
@pytest.mark.parametrize("k", [31, 90])
def test_other_forms_of_many_tiles(s, k):
    m, n = 1030, 1040
    rows = np.r_[0:20, 500:520, m - 20:m]
    A, B = wl.phi_pair(m, n, k, 1.0, seed=s)
    dA, dB = dev(A), dev(B)
    hi, lo = nan(m, n), nan(m, n)
    ozimmu.dgemm_dd(dA, dB, hi, lo, s, ozimmu.alloc_workspace(m, n, k, s))
    torch.cuda.synchronize()
    whi, wlo = oracle.dgemm_dd(A[rows], B, s)
    assert np.array_equal(bits(hi.cpu().numpy()[rows]), bits(whi)) and np.array_equal(bits(lo.cpu().numpy()[rows]), bits(wlo))

    C0 = np.random.default_rng(s).standard_normal((m, n))
    dC = dev(C0.T)
    ozimmu.dgemm_blas("N", "N", m, n, k, 0.5, dev(A.T), m, dev(B.T), k, -0.75, dC, m, s, ozimmu.alloc_workspace(n, m, k, s))
    torch.cuda.synchronize()
    assert np.array_equal(bits(dC.cpu().numpy().T[rows]), bits(oracle.dgemm_blas(False, False, 0.5, A[rows], B, -0.75, C0[rows], s)))


@pytest.mark.parametrize("s", SLICES)
@pytest.mark.parametrize("k", [31, 90])
def test_other_forms(s, k):
    m, n = 70, 90
    A, B = wl.phi_pair(m, n, k, 1.0, seed=s)
    hi, lo = nan(m, n), nan(m, n)
    ozimmu.dgemm_dd(dev(A), dev(B), hi, lo, s, ozimmu.alloc_workspace(m, n, k, s))
    torch.cuda.synchronize()
    whi, wlo = oracle.dgemm_dd(A, B, s)
    assert np.array_equal(bits(hi.cpu().numpy()), bits(whi)) and np.array_equal(bits(lo.cpu().numpy()), bits(wlo))

    C0 = np.random.default_rng(s).standard_normal((m, n))
    dC = dev(C0.T)
    ozimmu.dgemm_blas("N", "N", m, n, k, 0.5, dev(A.T), m, dev(B.T), k, -0.75, dC, m, s, ozimmu.alloc_workspace(n, m, k, s))
    torch.cuda.synchronize()
    assert np.array_equal(bits(dC.cpu().numpy().T), bits(oracle.dgemm_blas(False, False, 0.5, A, B, -0.75, C0, s)))

    A, B = wl.gaussian_complex(m, k, 1), wl.gaussian_complex(k, 140, 2)      # 140 columns: more than the gate kernel takes
    C = nan(m, 140, torch.complex128)
    ozimmu.zgemm(dev(A), dev(B), C, s, ozimmu.alloc_workspace(m, 140, k, s, True))
    torch.cuda.synchronize()
    assert np.array_equal(bits(C.cpu().numpy().view(np.float64)), bits(oracle.zgemm(A, B, s).view(np.float64)))
