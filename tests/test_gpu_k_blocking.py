"""Products beyond the INT32 block (num_slices * k_padded > 2^17) whose workgroups each walk the whole of k: the INT32 sums are
moved into INT64 sums in the workspace every 2^17 products. That is how every such product runs that has as many tiles as there
are compute units; one with fewer tiles does so with a workspace that holds no more than the call insists on (otherwise its walk
is shared, and every part of it fits the INT32 sums). Against the oracle, bit for bit."""
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


def least_workspace(call, reported):
    """A workspace of the smallest size that call(workspace) accepts (smaller ones are refused on the host)."""
    full = torch.empty(reported, dtype=torch.uint8, device="cuda")
    lo, hi = 0, reported
    while hi - lo > 256:
        mid = (lo + hi) // 2
        try:
            call(full[:mid])
            hi = mid
        except ozimmu.OzimmuError as e:
            assert e.code == ozimmu.ERR_WORKSPACE
            lo = mid
    torch.cuda.synchronize()
    assert reported - hi > 256 * 1024      # the shapes below have few tiles: room for shared walks is reported
    return full[:hi]


def assert_blocked(k, s):
    assert s * ozimmu.slice_geometry(1, k)[1] > ozimmu.INT32_BLOCK


# one band (up to eight slices, fourteen and fifteen) and two, both tile shapes, even and odd numbers of slabs of 32 positions
@pytest.mark.parametrize("m,n,k,s", [(40, 50, 70000, 2), (40, 50, 69970, 2), (129, 65, 20000, 8), (65, 130, 14000, 10), (70, 140, 13001, 13),
                                     (70, 66, 9000, 16), (70, 66, 9025, 15),
                                     (66, 70, 9450, 14), (66, 70, 9500, 14)])
def test_dgemm(m, n, k, s):
    assert_blocked(k, s)
    A, B = wl.phi_pair(m, n, k, 2.0, seed=k)
    dA, dB = dev(A), dev(B)
    C = torch.empty((m, n), dtype=torch.float64, device="cuda")
    ws = least_workspace(lambda w: ozimmu.dgemm(dA, dB, C, s, w), ozimmu.workspace_bytes(m, n, k, s))
    C.fill_(float("nan"))
    ozimmu.dgemm(dA, dB, C, s, ws)
    torch.cuda.synchronize()
    assert np.array_equal(bits(C.cpu().numpy()), bits(oracle.dgemm(A, B, s)))


@pytest.mark.parametrize("s", [3, 16])
def test_saturating_slices_across_the_block(s):
    # a single INT32 sum would overflow
    k = ozimmu.INT32_BLOCK + 640
    A, B = wl.saturating_matrix(2, k), wl.saturating_matrix(k, 2)
    dA, dB = dev(A), dev(B)
    C = torch.empty((2, 2), dtype=torch.float64, device="cuda")
    ws = least_workspace(lambda w: ozimmu.dgemm(dA, dB, C, s, w), ozimmu.workspace_bytes(2, 2, k, s))
    C.fill_(float("nan"))
    ozimmu.dgemm(dA, dB, C, s, ws)
    torch.cuda.synchronize()
    assert np.array_equal(bits(C.cpu().numpy()), bits(oracle.dgemm(A, B, s)))


@pytest.mark.parametrize("m,n,k,s", [(40, 50, 70000, 3), (50, 70, 69970, 3), (64, 120, 14000, 12), (66, 70, 9000, 16),
                                     (64, 70, 9450, 14), (66, 70, 9500, 14), (66, 70, 8830, 15), (50, 60, 8800, 15)])
def test_double_double(m, n, k, s):
    assert_blocked(k, s)
    A, B = wl.phi_pair(m, n, k, 1.0, seed=9)
    dA, dB = dev(A), dev(B)
    hi, lo = (torch.empty((m, n), dtype=torch.float64, device="cuda") for _ in range(2))
    ws = least_workspace(lambda w: ozimmu.dgemm_dd(dA, dB, hi, lo, s, w), ozimmu.workspace_bytes(m, n, k, s))
    hi.fill_(float("nan"))
    lo.fill_(float("nan"))
    ozimmu.dgemm_dd(dA, dB, hi, lo, s, ws)
    torch.cuda.synchronize()
    whi, wlo = oracle.dgemm_dd(A, B, s)
    assert np.array_equal(bits(hi.cpu().numpy()), bits(whi)) and np.array_equal(bits(lo.cpu().numpy()), bits(wlo))


@pytest.mark.parametrize("alpha,beta", [(0.5, 0.0), (1.0, 1.0), (1.7, -0.75)])
@pytest.mark.parametrize("m,n,k,s", [(90, 50, 33000, 4), (50, 90, 13990, 10)])
def test_blas_update(m, n, k, s, alpha, beta):
    assert_blocked(k, s)
    rng = np.random.default_rng(5)
    A, B, C0 = rng.standard_normal((m, k)), rng.standard_normal((k, n)), rng.standard_normal((m, n))
    dA, dB = dev(A.T), dev(B.T)
    dC = torch.empty((n, m), dtype=torch.float64, device="cuda")

    def call(w):
        ozimmu.dgemm_blas("N", "N", m, n, k, alpha, dA, m, dB, k, beta, dC, m, s, w)

    ws = least_workspace(call, ozimmu.workspace_bytes(n, m, k, s))
    dC.copy_(dev(C0.T) if beta else torch.full((n, m), float("nan"), dtype=torch.float64))
    call(ws)
    torch.cuda.synchronize()
    assert np.array_equal(bits(dC.cpu().numpy().T), bits(oracle.dgemm_blas(False, False, alpha, A, B, beta, C0, s)))


# four launches of the real kernel: real part, its second product subtracted, imaginary part, its second product added and C written
@pytest.mark.parametrize("m,n,k,s", [(20, 30, 70000, 2), (33, 40, 13990, 11), (30, 20, 9000, 16)])
def test_zgemm(m, n, k, s):
    assert_blocked(k, s)
    A, B = wl.gaussian_complex(m, k, 3), wl.gaussian_complex(k, n, 4)
    dA, dB = dev(A), dev(B)
    C = torch.empty((m, n), dtype=torch.complex128, device="cuda")
    ws = least_workspace(lambda w: ozimmu.zgemm(dA, dB, C, s, w), ozimmu.workspace_bytes(m, n, k, s, True))
    C.fill_(complex("nan"))
    ozimmu.zgemm(dA, dB, C, s, ws)
    torch.cuda.synchronize()
    assert np.array_equal(bits(C.cpu().numpy().view(np.float64)), bits(oracle.zgemm(A, B, s).view(np.float64)))


@pytest.mark.parametrize("beta", [0.0, 0.25 + 1.0j])
def test_complex_blas_update(beta):
    m, n, k, s, alpha = 30, 20, 33000, 4, 1.25 - 0.5j
    assert_blocked(k, s)
    A, B, C0 = wl.gaussian_complex(k, m, 3), wl.gaussian_complex(k, n, 4), wl.gaussian_complex(m, n, 5)
    dA, dB = dev(A.T), dev(B.T)     # column-major: A is k x m and enters conjugated and transposed
    dC = torch.empty((n, m), dtype=torch.complex128, device="cuda")

    def call(w):
        ozimmu.zgemm_blas("C", "N", m, n, k, alpha, dA, k, dB, k, beta, dC, m, s, w)

    ws = least_workspace(call, ozimmu.zgemm_blas_workspace_bytes(m, n, k, s, beta == 0))
    dC.copy_(dev(C0.T) if beta else torch.full((n, m), complex("nan"), dtype=torch.complex128))
    call(ws)
    torch.cuda.synchronize()
    want = oracle.zgemm_blas("C", "N", alpha, A, B, beta, C0, s)
    assert np.array_equal(bits(dC.cpu().numpy().T.copy().view(np.float64)), bits(want.copy().view(np.float64)))
