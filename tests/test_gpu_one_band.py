"""9 and 11 to 15 slices on 64 x 64 tiles with one workgroup to a compute unit, whose diagonals are all walked in one band: real, double-double
and complex products against the oracle, bit for bit; and 11 to 13 on 64 x 128 tiles, where those fill their rounds."""
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


# one slab, one step, a step and a slab, three slabs, an odd and an even number of slabs that fill the pipeline
SIZES = [(64, 64, 1), (65, 63, 64), (1, 130, 65), (129, 66, 96), (70, 200, 1000), (64, 128, 513)]


@pytest.mark.parametrize("s", [9, 11, 12, 13, 14, 15])
@pytest.mark.parametrize("m,n,k", SIZES)
def test_real(m, n, k, s):
    """By stages: the call itself takes another kernel where k is short."""
    assert ozimmu.launch_plan(m, n, k, s)["bands"] == 1
    A, B = wl.phi_pair(m, n, k, 1.0, seed=k + s)
    dA, dB = dev(A), dev(B)
    C = torch.full((m, n), float("nan"), dtype=torch.float64, device="cuda")
    ws = ozimmu.alloc_workspace(m, n, k, s)
    for stage in range(3):
        ozimmu.dgemm_stage(stage, dA, dB, C, s, ws)
    assert np.array_equal(bits(C.cpu().numpy()), bits(oracle.dgemm(A, B, s)))


# (1030 x 1030: more tiles than the kernel for small products takes, so that the shortest walks are reached)
@pytest.mark.parametrize("s", [11, 12, 13, 14, 15])
@pytest.mark.parametrize("m,n,k", [(1030, 1030, 20), (1030, 1030, 64), (1030, 1030, 90), (70, 200, 1000), (64, 128, 513), (129, 66, 300)])
def test_double_double(m, n, k, s):
    A, B = wl.phi_matrix_device(m, k, 1.0, k + s), wl.phi_matrix_device(k, n, 1.0, k + s + 1)
    C = torch.full((m, n), float("nan"), dtype=torch.float64, device="cuda")
    lo = torch.full_like(C, float("nan"))
    ozimmu.dgemm_dd(A, B, C, lo, s, ozimmu.alloc_workspace(m, n, k, s))
    rows = torch.arange(0, m, 1 + m // 40, device="cuda")
    hi_want, lo_want = oracle.dgemm_dd(A[rows].cpu().numpy(), B.cpu().numpy(), s)
    assert np.array_equal(bits(C[rows].cpu().numpy()), bits(hi_want)) and np.array_equal(bits(lo[rows].cpu().numpy()), bits(lo_want))
    assert not torch.isnan(C).any()


@pytest.mark.parametrize("s", [9, 11, 12, 13, 14, 15])
@pytest.mark.parametrize("m,n,k", [(33, 200, 129), (64, 140, 1000)])
def test_complex(m, n, k, s):
    rng = np.random.default_rng(s + k)
    A = rng.standard_normal((m, k)) + 1j * rng.standard_normal((m, k))
    B = rng.standard_normal((k, n)) + 1j * rng.standard_normal((k, n))
    C = torch.full((m, n), float("nan"), dtype=torch.complex128, device="cuda")
    ozimmu.zgemm(dev(A), dev(B), C, s, ozimmu.alloc_workspace(m, n, k, s, True))
    assert np.array_equal(bits(C.cpu().numpy()), bits(oracle.zgemm(A, B, s)))


@pytest.mark.parametrize("s", [9, 11, 15])
def test_largest_sums(s):
    """Every slice at its largest: the sums of all diagonals at once, up to the INT32 block's end."""
    k = ozimmu.INT32_BLOCK // s // 64 * 64
    A = np.full((3, k), 1.0 - 2.0 ** -53)
    B = np.full((k, 70), 1.0 - 2.0 ** -53)
    C = torch.full((3, 70), float("nan"), dtype=torch.float64, device="cuda")
    ozimmu.dgemm(dev(A), dev(B), C, s, ozimmu.alloc_workspace(3, 70, k, s))
    assert np.array_equal(bits(C.cpu().numpy()), bits(oracle.dgemm(A, B, s)))


# 256 tiles of 64 x 128: one round of them, two of the smaller ones
@pytest.mark.parametrize("s", [11, 12, 13])
@pytest.mark.parametrize("k", [97, 128])
def test_large_tiles(k, s):
    m, n = 1024, 2048
    assert ozimmu.launch_plan(m, n, k, s)["tile_cols"] == 128
    A, B = wl.phi_matrix_device(m, k, 1.0, 31), wl.phi_matrix_device(k, n, 1.0, 32)
    C = torch.full((m, n), float("nan"), dtype=torch.float64, device="cuda")
    lo = torch.full_like(C, float("nan"))
    rows = torch.arange(5, m, 48, device="cuda")
    a, b = A[rows].cpu().numpy(), B.cpu().numpy()
    ozimmu.dgemm(A, B, C, s, ozimmu.alloc_workspace(m, n, k, s))
    assert np.array_equal(bits(C[rows].cpu().numpy()), bits(oracle.dgemm(a, b, s)))
    ozimmu.dgemm_dd(A, B, C, lo, s, ozimmu.alloc_workspace(m, n, k, s))
    hi_want, lo_want = oracle.dgemm_dd(a, b, s)
    assert np.array_equal(bits(C[rows].cpu().numpy()), bits(hi_want)) and np.array_equal(bits(lo[rows].cpu().numpy()), bits(lo_want))
    assert not torch.isnan(C).any()
    Z = wl.gaussian_complex_device(m // 2, k, 33)
    W = wl.gaussian_complex_device(k, n // 2, 34)
    D = torch.full((m // 2, n // 2), float("nan"), dtype=torch.complex128, device="cuda")
    ozimmu.zgemm(Z, W, D, s, ozimmu.alloc_workspace(m // 2, n // 2, k, s, True))
    half = rows[rows < m // 2]
    assert np.array_equal(bits(D[half].cpu().numpy()), bits(oracle.zgemm(Z[half].cpu().numpy(), W.cpu().numpy(), s)))
    assert not torch.isnan(D).any()
