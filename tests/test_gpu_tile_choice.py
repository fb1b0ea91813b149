"""Either side of the rule that picks 64 x 64 tiles by an estimate (more than one round of the larger ones, k > 512), and complex products
on both, against the oracle on sampled rows, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2306_11975_amd import ozimmu
from paper_2306_11975_amd import workloads as wl

pytestmark = pytest.mark.gpu


def bits(x):
    return np.ascontiguousarray(x).view(np.uint64)


def sampled(m):
    """A row of every 16: every fragment and, complex, every 32-row tile is among them, and the last."""
    rows = list(range(3, m, 16)) + [m - 1]
    return torch.tensor(sorted(set(rows)), device="cuda")


# just beyond one round of 64 x 128 tiles (257 .. 288 of them); two rounds of either; odd sizes, odd numbers of slabs; long walks of few slices
@pytest.mark.parametrize("m,n,k,s,cols", [(1030, 2050, 545, 9, 64), (1030, 2050, 545, 8, 64), (1601, 1409, 700, 3, 64), (2049, 1111, 513, 5, 64),
                                          (1024, 4096, 2300, 6, 128), (1024, 4096, 576, 6, 64), (1500, 1800, 1033, 7, 64), (2048, 2048, 4100, 7, 128),
                                          (899, 3001, 7814, 5, 128), (2535, 1020, 13160, 2, 128)])
def test_real_products_across_the_estimate(m, n, k, s, cols):
    assert ozimmu.launch_plan(m, n, k, s)["tile_cols"] == cols
    A, B = wl.phi_matrix_device(m, k, 1.0, 11), wl.phi_matrix_device(k, n, 1.0, 12)
    C = torch.full((m, n), float("nan"), dtype=torch.float64, device="cuda")
    ozimmu.dgemm(A, B, C, s, ozimmu.alloc_workspace(m, n, k, s))
    rows = sampled(m)[::4]
    want = oracle.dgemm(A[rows].cpu().numpy(), B.cpu().numpy(), s)
    assert not torch.isnan(C).any()
    assert np.array_equal(bits(C[rows].cpu().numpy()), bits(want))


# few of the larger tiles with three workgroups on each, ahead of the smaller ones with one; double-double and complex products on the same
@pytest.mark.parametrize("m,n,k,s", [(410, 1174, 3391, 13), (298, 1891, 4479, 11)])
def test_shared_larger_tiles(m, n, k, s):
    plan = ozimmu.launch_plan(m, n, k, s)
    assert plan["tile_cols"] == 128 and plan["workgroups"] > -(-m // 64) * -(-n // 128)
    A, B = wl.phi_matrix_device(m, k, 1.0, 11), wl.phi_matrix_device(k, n, 1.0, 12)
    hi, lo = (torch.full((m, n), float("nan"), dtype=torch.float64, device="cuda") for _ in range(2))
    ws = ozimmu.alloc_workspace(m, n, k, s)
    rows = sampled(m)[::2]
    a, b = A[rows].cpu().numpy(), B.cpu().numpy()
    ozimmu.dgemm(A, B, hi, s, ws)
    assert not torch.isnan(hi).any() and np.array_equal(bits(hi[rows].cpu().numpy()), bits(oracle.dgemm(a, b, s)))
    ozimmu.dgemm_dd(A, B, hi, lo, s, ws)
    want_hi, want_lo = oracle.dgemm_dd(a, b, s)
    assert np.array_equal(bits(hi[rows].cpu().numpy()), bits(want_hi)) and np.array_equal(bits(lo[rows].cpu().numpy()), bits(want_lo))
    # (a complex element is two real rows and columns)
    Z, W = wl.gaussian_complex_device(m // 2, k, 13), wl.gaussian_complex_device(k, n // 2, 14)
    C = torch.full((m // 2, n // 2), float("nan"), dtype=torch.complex128, device="cuda")
    ozimmu.zgemm(Z, W, C, s, ozimmu.alloc_workspace(m // 2, n // 2, k, s, True))
    rows = sampled(m // 2)[::2]
    assert not torch.isnan(C.real).any() and np.array_equal(bits(C[rows].cpu().numpy()), bits(oracle.zgemm(Z[rows].cpu().numpy(), W.cpu().numpy(), s)))


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
    return full[:hi]


@pytest.mark.parametrize("m,n,k,s", [(410, 1174, 3391, 13), (298, 1891, 4479, 11)])
def test_the_same_without_room_for_shared_walks(m, n, k, s):
    """The call's least workspace, which leaves no room for the sums of shared walks: the product is formed on the smaller tiles, with the same bits."""
    A, B = wl.phi_matrix_device(m, k, 1.0, 11), wl.phi_matrix_device(k, n, 1.0, 12)
    want_hi, want_lo, hi, lo = (torch.full((m, n), float("nan"), dtype=torch.float64, device="cuda") for _ in range(4))
    full = ozimmu.alloc_workspace(m, n, k, s)
    ozimmu.dgemm(A, B, want_hi, s, full)
    least = least_workspace(lambda ws: ozimmu.dgemm(A, B, hi, s, ws), full.numel())
    assert least.numel() < full.numel()
    ozimmu.dgemm(A, B, hi.fill_(float("nan")), s, least)
    assert torch.equal(hi, want_hi)
    ozimmu.dgemm_dd(A, B, want_hi, want_lo, s, full)
    ozimmu.dgemm_dd(A, B, hi, lo, s, least)
    assert torch.equal(hi, want_hi) and torch.equal(lo, want_lo)
    Z, W = wl.gaussian_complex_device(m // 2, k, 13), wl.gaussian_complex_device(k, n // 2, 14)
    want, C = (torch.full((m // 2, n // 2), float("nan"), dtype=torch.complex128, device="cuda") for _ in range(2))
    full = ozimmu.alloc_workspace(m // 2, n // 2, k, s, True)
    ozimmu.zgemm(Z, W, want, s, full)
    least = least_workspace(lambda ws: ozimmu.zgemm(Z, W, C, s, ws), full.numel())
    ozimmu.zgemm(Z, W, C.fill_(float("nan")), s, least)
    assert least.numel() < full.numel() and torch.equal(torch.view_as_real(C), torch.view_as_real(want))


# complex: 64 x 64 tiles hold 32 x 32 complex elements; more than 256 of the larger tiles each, so that k and the slice count decide
@pytest.mark.parametrize("m,n,k,s", [(520, 1030, 33, 1), (520, 1030, 100, 7), (511, 1057, 512, 9), (530, 1000, 700, 8), (515, 1030, 1600, 5), (520, 1030, 64, 10)])
def test_complex_products_on_small_and_large_tiles(m, n, k, s):
    A, B = wl.gaussian_complex_device(m, k, 21), wl.gaussian_complex_device(k, n, 22)
    C = torch.full((m, n + 2), float("nan"), dtype=torch.complex128, device="cuda")
    ozimmu.zgemm(A, B, C[:, :n], s, ozimmu.alloc_workspace(m, n, k, s, True))
    rows = sampled(m)
    want = oracle.zgemm(A[rows].cpu().numpy(), B.cpu().numpy(), s)
    got = C.cpu().numpy()
    assert np.array_equal(bits(got[rows.cpu().numpy()][:, :n]), bits(want))
    assert np.isnan(got[:, n:]).all() and not np.isnan(got[:, :n]).any()
