"""Products whose tiles are walked by several workgroups, each with a part of k (few tiles, long k), and the walk's step of
64 positions at its edges: against the oracle, bit for bit (integer sums are exact in any order and the FP64 sum has one order)."""
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


def smallest_workspace(m, n, k, s, cplx, A, B, C):
    """The smallest size the call accepts (too small ones are refused on the host, before anything is launched)."""
    full = ozimmu.alloc_workspace(m, n, k, s, cplx)
    call = ozimmu.zgemm if cplx else ozimmu.dgemm
    lo, hi = 0, full.numel()
    while hi - lo > 256:
        mid = (lo + hi) // 2
        try:
            call(A, B, C, s, full[:mid])
            hi = mid
        except ozimmu.OzimmuError as e:
            assert e.code == ozimmu.ERR_WORKSPACE
            lo = mid
    torch.cuda.synchronize()
    return full, hi


# k = 1024: the fewest steps that are shared; odd numbers of slabs, a last part shorter than the others, one step in it;
# one and two bands; both tile shapes; beyond the INT32 block
@pytest.mark.parametrize("m,n,k,s", [(64, 64, 1024, 8), (35, 154, 2251, 9), (100, 300, 1057, 3), (130, 70, 5000, 6), (33, 200, 1500, 10),
                                     (70, 140, 2100, 13), (64, 64, 3000, 16), (129, 65, 40000, 5), (1, 1, 4100, 1)])
def test_dgemm_shared_walk_bit_exact(m, n, k, s):
    A, B = wl.phi_pair(m, n, k, 1.0, seed=k + s)
    dA, dB = dev(A), dev(B)
    C = torch.full((m, n + 3), float("nan"), dtype=torch.float64, device="cuda")
    full, least = smallest_workspace(m, n, k, s, False, dA, dB, C[:, :n])
    assert least <= full.numel()     # room for the parts' sums is reported, and not asked for
    if k >= 2000:
        assert least + 2 * 4 * s * m * n <= full.numel()
    want = oracle.dgemm(A, B, s)
    for ws in (full, full[:least]):
        C[:, :n] = float("nan")
        ozimmu.dgemm(dA, dB, C[:, :n], s, ws)
        torch.cuda.synchronize()
        out = C.cpu().numpy()
        assert np.array_equal(bits(out[:, :n]), bits(want))
        assert np.isnan(out[:, n:]).all()


@pytest.mark.parametrize("m,n,k,s", [(40, 50, 1300, 7), (33, 100, 2049, 8), (64, 64, 1024, 11), (20, 30, 3000, 16)])
def test_zgemm_shared_walk_bit_exact(m, n, k, s):
    A, B = wl.gaussian_complex(m, k, 3), wl.gaussian_complex(k, n, 4)
    dA, dB = dev(A), dev(B)
    C = torch.full((m, n), complex("nan"), dtype=torch.complex128, device="cuda")
    full, least = smallest_workspace(m, n, k, s, True, dA, dB, C)
    assert least <= full.numel()
    want = oracle.zgemm(A, B, s)
    for ws in (full, full[:least]):
        C.fill_(complex("nan"))
        ozimmu.zgemm(dA, dB, C, s, ws)
        torch.cuda.synchronize()
        assert np.array_equal(bits(C.cpu().numpy().view(np.float64)), bits(want.view(np.float64)))


@pytest.mark.parametrize("m,n,k,s", [(64, 64, 1024, 12), (153, 207, 2131, 13), (40, 50, 70000, 3), (50, 60, 1500, 16)])
def test_double_double_shared_walk_bit_exact(m, n, k, s):
    A, B = wl.phi_pair(m, n, k, 1.0, seed=9)
    hi, lo = (torch.full((m, n), float("nan"), dtype=torch.float64, device="cuda") for _ in range(2))
    ozimmu.dgemm_dd(dev(A), dev(B), hi, lo, s, ozimmu.alloc_workspace(m, n, k, s))
    torch.cuda.synchronize()
    whi, wlo = oracle.dgemm_dd(A, B, s)
    assert np.array_equal(bits(hi.cpu().numpy()), bits(whi)) and np.array_equal(bits(lo.cpu().numpy()), bits(wlo))


@pytest.mark.parametrize("beta", [0.0, 1.0, -0.75])
def test_blas_update_shared_walk_bit_exact(beta):
    m, n, k, s = 50, 90, 1999, 7
    rng = np.random.default_rng(5)
    A, B, C = rng.standard_normal((m, k)), rng.standard_normal((k, n)), rng.standard_normal((m, n))
    dC = dev(C.T) if beta else torch.full((n, m), float("nan"), dtype=torch.float64, device="cuda")
    ozimmu.dgemm_blas("N", "N", m, n, k, 0.5, dev(A.T), m, dev(B.T), k, beta, dC, m, s, ozimmu.alloc_workspace(n, m, k, s))
    torch.cuda.synchronize()
    assert np.array_equal(bits(dC.cpu().numpy().T), bits(oracle.dgemm_blas(False, False, 0.5, A, B, beta, C, s)))


def test_static_scratch_takes_what_its_size_allows():
    # at the limit of the built-in scratch the room for the parts' sums shrinks, and nothing is refused that fits without it
    m, n, k, s = 64, 64, 250000, 1
    assert 2 * 128 * k < ozimmu.workspace_bytes(m, n, k, s) <= ozimmu.STATIC_SCRATCH_BYTES
    A, B = wl.phi_pair(m, n, k, 0.5, seed=2)
    C = torch.empty((m, n), dtype=torch.float64, device="cuda")
    ozimmu.dgemm_static(dev(A), dev(B), C, s)
    torch.cuda.synchronize()
    assert np.array_equal(bits(C.cpu().numpy()), bits(oracle.dgemm(A, B, s)))


# one workgroup per compute unit and two; one slab, two, three; every slice count of the small tiles
@pytest.mark.parametrize("s", range(1, 10))
@pytest.mark.parametrize("m,n", [(65, 130), (1040, 1040)])
def test_few_and_many_small_tiles_bit_exact(m, n, s):
    for k in (31, 33, 65, 100):
        A, B = wl.phi_pair(m, n, k, 1.0, seed=s)
        C = torch.empty((m, n), dtype=torch.float64, device="cuda")
        ozimmu.dgemm(dev(A), dev(B), C, s, ozimmu.alloc_workspace(m, n, k, s))
        torch.cuda.synchronize()
        rows = np.r_[0:40, m - 30:m]
        assert np.array_equal(bits(C.cpu().numpy()[rows]), bits(oracle.dgemm(A[rows], B, s))), k


@pytest.mark.parametrize("m,n,k,s", [(700, 700, 96, 8), (700, 700, 96, 9), (600, 600, 33, 12), (40, 1000, 200, 15)])
def test_zgemm_tiles_of_both_planes_bit_exact(m, n, k, s):
    A, B = wl.gaussian_complex(m, k, 7), wl.gaussian_complex(k, n, 8)
    C = torch.empty((m, n), dtype=torch.complex128, device="cuda")
    ozimmu.zgemm(dev(A), dev(B), C, s, ozimmu.alloc_workspace(m, n, k, s, True))
    torch.cuda.synchronize()
    rows = np.r_[0:20, m - 20:m]
    assert np.array_equal(bits(C.cpu().numpy()[rows].view(np.float64)), bits(oracle.zgemm(A[rows], B, s).view(np.float64)))
