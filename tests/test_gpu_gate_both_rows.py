"""The gate kernel where a wavefront takes both row fragments of a tile, or only one by the number of the gate's fragments: every number of
fragments, ragged rows and columns, with and without counting, every slice count and the largest sums, against the oracle on sampled
rows, bit for bit. (States of more than 256 tiles of 32 x 32: fewer are taken by the kernel for small complex products.)"""
import numpy as np
import pytest
import torch

import oracle
from paper_2306_11975_amd import ozimmu
from paper_2306_11975_amd import workloads as wl

pytestmark = pytest.mark.gpu


def bits(x):
    return np.ascontiguousarray(x).view(np.uint64)


# m = 8225: tiles of four wavefronts, the last of one row; 4200: eight wavefronts to a tile where n > 32
@pytest.mark.parametrize("n", [1, 8, 9, 17, 25, 32, 33, 41, 50, 57, 64])
@pytest.mark.parametrize("m,k,s", [(8225, 64, 8), (8225, 30, 5), (8225, 47, 11), (8225, 16, 8), (4200, 64, 8), (4200, 20, 16)])
def test_every_number_of_fragments(m, n, k, s):
    A = wl.gaussian_complex_device(m, k, 41)
    A[m // 2] = 0
    B = wl.unit_column_complex_device(k, n, 42)
    rows = torch.tensor(sorted(set(range(0, 70)) | set(range(100, m, 391)) | {m - 17, m - 2, m - 1}), device="cuda")
    want = oracle.zgemm(A[rows].cpu().numpy(), B.cpu().numpy(), s)
    C = torch.full((m, n + 1), float("nan"), dtype=torch.complex128, device="cuda")
    ws = torch.empty(max(ozimmu.workspace_bytes(m, n, k, t, True) for t in range(1, 17)), dtype=torch.uint8, device="cuda")
    ozimmu.zgemm(A, B, C[:, :n], s, ws)
    assert np.array_equal(bits(C[rows][:, :n].cpu().numpy()), bits(want))
    assert torch.isnan(C[:, n:].real).all() and not torch.isnan(C[:, :n].real).any()
    # counting on the way; a threshold that every count meets, and s the largest allowed: the guess s = 1 is the choice, any other is not
    count, confirmed = ozimmu.zgemm_auto(A, B, C[:, :n], 1e9, guess=s, max_slices=s, workspace=ws)
    assert count == 1 and not confirmed
    count, confirmed = ozimmu.zgemm_auto(A, B, C[:, :n], 0.0, guess=s, max_slices=s, workspace=ws)
    assert count == ozimmu.auto_num_slices(A, B, 0.0, max_slices=s)[0] and confirmed == (count == s)


def check(A, B, s, step):
    m, k = A.shape
    n = B.shape[1]
    rows = torch.tensor(sorted(set(range(0, m, step)) | {1, 31, 32, m - 33, m - 2, m - 1}), device="cuda")
    C = torch.full((m, n), float("nan"), dtype=torch.complex128, device="cuda")
    ozimmu.zgemm(A, B, C, s, ozimmu.alloc_workspace(m, n, k, s, True))
    want = oracle.zgemm(A[rows].cpu().numpy(), B.cpu().numpy(), s)
    assert np.array_equal(bits(C[rows].cpu().numpy()), bits(want)) and not torch.isnan(C).any()


# one step: 32, 64 and 8 columns; two steps (16 fragments, eight wavefronts)
@pytest.mark.parametrize("s", range(1, 17))
@pytest.mark.parametrize("m,n,k", [(8225, 30, 32), (8225, 64, 33), (8225, 7, 13), (2100, 128, 65)])
def test_every_slice_count(m, n, k, s):
    check(wl.gaussian_complex_device(m, k, 50 + s), wl.unit_column_complex_device(k, n, 60 + s), s, 211)


@pytest.mark.parametrize("m,n,k,s", [(8225, 64, 64, 8), (8225, 64, 64, 12), (8225, 64, 64, 16), (8225, 32, 32, 5), (2100, 128, 128, 8), (2100, 128, 128, 9),
                                     (2100, 128, 128, 10)])
@pytest.mark.parametrize("signs", ["same", "mixed"])
def test_largest_sums(m, n, k, s, signs):
    """Every slice +-127: what the fold's 32-bit merge of neighbouring diagonals must hold."""
    rng = np.random.default_rng(k + s)

    def plane(r, c):
        x = np.full((r, c), 1.0 - 2.0 ** -53)
        return x if signs == "same" else x * rng.choice([-1.0, 1.0], size=(r, c))

    A = torch.from_numpy(plane(m, k) + 1j * plane(m, k)).cuda()
    B = torch.from_numpy(plane(k, n) + 1j * plane(k, n)).cuda()
    check(A, B, s, 401)
