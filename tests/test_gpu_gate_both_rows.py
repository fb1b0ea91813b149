"""Gates of one step on states of more rows than compute units times 32, where a wavefront takes both row fragments of a tile or only one by
the number of the gate's fragments: every number of fragments, ragged rows and columns, with and without counting, against the
oracle on sampled rows, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2306_11975_amd import ozimmu
from paper_2306_11975_amd import workloads as wl

pytestmark = pytest.mark.gpu


def bits(x):
    return np.ascontiguousarray(x).view(np.uint64)


# m = 8225: tiles of four wavefronts, the last of one row; 900: eight wavefronts to a tile
@pytest.mark.parametrize("n", [1, 8, 9, 17, 25, 32, 33, 41, 50, 57, 64])
@pytest.mark.parametrize("m,k,s", [(8225, 64, 8), (8225, 30, 5), (8225, 47, 11), (8225, 16, 8), (900, 64, 8), (900, 20, 16)])
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
