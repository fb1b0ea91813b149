"""The gate kernel's workgroup shapes at the edges of their rules (k and n up to 16 and 8, few and many tiles), and its cut of the
state by FP64 conversions: against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2306_11975_amd import ozimmu
from paper_2306_11975_amd import workloads as wl

pytestmark = pytest.mark.gpu


def bits(x):
    return np.ascontiguousarray(x).view(np.float64).view(np.uint64)


@pytest.mark.parametrize("s", [1, 3, 4, 5, 8, 9, 11, 16])
@pytest.mark.parametrize("k,n", [(2, 2), (8, 8), (16, 8), (16, 9), (17, 8), (5, 3), (64, 64), (33, 8)])
def test_shapes_of_the_smallest_class_bit_exact(k, n, s):
    for m in (1, 33, 8192, 8193 + 64):    # 8192 rows: the last size of the shape for few tiles
        Z, G = wl.gaussian_complex(m, k, 1), wl.unit_column_complex(k, n, 2)
        C = torch.full((m, n), complex("nan"), dtype=torch.complex128, device="cuda")
        ozimmu.zgemm(torch.from_numpy(Z).cuda(), torch.from_numpy(G).cuda(), C, s, ozimmu.alloc_workspace(m, n, k, s, True))
        torch.cuda.synchronize()
        rows = np.r_[0:min(m, 70), max(0, m - 70):m]
        assert np.array_equal(bits(C.cpu().numpy()[rows]), bits(oracle.zgemm(Z[rows], G, s))), m


@pytest.mark.parametrize("s", [2, 6, 8])
@pytest.mark.parametrize("k", [3, 16, 64, 200])
def test_cut_of_extreme_values_bit_exact(k, s):
    # random bit patterns of every exponent, subnormals, exact powers of two, saturating fractions, zeros, rows of one kind
    rng = np.random.default_rng(k + s)
    m, n = 9000, 7
    raw = rng.integers(0, 1 << 63, size=(m, 2 * k), dtype=np.int64).view(np.float64)
    raw = np.where(np.isfinite(raw), raw, 1.0) * rng.choice([-1.0, 1.0], size=raw.shape)
    raw[0] = 0.0
    raw[1] = 4.9406564584124654e-324 * rng.integers(0, 1 << 20, size=2 * k)
    raw[2] = 2.0 ** rng.integers(-60, 60, size=2 * k)
    raw[3] = 1.0 - 2.0 ** -53
    raw[4] = np.finfo(np.float64).max
    raw[5, : k] = 2.0 ** 1023
    raw[5, k:] = 2.0 ** -1074
    raw[6] = -0.0
    Z = (raw[:, :k] + 1j * raw[:, k:])
    Z.imag = raw[:, k:]                  # (the sum above may lose a -0.0)
    Z.real = raw[:, :k]
    G = wl.unit_column_complex(k, n, 3)
    C = torch.empty((m, n), dtype=torch.complex128, device="cuda")
    ozimmu.zgemm(torch.from_numpy(Z).cuda(), torch.from_numpy(G).cuda(), C, s, ozimmu.alloc_workspace(m, n, k, s, True))
    torch.cuda.synchronize()
    rows = np.r_[0:60, m - 20:m]
    assert np.array_equal(bits(C.cpu().numpy()[rows]), bits(oracle.zgemm(np.ascontiguousarray(Z[rows]), G, s)))
