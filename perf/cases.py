"""The work a user of this library has it do, as cases for timing and for comparing two builds' results.

Real products (ozimmu.dgemm, dgemm_blas, dgemm_dd, dgemm_auto) of matrices with the element distribution of the
accuracy experiment, (U(0,1) - 0.5) exp(phi N(0,1)), from a single tile to the inner dimension that needs INT64 sums, and
complex products (ozimmu.zgemm, zgemm_auto): a d-qubit gate applied to the state vector of N qubits, which is the product
2^(N-d) x 2^d times 2^d x 2^d, and a rectangular one. Slice counts are those the automatic mode picks for such inputs
(8 for an average loss of at most one bit, 11 to 13 for a lossless split) and the ones the accuracy experiment sweeps.
"""
import math

import torch

from paper_2306_11975_amd import ozimmu
from paper_2306_11975_amd import workloads


def listed():
    return [
        # one 64 x 64 tile: what a call costs when there is next to nothing to compute
        dict(name="dgemm_64", kind="dgemm", m=64, n=64, k=64, s=5, phi=0.5, pad=0),
        # the accuracy experiment's size and the count that beats the FP64 product at phi = 1
        dict(name="dgemm_1024", kind="dgemm", m=1024, n=1024, k=1024, s=9, phi=1.0, pad=0),
        # the headline product
        dict(name="dgemm_8192", kind="dgemm", m=8192, n=8192, k=8192, s=8, phi=1.0, pad=0),
        # lossless automatic mode (threshold 0: 12 or 13 slices), the previous product's count as the guess
        dict(name="dgemm_auto_2048", kind="dgemm_auto", m=2048, n=2048, k=2048, s=16, phi=1.0, pad=0, threshold=0.0),
        # an inner dimension beyond the INT32 block: INT64 sums, rows longer than the splitter's register cache
        dict(name="dgemm_long_k", kind="dgemm", m=4096, n=4096, k=131072, s=8, phi=2.0, pad=0),
        # the vendor-BLAS form as a library user calls it: column-major, one operand transposed, an update of C, odd sizes
        dict(name="dgemm_blas_ragged", kind="dgemm_blas", m=3001, n=1777, k=1203, s=6, phi=1.0, pad=3, transa="T", transb="N",
             alpha=0.5, beta=1.0),
        # more than FP64: many slices, double-double sum, odd sizes
        dict(name="dgemm_dd_ragged", kind="dgemm_dd", m=1501, n=1301, k=1107, s=14, phi=0.5, pad=0),
        # the complex product with a short inner dimension
        dict(name="zgemm_4096_256", kind="zgemm", m=4096, n=4096, k=256, s=7, pad=0),
        # a simulator's gate on a small register, slice count chosen in the call: latency
        dict(name="gate_6_of_16", kind="zgemm_auto", m=1 << 10, n=64, k=64, s=16, pad=0, threshold=1.0),
        # the same gate on a register that fills the chip, slice count known
        dict(name="gate_6_of_24", kind="zgemm", m=1 << 18, n=64, k=64, s=8, pad=0),
        # wider gates, slice count chosen in the call: the last size of the one-kernel path, and the general path
        dict(name="gate_8_of_24", kind="zgemm_auto", m=1 << 16, n=256, k=256, s=16, pad=0, threshold=1.0),
        dict(name="gate_10_of_24", kind="zgemm_auto", m=1 << 14, n=1024, k=1024, s=16, pad=0, threshold=1.0),
    ]


def _between(rng, lo, hi):
    """A whole number whose logarithm is uniform: odd ones, and now and then a power of two, among them."""
    x = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    if rng.random() < 0.15:
        return max(lo, min(hi, 1 << round(math.log2(x))))
    return max(lo, min(hi, round(x)))


def draw(rng):
    kind = rng.choice(["dgemm", "dgemm", "dgemm_auto", "dgemm_blas", "dgemm_dd", "zgemm", "gate", "gate"])
    if kind == "gate":   # the state's rows, the gate's size: 1 to 10 qubits of 12 to 24
        d = rng.randint(1, 10)
        m, dim = 1 << (rng.randint(max(12, d), 24) - d), 1 << d
        if rng.random() < 0.3:   # part of a register
            m = max(1, m - rng.randint(0, m // 3))
        pad = rng.choice([0, 0, rng.randint(1, 9)])
        if rng.random() < 0.5:
            return dict(kind="zgemm", m=m, n=dim, k=dim, s=rng.choice([7, 8, 8, 9, 11]), pad=pad)
        return dict(kind="zgemm_auto", m=m, n=dim, k=dim, s=16, pad=pad, threshold=rng.choice([0.0, 1.0, 1.0]))
    c = dict(kind=kind, m=_between(rng, 33, 8192), n=_between(rng, 33, 8192), k=_between(rng, 33, 8192),
             pad=rng.choice([0, 0, rng.randint(1, 9)]))
    if kind == "zgemm":
        c.update(m=_between(rng, 33, 4096), n=_between(rng, 33, 4096), k=_between(rng, 33, 2048), s=rng.randint(5, 9))
    elif kind == "dgemm_auto":
        c.update(m=_between(rng, 33, 4096), n=_between(rng, 33, 4096), k=_between(rng, 33, 4096), s=16,
                 phi=rng.choice([0.5, 1.0, 2.0]), threshold=rng.choice([0.0, 1.0]))
    elif kind == "dgemm_dd":
        c.update(m=_between(rng, 33, 3000), n=_between(rng, 33, 3000), k=_between(rng, 33, 3000), s=rng.randint(11, 16), phi=0.5)
    elif kind == "dgemm_blas":
        beta = rng.choice([0.0, 1.0, -0.75])
        c.update(s=rng.randint(5, 10), phi=1.0, transa=rng.choice("NT"), transb=rng.choice("NT"),
                 alpha=rng.choice([1.0, 0.5]), beta=beta)
    else:
        c.update(s=rng.randint(3, 13), phi=rng.choice([0.5, 1.0, 2.0]))
        if rng.random() < 0.2:
            c.update(m=_between(rng, 33, 2048), n=_between(rng, 33, 2048), k=_between(rng, 8192, 131072))
    return c


def _padded(x, pad):
    """x as the left part of a wider array: a leading dimension that is larger than the row."""
    if not pad:
        return x
    wide = torch.zeros((x.shape[0], x.shape[1] + pad), dtype=x.dtype, device=x.device)
    wide[:, : x.shape[1]] = x
    return wide[:, : x.shape[1]]


def prepare(case, seed):
    m, n, k, s, pad, kind = case["m"], case["n"], case["k"], case["s"], case["pad"], case["kind"]
    cplx = kind.startswith("zgemm")
    st = dict(kind=kind, s=s, case=case)
    dtype = torch.complex128 if cplx else torch.float64
    if kind == "dgemm_blas":   # column-major storage: a column-major r x c array is a row-major c x r one
        rows_a, cols_a = (m, k) if case["transa"] == "N" else (k, m)
        rows_b, cols_b = (k, n) if case["transb"] == "N" else (n, k)
        st["A"] = _padded(workloads.phi_matrix_device(cols_a, rows_a, case["phi"], 1000 + seed), pad)
        st["B"] = _padded(workloads.phi_matrix_device(cols_b, rows_b, case["phi"], 2000 + seed), pad)
        st["C0"] = _padded(workloads.phi_matrix_device(n, m, case["phi"], 3000 + seed), pad)
        st["C"] = st["C0"].clone() if not pad else _padded(st["C0"], pad)
        st["workspace"] = ozimmu.alloc_workspace(n, m, k, s)
        return st
    if cplx:
        A = workloads.gaussian_complex_device(m, k, 1000 + seed)
        st["A"] = _padded(A / torch.linalg.vector_norm(torch.view_as_real(A)), pad)   # a normalised state
        st["B"] = _padded(workloads.unit_column_complex_device(k, n, 2000 + seed), pad)
    else:
        st["A"] = _padded(workloads.phi_matrix_device(m, k, case["phi"], 1000 + seed), pad)
        st["B"] = _padded(workloads.phi_matrix_device(k, n, case["phi"], 2000 + seed), pad)
    st["C"] = _padded(torch.zeros((m, n), dtype=dtype, device="cuda"), pad)
    if kind == "dgemm_dd":
        st["C_lo"] = _padded(torch.zeros((m, n), dtype=dtype, device="cuda"), pad)
    if kind.endswith("_auto"):   # the workspace and scratch serve whichever count comes out
        need = max(ozimmu.workspace_bytes(m, n, k, t, cplx) for t in range(1, s + 1))
        st["workspace"] = torch.empty(need, dtype=torch.uint8, device="cuda")
        st["scratch"] = torch.empty(ozimmu.auto_scratch_bytes(n), dtype=torch.uint8, device="cuda")
        # the count that the previous product of a run took
        st["guess"] = ozimmu.auto_num_slices(st["A"], st["B"], case["threshold"], max_slices=s, scratch=st["scratch"])[0]
    else:
        st["workspace"] = ozimmu.alloc_workspace(m, n, k, s, cplx)
    return st


def run(st):
    kind, A, B, C, ws = st["kind"], st["A"], st["B"], st["C"], st["workspace"]
    if kind == "dgemm":
        ozimmu.dgemm(A, B, C, st["s"], ws)
        return C
    if kind == "zgemm":
        ozimmu.zgemm(A, B, C, st["s"], ws)
        return C
    if kind == "dgemm_dd":
        ozimmu.dgemm_dd(A, B, C, st["C_lo"], st["s"], ws)
        return {"C": C, "C_lo": st["C_lo"]}
    if kind == "dgemm_blas":
        c = st["case"]
        if c["beta"] != 0.0:   # every pass updates the same C
            C.copy_(st["C0"])
        ozimmu.dgemm_blas(c["transa"], c["transb"], c["m"], c["n"], c["k"], c["alpha"], A, A.stride(0), B, B.stride(0),
                          c["beta"], C, C.stride(0), st["s"], ws)
        return C
    auto = ozimmu.zgemm_auto if kind == "zgemm_auto" else ozimmu.dgemm_auto
    count, confirmed = auto(A, B, C, st["case"]["threshold"], guess=st["guess"], max_slices=st["s"], workspace=ws,
                            scratch=st["scratch"])
    return {"C": C, "num_slices": count, "confirmed": int(confirmed)}


def work(case):
    """Operands read once, result written once; the INT8 operations of the slice pairs p + q <= s + 1."""
    m, n, k, kind = case["m"], case["n"], case["k"], case["kind"]
    cplx = kind.startswith("zgemm")
    s = case["s"] if not kind.endswith("_auto") else (12 if case["threshold"] == 0.0 else 8)
    results = m * n * (2 if kind == "dgemm_dd" or (kind == "dgemm_blas" and case["beta"] != 0.0) else 1)
    return {"bytes": (16 if cplx else 8) * (m * k + k * n + results),
            "flops": (4 if cplx else 1) * (s * (s + 1) // 2) * 2 * m * n * k}


def tolerance(case):
    """The C interface fixes the slices, the order of every rounded sum and with them every bit of the result."""
    return "exact"


def exact(case, seed):
    """The product as torch forms it in FP64, from the same inputs. Up to nine or so slices the library's result differs
    from it by what those slices leave out."""
    st = prepare(case, seed)
    A, B = st["A"], st["B"]
    if case["kind"] == "dgemm_blas":   # row-major views of the column-major operands
        a = A.T if case["transa"] == "N" else A
        b = B.T if case["transb"] == "N" else B
        c = torch.matmul(a.contiguous(), b.contiguous()).T * case["alpha"]
        return c + case["beta"] * st["C0"] if case["beta"] != 0.0 else c
    c = torch.matmul(A, B)
    if case["kind"] == "dgemm_dd":
        return {"C": c, "C_lo": None}
    if case["kind"].endswith("_auto"):
        return {"C": c, "num_slices": None, "confirmed": None}
    return c
