"""Infinities and NaN through the products of several columns, the scatter by bins
and the sorted rows of SpGEMM: they reach the outputs that hold them, as in exact
arithmetic (an infinity of one sign stays, opposite ones give NaN), and no other.
Finite outputs keep the usual tolerance."""
import numpy as np
import pytest
import torch

import paper_2301_04792_amd as lb
import synthetic as S
from tests.gpu_util import RTOL

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _special(v, seed, share):
    """v with a share of its entries made inf, -inf or NaN."""
    v = v.copy()
    rng = np.random.default_rng(seed)
    at = rng.random(v.shape) < share
    v[at] = rng.choice(np.array([np.inf, -np.inf, np.nan], np.float32), int(at.sum()))
    return v


def _sum(where, terms, shape):
    """float64 sums of terms at the given places, and of their absolute values."""
    out, scale = np.zeros(shape), np.zeros(shape)
    with np.errstate(invalid="ignore"):
        np.add.at(out, where, terms)
        np.add.at(scale, where, np.abs(terms))
    return out, scale


def _agree(got, want, scale, what):
    got = got.astype(np.float64)
    special = ~np.isfinite(want)
    assert special.any() and not special.all(), what
    assert np.array_equal(got[special], want[special], equal_nan=True), what
    assert np.all(np.abs(got[~special] - want[~special]) <= RTOL * scale[~special]), what


def _bf16(v):
    """The float32 values that v rounds to, and its BF16 tensor."""
    t = torch.from_numpy(v).to(torch.bfloat16)
    return t.float().numpy(), t.to(DEV)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("k", [2, 8, 19])
def test_spmm(k, dtype):
    A, _ = S.powerlaw_csr(7, 6000, 5000, 1.7, 4500, 0.1)
    val, X = _special(A.values, 1, 2e-3), _special(S.random_vector(3, A.n * k).reshape(A.n, k), 2, 1e-3)
    if dtype == "bf16":
        (val, vd), (X, Xd) = _bf16(val), _bf16(X)
    else:
        vd, Xd = torch.from_numpy(val).to(DEV), torch.from_numpy(X).to(DEV)
    ro, ci = torch.from_numpy(A.row_offsets).to(DEV), torch.from_numpy(A.col_idx).to(DEV)
    row = np.repeat(np.arange(A.m), np.diff(A.row_offsets))
    with np.errstate(invalid="ignore"):
        terms = val.astype(np.float64)[:, None] * X.astype(np.float64)[A.col_idx]
    want, scale = _sum(row, terms, (A.m, k))
    _agree(lb.spmm(lb.CSR(ro, ci, vd, (A.m, A.n)), Xd).cpu().numpy(), want, scale, f"spmm k={k}")
    # the same matrix as a batch of one
    base = lambda n: torch.tensor([0, n], dtype=torch.int64, device=DEV)  # noqa: E731
    B = lb.Batch(ro, ci, vd, base(A.m), base(A.nnz), base(A.n))
    _agree(lb.batched_spmm(B, Xd).cpu().numpy(), want, scale, f"batched k={k}")


@pytest.mark.parametrize("shape", ["powerlaw", "stencil", "few_targets"])
def test_scatter_by_bins(shape):
    if shape == "powerlaw":
        A, _ = S.powerlaw_csr(9, 60_000, 50_000, 1.7, 20_000, 0.1)
    elif shape == "stencil":  # units summed in windows
        A, _ = S.laplacian_5pt(3, 320)
    else:  # targets that many lanes share
        A, _ = S.uniform_csr(4, 100_000, 40, 10)
    assert A.nnz > 400_000
    m, n = A.m, A.n
    # whole columns stay finite: special values fall into every 17th column only
    val = np.where(A.col_idx % 17 == 3, _special(A.values, 5, 5e-4), A.values)
    dy = S.random_vector(5, m)
    row = np.repeat(np.arange(m), np.diff(A.row_offsets))
    want, scale = _sum(A.col_idx, val.astype(np.float64) * dy.astype(np.float64)[row], n)
    ro, ci, vd = (torch.from_numpy(v).to(DEV) for v in (A.row_offsets, A.col_idx, val))
    dyd = torch.from_numpy(dy).to(DEV)
    dx, _ = lb.spmv_backward(lb.CSR(ro, ci, vd, (m, n)), torch.zeros(n, device=DEV), dyd)
    _agree(dx.cpu().numpy(), want, scale, f"dx {shape}")
    y = lb.spmv_csc(lb.CSC(ro, ci, vd, (n, m)), dyd)  # the same scatter: A^T by columns
    _agree(y.cpu().numpy(), want, scale, f"csc {shape}")


def test_transposed_products():
    A, _ = S.powerlaw_csr(31, 90_000, 50_000, 1.6, 30_000, 0.1)
    assert A.nnz > 1_000_000
    val, dy = _special(A.values, 5, 1e-3), S.random_vector(5, A.m)
    row = np.repeat(np.arange(A.m), np.diff(A.row_offsets))
    want, scale = _sum(A.col_idx, val.astype(np.float64) * dy.astype(np.float64)[row], A.n)
    Ad = lb.CSR.from_host(A.with_values(val), DEV)
    dx, _ = lb.spmv_backward(Ad, torch.zeros(A.n, device=DEV), torch.from_numpy(dy).to(DEV), transposed=lb.transpose_pattern(Ad.pattern))
    _agree(dx.cpu().numpy(), want, scale, "transposed dx")


@pytest.mark.parametrize("n", [3000, 300_000])  # the largest rows' sums in LDS and in a slot
def test_spgemm(n):
    # rows of A of up to 32, 256, 4096 and more products
    lengths = np.concatenate([np.tile([0, 1, 2], 20), np.tile([15, 20], 10), np.tile([150, 300], 5), [700, 900]])
    A, _ = S.csr._from_lengths(21, lengths, 2000)
    B, _ = S.uniform_csr(22, 2000, n, 24)
    av, bv = _special(A.values, 5, 0.02), _special(B.values, 6, 0.001)
    row = np.repeat(np.arange(A.m), lengths)
    blen = np.diff(B.row_offsets)[A.col_idx]
    e = np.repeat(np.arange(A.nnz), blen)
    f = np.arange(e.size) - np.repeat(np.cumsum(blen) - blen, blen) + B.row_offsets[A.col_idx][e]
    key = row[e].astype(np.int64) * n + B.col_idx[f]
    keys, at = np.unique(key, return_inverse=True)
    with np.errstate(invalid="ignore"):
        terms = av.astype(np.float64)[e] * bv.astype(np.float64)[f]
    want, scale = _sum(at, terms, keys.size)
    C = lb.spgemm(lb.CSR.from_host(A.with_values(av), DEV), lb.CSR.from_host(B.with_values(bv), DEV))
    assert np.array_equal(C.row_offsets.cpu().numpy(), np.concatenate([[0], np.cumsum(np.bincount(keys // n, minlength=A.m))]))
    assert np.array_equal(C.col_idx.cpu().numpy(), keys % n)
    _agree(C.values.cpu().numpy(), want, scale, f"spgemm n={n}")
