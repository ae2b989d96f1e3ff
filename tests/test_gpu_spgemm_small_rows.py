"""SpGEMM rows of at most 32 products (the register-sorted tier): every product
count from 0 to past its limit, repeated columns, unsorted factors and the
widest column range of its keys, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2301_04792_amd as lb
import synthetic as S
from tests.gpu_util import assert_rows_close

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _csr(rows, n):
    """A matrix from lists of columns, values by position."""
    ro = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    ci = np.array([c for r in rows for c in r], np.int32)
    return S.CSRHost(ro, ci, (np.random.default_rng(7).uniform(-1, 1, ci.size)).astype(np.float32), (len(rows), n))


def _check(A, B, what):
    C = lb.spgemm(lb.CSR.from_host(A, DEV), lb.CSR.from_host(B, DEV))
    ero, eci, ev = oracle.spgemm(A, B)
    scale = oracle.spgemm(A, B, abs_terms=True)[2]
    assert np.array_equal(C.row_offsets.cpu().numpy(), ero), what
    assert np.array_equal(C.col_idx.cpu().numpy(), eci), what
    assert_rows_close(C.values.cpu().numpy(), ev, scale, what=what)


@pytest.mark.parametrize("distinct", [1, 3, 40])
def test_every_product_count(distinct):
    rng = np.random.default_rng(distinct)
    # B's row j has j columns (any order, no repeats in a row); A's row i picks rows of B whose lengths add up to i
    B = _csr([list(rng.permutation(max(distinct, j))[:j]) for j in range(34)], 64)
    picks = []
    for i in range(36):
        parts, left = [], i
        while left > 0:
            take = int(rng.integers(1, min(left, 33) + 1))
            parts.append(take)
            left -= take
        picks.append(parts + [0] * int(rng.integers(0, 3)))  # empty rows of B too
    A = _csr([p for p in picks for _ in range(9)], 34)
    _check(A, B, f"{distinct} columns")


@pytest.mark.parametrize("n", [2**27 - 1, 2**27])
def test_widest_columns(n):
    rng = np.random.default_rng(1)
    cols = [sorted({0, n - 1, n - 2, int(rng.integers(n))}) for _ in range(50)]
    B = _csr(cols, n)
    A = _csr([list(rng.permutation(50)[: i % 9]) for i in range(300)], 50)
    C = lb.spgemm(lb.CSR.from_host(A, DEV), lb.CSR.from_host(B, DEV))
    # a dense oracle of n columns would not fit: the same sums over the columns that occur
    used = np.unique(B.col_idx)
    D = S.CSRHost(B.row_offsets, np.searchsorted(used, B.col_idx).astype(np.int32), B.values, (B.m, used.size))
    ero, eci, ev = oracle.spgemm(A, D)
    assert np.array_equal(C.row_offsets.cpu().numpy(), ero)
    assert np.array_equal(C.col_idx.cpu().numpy(), used[eci])
    assert_rows_close(C.values.cpu().numpy(), ev, oracle.spgemm(A, D, abs_terms=True)[2], what=f"n={n}")
