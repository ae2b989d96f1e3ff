"""SpGEMM rows of 33 to 4096 products (the tiers sorted by a wavefront and by a
block): the edges of every network size, few long and many short B rows, repeated
columns, and column ranges on both sides of the 32-bit key, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2301_04792_amd as lb
import synthetic as S
from tests.gpu_util import assert_rows_close

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
EDGES = (31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097)


def _csr(rows, n, seed):
    ro = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    ci = np.array([c for r in rows for c in r], np.int32)
    return S.CSRHost(ro, ci, (np.random.default_rng(seed).uniform(-1, 1, ci.size)).astype(np.float32), (len(rows), n))


@pytest.mark.parametrize("piece", [1, 7, 300, 4097])
@pytest.mark.parametrize("n", [5000, 2**20, 2**20 + 1, 2**24, 2**24 + 1])
def test_edges_of_the_networks(piece, n):
    # Row i of A picks rows of B of at most `piece` entries until it has EDGES[i] products, with empty rows of B between.
    rng = np.random.default_rng(piece + n)
    pool = np.unique(np.concatenate([[0, n - 1], rng.integers(0, n, 4998)]))
    used = pool if pool.size > 4097 else np.arange(5000)
    lengths = sorted({0, *(e % piece or piece for e in EDGES), *(e for e in EDGES if e <= piece), piece})
    by_length = {}
    b_rows = []
    for ln in lengths:
        by_length[ln] = []
        for _ in range(3 if ln > 64 else 12):
            by_length[ln].append(len(b_rows))
            b_rows.append(list(rng.permutation(used)[:ln]))
    a_rows = []
    for total in EDGES:
        for _ in range(3):
            left, row = total, []
            while left:
                take = left if left in by_length else min(piece, left)
                row.append(int(rng.choice(by_length[take])))
                left -= take
                if rng.random() < 0.1:
                    row.append(int(rng.choice(by_length[0])))
            a_rows.append([row[k] for k in rng.permutation(len(row))])
    A, B = _csr(a_rows, len(b_rows), 1), _csr(b_rows, n, 2)
    C = lb.spgemm(lb.CSR.from_host(A, DEV), lb.CSR.from_host(B, DEV))
    # the oracle over the columns that occur
    cols = np.unique(B.col_idx)
    D = S.CSRHost(B.row_offsets, np.searchsorted(cols, B.col_idx).astype(np.int32), B.values, (B.m, cols.size))
    ero, eci, ev = oracle.spgemm(A, D)
    assert np.array_equal(C.row_offsets.cpu().numpy(), ero)
    assert np.array_equal(C.col_idx.cpu().numpy(), cols[eci])
    assert_rows_close(C.values.cpu().numpy(), ev, oracle.spgemm(A, D, abs_terms=True)[2], what=f"piece={piece} n={n}")
    again = lb.spgemm(lb.CSR.from_host(A, DEV), lb.CSR.from_host(B, DEV))
    rows = np.repeat(np.arange(len(a_rows)), np.diff(ero))
    small = np.repeat(EDGES, 3)[rows] <= 4096  # larger rows add in any order
    same = (again.values == C.values).cpu().numpy()
    assert same[small].all()
