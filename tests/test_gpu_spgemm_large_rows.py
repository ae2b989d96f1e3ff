"""SpGEMM rows of more than 4096 products, with the row's bitmap in LDS (up to
2^18 columns) and in memory (more): the edges of the column chunks, rows of C of
one pass of sums, of several and of too many for LDS, more rows than slots, rows
of A longer than one deal of products, against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2301_04792_amd as lb
import synthetic as S
from tests.gpu_util import assert_rows_close

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _csr(rows, n, seed):
    ro = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    ci = np.concatenate([np.asarray(r, np.int32) for r in rows])
    return S.CSRHost(ro, ci, (np.random.default_rng(seed).uniform(-1, 1, ci.size)).astype(np.float32), (len(rows), n))


@pytest.mark.parametrize("n", [40, 16383, 16384, 16385, 2**18, 2**18 + 1])
@pytest.mark.parametrize("shape", ["many rows", "long rows", "wide rows"])
def test_large_rows(n, shape):
    rng = np.random.default_rng(n)
    cols = np.unique(np.concatenate([[0, n - 1, n // 2], rng.integers(0, n, 100_000 if shape == "wide rows" else 6000)]))
    longest = min(cols.size, {"many rows": 60, "long rows": 3000, "wide rows": 40_000}[shape])
    b_rows = [rng.permutation(cols)[: int(rng.integers(0, longest + 1))] for _ in range(300)] + [cols[:longest], cols[-longest:]]
    count, per = {"many rows": (530, 260), "long rows": (4, 900), "wide rows": (9, 0)}[shape]
    if shape == "wide rows":  # 16384 and 65536 entries are the edges of one pass and of the last
        parts = np.array_split(cols, 7)
        b_rows[:5] = [cols[:16384], cols[:16385], cols[:65536], cols[:65537], cols]
        b_rows[5:12] = [rng.permutation(q) for q in parts]
        a_rows = [np.array(r) for r in ([0], [1, 0], [2], [3, 1], [4, 5], [5, 6, 5, 7], list(range(5, 12)), [300, 301, 20], [6, 4, 4])]
    a_rows = a_rows if shape == "wide rows" else [np.concatenate([rng.integers(0, len(b_rows), per + int(rng.integers(0, 9))), [300, 301]]) for _ in range(count)]
    A, B = _csr(a_rows, len(b_rows), 1), _csr(b_rows, n, 2)
    C = lb.spgemm(lb.CSR.from_host(A, DEV), lb.CSR.from_host(B, DEV))
    used = np.unique(B.col_idx)
    D = S.CSRHost(B.row_offsets, np.searchsorted(used, B.col_idx).astype(np.int32), B.values, (B.m, used.size))
    ero, eci, ev = oracle.spgemm(A, D)
    assert np.array_equal(C.row_offsets.cpu().numpy(), ero)
    assert np.array_equal(C.col_idx.cpu().numpy(), used[eci])
    assert_rows_close(C.values.cpu().numpy(), ev, oracle.spgemm(A, D, abs_terms=True)[2], what=f"n={n} {shape}")
