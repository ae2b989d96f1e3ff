"""Unplanned merge path on matrices of short rows on average (a row per thread,
four nonzeros per lane): the limits of a short row, units with one longer row,
empty rows, unaligned arrays, CSR and COO, against the oracle; CSR and COO bit
for bit alike."""
import numpy as np
import pytest
import torch

import paper_2301_04792_amd as lb
import synthetic as S
from tests.gpu_util import assert_rows_close, oracle_spmv

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _matrix(name):
    rng = np.random.default_rng(len(name))
    n = 250_000  # more than 256 units of every shape: the one-launch form is another
    lengths = {
        "stencil": lambda: None,
        "up_to_16": lambda: rng.choice([0, 1, 2, 16], n, p=[0.2, 0.4, 0.2, 0.2]),
        "a_17": lambda: np.where(np.arange(n) % 601 == 0, 17, 4),
        "a_long_one": lambda: np.where(np.arange(n) % 50_000 == 7, 9000, 5),
        "empty": lambda: np.where(np.arange(n) % 9 == 0, 30, 0),
        "long_first_and_last": lambda: np.where((np.arange(n) == 0) | (np.arange(n) == n - 1), 70_000, 6),
        "mean_8": lambda: np.full(n, 8),
        "mean_past_8": lambda: np.where(np.arange(n) == 3, 9, 8),
    }[name]()
    if lengths is None:
        return S.laplacian_5pt(3, 520)
    return S.csr._from_lengths(8, lengths, 90_001)


NAMES = ["stencil", "up_to_16", "a_17", "a_long_one", "empty", "long_first_and_last", "mean_8", "mean_past_8"]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("name", NAMES)
def test_short_rows(name, dtype):
    A, x = _matrix(name)
    if dtype == "bf16":
        A, x = A.with_values(S.to_bf16_bits(A.values)), S.to_bf16_bits(x)
        xd = torch.from_numpy(x.view(np.int16)).view(torch.bfloat16).to(DEV)
    else:
        xd = torch.from_numpy(x).to(DEV)
    ref, scale = oracle_spmv(A, x)
    Ad, Cd = lb.CSR.from_host(A, DEV), lb.COO.from_host(S.to_coo(A), DEV)
    for params in ({}, {"block_size": 128, "items_per_thread": 4}, {"block_size": 256, "items_per_thread": 12}):
        y = lb.spmv(Ad, xd, "merge_path", **params)
        assert_rows_close(y.cpu().numpy(), ref, scale, what=f"{name} {dtype} {params}")
        assert torch.equal(y, lb.spmv(Ad, xd, "merge_path", **params))
        assert torch.equal(y, lb.spmv_coo(Cd, xd, "merge_path", **params))
    y4 = lb.spmv(Ad, xd, "merge_path", vector_width=4)
    assert_rows_close(y4.cpu().numpy(), ref, scale, what=f"{name} {dtype} vector_width 4")
    # the same arrays one element past an aligned start: one nonzero per lane, the same sums
    ci = torch.empty(A.nnz + 1, dtype=torch.int32, device=DEV)
    val = torch.empty(A.nnz + 1, dtype=Ad.values.dtype, device=DEV)
    ci[1:], val[1:] = Ad.col_idx, Ad.values
    U = lb.CSR(Ad.row_offsets, ci[1:], val[1:], A.shape)
    assert U.col_idx.data_ptr() % 16 and torch.equal(lb.spmv(U, xd, "merge_path"), lb.spmv(Ad, xd, "merge_path"))
