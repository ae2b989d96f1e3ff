"""The scatter by bins (the backward's dx and the CSC product of larger
matrices) at the edges of its bins and of its rule, against the oracle: the
usual tolerance on random values, exact sums on whole numbers."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2301_04792_amd as lb
import synthetic as S
from tests.gpu_util import assert_rows_close

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BIN = 8192


def _matrix(n, shape="mixed"):
    rng = np.random.default_rng(n)
    if shape == "one_column":  # every product into one target, chunk after chunk
        ro = np.minimum(np.arange(450_001), 450_000).astype(np.int32)
        ci = np.full(450_000, n - 1, np.int32)
        vals = rng.uniform(-1, 1, ci.size).astype(np.float32)
        return S.CSRHost(ro, ci, vals, (450_000, n))
    # rows longer than units, many empty rows, short rows; 410k nonzeros or more
    lengths = np.concatenate([np.minimum([20_000, 0, 9000], n), np.zeros(30_000, int), rng.integers(0, min(60, n), 13_000), [0]])
    while lengths.sum() < 410_000:
        lengths = np.concatenate([lengths, lengths[-20_000:]])
    return S.csr._from_lengths(n % 1000, lengths, n)[0]


CASES = [(1, "one_column"), (BIN - 1, "mixed"), (BIN, "mixed"), (BIN + 1, "mixed"), (70_001, "one_column"), (300_000, "mixed"),
         (512 * BIN, "mixed"), (512 * BIN + 1, "mixed")]


@pytest.mark.parametrize("n,shape", CASES)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_backward(n, shape, dtype):
    A = _matrix(n, shape)
    x, dy = S.random_vector(4, n), S.random_vector(5, A.m)
    if dtype == "bf16":
        A, x = A.with_values(S.to_bf16_bits(A.values)), S.to_bf16_bits(x)
        xd = torch.from_numpy(x.view(np.int16)).view(torch.bfloat16).to(DEV)
    else:
        xd = torch.from_numpy(x).to(DEV)
    Ad, dyd = lb.CSR.from_host(A, DEV), torch.from_numpy(dy).to(DEV)
    args = (A.row_offsets, A.col_idx, A.values, dy, n)
    ref, scale = oracle.spmv_transpose(*args), oracle.spmv_transpose(*args, abs_terms=True)
    rdv = oracle.dvalues(A.row_offsets, A.col_idx, dy.astype(np.float64), x).astype(np.float32)
    dx, dv = lb.spmv_backward(Ad, xd, dyd)
    assert np.array_equal(dv.cpu().numpy(), rdv)
    assert_rows_close(dx.cpu().numpy(), ref, scale, what=f"dx n={n} {shape}")
    dx, dv = lb.spmv_backward(Ad, xd, dyd, need_dvalues=False)
    assert dv is None
    assert_rows_close(dx.cpu().numpy(), ref, scale, what=f"dx alone n={n} {shape}")


@pytest.mark.parametrize("n,shape", CASES)
def test_csc_product(n, shape):
    A = _matrix(n, shape)  # its transpose by columns: targets are A's columns
    T = lb.CSC(torch.from_numpy(A.row_offsets).to(DEV), torch.from_numpy(A.col_idx).to(DEV), torch.from_numpy(A.values).to(DEV),
               (n, A.m))
    x = S.random_vector(6, A.m)
    args = (A.row_offsets, A.col_idx, A.values, x, n)
    y = lb.spmv_csc(T, torch.from_numpy(x).to(DEV)).cpu().numpy()
    assert_rows_close(y, oracle.spmv_transpose(*args), oracle.spmv_transpose(*args, abs_terms=True), what=f"csc n={n} {shape}")


def test_whole_numbers_are_exact_and_small_workspace_scatters():
    A = _matrix(300_000)
    Ai, _ = S.integer_valued(A, 7)
    dy = np.random.default_rng(1).integers(-3, 4, A.m).astype(np.float32)
    ref = oracle.spmv_transpose(Ai.row_offsets, Ai.col_idx, Ai.values, dy, A.n).astype(np.float32)
    T = lb.CSC(*(torch.from_numpy(v).to(DEV) for v in (Ai.row_offsets, Ai.col_idx, Ai.values)), (A.n, A.m))
    xd = torch.from_numpy(dy).to(DEV)
    need = lb.csc_workspace_size(T)
    assert np.array_equal(lb.spmv_csc(T, xd).cpu().numpy(), ref)
    s = lb.make_schedule("merge_path")
    ws = torch.empty(1 << 16,  # the split alone, as a call took before the bins
                      dtype=torch.uint8, device=DEV)
    assert ws.numel() < need
    y = torch.full((A.n,), 9.0, device=DEV)
    a = T.c_struct()
    st = lb._lib.lb_spmv_csc(ctypes.byref(a), lb._ptr(xd), 0, lb._ptr(y), ctypes.byref(s), lb._ptr(ws), ws.numel(),
                             lb._stream(T.device))
    assert st == 0
    assert np.array_equal(y.cpu().numpy(), ref)
