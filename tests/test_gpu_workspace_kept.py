"""A caller's workspace from before the one-pass products and the bins (eight
columns of carries, the split alone) still serves, through the Python calls too;
one below that is refused."""
import pytest
import torch

import paper_2301_04792_amd as lb
import synthetic as S
from tests.gpu_util import assert_rows_close, oracle_spmm, oracle_spmv

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_spmm():
    A, _ = S.powerlaw_csr(7, 30_000, 20_000, 1.7, 9000, 0.1)
    X = S.random_vector(3, A.n * 24).reshape(A.n, 24)
    Ad, Xd = lb.CSR.from_host(A, DEV), torch.from_numpy(X).to(DEV)
    n = lb.workspace_size(Ad, "merge_path", k=8, block_size=128, items_per_thread=16)  # as many units as of 256 x 8
    ws = torch.empty(n, dtype=torch.uint8, device=DEV)
    assert_rows_close(lb.spmm(Ad, Xd, workspace=ws).cpu().numpy(), *oracle_spmm(A, X), what="spmm")
    assert_rows_close(lb.spmm(Ad, Xd, workspace=ws.view(torch.int32)).cpu().numpy(), *oracle_spmm(A, X), what="spmm, int32")
    with pytest.raises(ValueError):
        lb.spmm(Ad, Xd, workspace=ws[:n - 4])


def test_batched():
    import oracle
    B = S.batched_powerlaw(8, 23, 1, 4000)
    X = S.random_vector(9, B.total_cols * 17).reshape(-1, 17)
    Bd, Xd = lb.Batch.from_host(B, DEV), torch.from_numpy(X).to(DEV)
    units = (Bd.total_rows + Bd.total_nnz + 2047) // 2048  # of 256 x 8
    words = lambda k: -(-4 * k // 256) * 256  # noqa: E731
    n = 2 * words(units + 1) + words(units) + words(8 * units) + words(units + 1)  # split, carries of 8, matrices
    ws = torch.empty(n, dtype=torch.uint8, device=DEV)
    Y = lb.batched_spmm(Bd, Xd, workspace=ws).cpu().numpy()
    assert_rows_close(Y, oracle.batched_spmm(B, X), oracle.batched_spmm(B, X, abs_terms=True), what="batched")
    with pytest.raises(ValueError):
        lb.batched_spmm(Bd, Xd, workspace=ws[:n // 2])


def test_csc():
    A, x = S.powerlaw_csr(9, 60_000, 50_000, 1.7, 20_000, 0.1)
    assert A.nnz > 400_000
    import scipy.sparse as sp
    At = sp.csr_matrix((A.values, A.col_idx, A.row_offsets), shape=(A.m, A.n)).tocsc()
    T = lb.CSC(torch.from_numpy(At.indptr).to(DEV), torch.from_numpy(At.indices).to(DEV), torch.from_numpy(At.data).to(DEV), (A.m, A.n))
    split = torch.empty(1 << 16, dtype=torch.uint8, device=DEV)
    assert split.numel() < lb.csc_workspace_size(T)
    xd = torch.from_numpy(x).to(DEV)
    assert_rows_close(lb.spmv_csc(T, xd, workspace=split).cpu().numpy(), *oracle_spmv(A, x), what="csc")
    with pytest.raises(ValueError):
        lb.spmv_csc(T, xd, workspace=split[:256])
