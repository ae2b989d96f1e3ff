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


@pytest.mark.parametrize("k", [2, 8, 24])
def test_batched_of_larger_units(k):
    """Batches of 1024 to 2047 units of 512 x 8 items: their workspace still serves."""
    import oracle
    B = S.batched_powerlaw(8, 8, 20_000, 50_000)
    Bd = lb.Batch.from_host(B, DEV)
    units = (Bd.total_rows + Bd.total_nnz + 4095) // 4096
    assert 1024 <= units < 2048, units
    X = S.random_vector(9, B.total_cols * k).reshape(-1, k)
    Xd = torch.from_numpy(X).to(DEV)
    words = lambda n: -(-4 * n // 256) * 256  # noqa: E731
    n = 2 * words(units + 1) + words(units) + words(max(k, 8) * units) + words(units + 1)
    ref, scale = oracle.batched_spmm(B, X), oracle.batched_spmm(B, X, abs_terms=True)
    Y = lb.batched_spmm(Bd, Xd, workspace=torch.empty(n, dtype=torch.uint8, device=DEV))
    assert_rows_close(Y.cpu().numpy(), ref, scale, what=f"batched k={k}")
    assert_rows_close(lb.batched_spmm(Bd, Xd).cpu().numpy(), ref, scale, what=f"batched k={k}, its own workspace")
