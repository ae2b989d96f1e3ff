"""The backward's dx by bins over many targets and few merge units: the launch
that splits the matrix also clears dx, on more blocks than there are unit
boundaries.  Against the oracle, untouched targets exactly zero."""
import numpy as np
import pytest
import torch

import oracle
import paper_2301_04792_amd as lb
import synthetic as S
from tests.gpu_util import assert_rows_close

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n,rows,per", [(512 * 8192, 100_000, 30), (2_500_003, 20_001, 110)])
def test_wide_dx_is_cleared(n, rows, per):
    A, _ = S.csr._from_lengths(11, np.full(rows, per), n)
    dy, x = S.random_vector(5, rows), S.random_vector(4, n)
    Ad = lb.CSR.from_host(A, DEV)
    args = (A.row_offsets, A.col_idx, A.values, dy, n)
    junk = torch.full((n,), 7.0, device=DEV)  # what dx's allocation holds before the call
    del junk
    dx, _ = lb.spmv_backward(Ad, torch.from_numpy(x).to(DEV), torch.from_numpy(dy).to(DEV))
    ref, scale = oracle.spmv_transpose(*args), oracle.spmv_transpose(*args, abs_terms=True)
    assert np.count_nonzero(scale == 0) > 100_000
    assert_rows_close(dx.cpu().numpy(), ref, scale, what=f"dx n={n}")
