"""The transposed backward through products formed in A's order: dx equal bit
for bit to the form that gathers A's values (dx alone, or a workspace without
room for the products), and within the usual tolerance of the oracle."""
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

MATRICES = {  # at least a million nonzeros each, from where the products are used
    "powerlaw": lambda: S.powerlaw_csr(31, 90_000, 50_000, 1.6, 30_000, 0.1)[0],
    "stencil": lambda: S.laplacian_5pt(3, 460)[0],
    "short_rows": lambda: S.uniform_csr(5, 400_000, 7001, 6)[0],
    "long_column": lambda: S.csr._from_lengths(4, [1] * 1_000_000, 1)[0],
}


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("name", sorted(MATRICES))
def test_products_and_values_agree(name, dtype):
    A = MATRICES[name]()
    assert A.nnz >= 1_000_000
    x, dy = S.random_vector(4, A.n), S.random_vector(5, A.m)
    if dtype == "bf16":
        A, x = A.with_values(S.to_bf16_bits(A.values)), S.to_bf16_bits(x)
        xd = torch.from_numpy(x.view(np.int16)).view(torch.bfloat16).to(DEV)
    else:
        xd = torch.from_numpy(x).to(DEV)
    Ad, dyd = lb.CSR.from_host(A, DEV), torch.from_numpy(dy).to(DEV)
    tr = lb.transpose_pattern(Ad.pattern)
    dx, dv = lb.spmv_backward(Ad, xd, dyd, transposed=tr)
    args = (A.row_offsets, A.col_idx, A.values, dy, A.n)
    assert_rows_close(dx.cpu().numpy(), oracle.spmv_transpose(*args), oracle.spmv_transpose(*args, abs_terms=True), what=name)
    assert torch.equal(dx, lb.spmv_backward(Ad, xd, dyd, need_dvalues=False, transposed=tr)[0])

    s, c, n = lb.make_schedule("merge_path"), Ad.c_struct(), ctypes.c_size_t(0)
    assert lb._lib.lb_backward_transposed_workspace_size(ctypes.byref(c), ctypes.byref(s), ctypes.byref(n)) == 0
    less = n.value - (A.nnz * 4 + 255) // 256 * 256
    ws = torch.empty(less, dtype=torch.uint8, device=DEV)
    dx2, dv2 = torch.full_like(dx, 3.0), torch.full_like(dv, 3.0)
    st = lb._lib.lb_spmv_backward_transposed(ctypes.byref(c), *(lb._ptr(t) for t in tr), lb._ptr(xd), lb._dtype_code(xd), lb._ptr(dyd),
                                             lb._ptr(dx2), lb._ptr(dv2), ctypes.byref(s), lb._ptr(ws), less, lb._stream(Ad.device))
    assert st == 0
    assert torch.equal(dx2, dx) and torch.equal(dv2, dv)
