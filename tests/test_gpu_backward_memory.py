"""The backward of one gradient allocates no room for the products that only the
other one needs (4 to 6 bytes per nonzero), and gives the same bits."""
import pytest
import torch

import paper_2301_04792_amd as lb
import synthetic as S

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("transposed", [False, True])
@pytest.mark.parametrize("need_dx,need_dvalues", [(False, True), (True, False)])
def test_one_gradient_allocates_no_products(transposed, need_dx, need_dvalues):
    A = S.uniform_csr(5, 300_000, 90_001, 10)[0]
    assert A.nnz > 1_000_000
    Ad = lb.CSR.from_host(A, DEV)
    x, dy = torch.from_numpy(S.random_vector(4, A.n)).to(DEV), torch.from_numpy(S.random_vector(5, A.m)).to(DEV)
    tr = lb.transpose_pattern(Ad.pattern) if transposed else None
    both = lb.spmv_backward(Ad, x, dy, transposed=tr)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    before = torch.cuda.memory_allocated()
    torch.cuda.reset_peak_memory_stats()
    dx, dv = lb.spmv_backward(Ad, x, dy, need_dx=need_dx, need_dvalues=need_dvalues, transposed=tr)
    used = torch.cuda.max_memory_allocated() - before
    if need_dvalues:
        assert torch.equal(dv, both[1])
    if transposed and need_dx:
        assert torch.equal(dx, both[0])
    outputs = 4 * (A.n * need_dx + A.nnz * need_dvalues)
    if transposed or not need_dx:  # the scatter by bins needs its products for dx
        assert used < outputs + A.nnz, (used, outputs)
    else:
        assert used >= outputs + 6 * A.nnz
