"""lb_resolve_schedule tells what lb_spmm runs: the schedule that it reports, passed
back, takes the same workspace and (on the GPU) gives the same bits."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
lb = pytest.importorskip("paper_2301_04792_amd", reason="liblb.so not built")
import synthetic as S  # noqa: E402
from paper_2301_04792_amd import _abi  # noqa: E402
from tests.gpu_util import assert_rows_close, oracle_spmm  # noqa: E402

FAKE = 0x10000  # never dereferenced


def _resolved(A, s, k):
    out = _abi.Schedule()
    assert _abi.load().lb_resolve_schedule(ctypes.byref(A), k, ctypes.byref(s), ctypes.byref(out)) == _abi.OK
    return out


@pytest.mark.parametrize("k", [1, 2, 8, 32, 64])
@pytest.mark.parametrize("kind", ["merge_path", "auto"])
@pytest.mark.parametrize("rows,nnz", [(4096, 64_248), (500_003, 11_700_000)])
def test_resolved_schedule_takes_the_same_workspace(rows, nnz, kind, k):
    A = _abi.CSR(rows, rows, nnz, FAKE, FAKE, FAKE, _abi.F32)
    sizes = []
    for s in (lb.make_schedule(kind), _resolved(A, lb.make_schedule(kind), k)):
        n = ctypes.c_size_t(0)
        assert _abi.load().lb_workspace_size(ctypes.byref(A), ctypes.byref(s), k, ctypes.byref(n)) == _abi.OK
        sizes.append(n.value)
    assert sizes[0] == sizes[1]


def _bytes(rows, nnz, k, dtype=_abi.F32, **units):
    n = ctypes.c_size_t(0)
    A = _abi.CSR(rows, rows, nnz, FAKE, FAKE, FAKE, dtype)
    assert _abi.load().lb_workspace_size(ctypes.byref(A), ctypes.byref(lb.make_schedule("merge_path", **units)), k,
                                         ctypes.byref(n)) == _abi.OK
    return n.value


@pytest.mark.parametrize("dtype", [_abi.F32, _abi.BF16])
@pytest.mark.parametrize("k,one_lane", [(2, True), (3, False), (4, True), (5, False), (8, False), (32, False)])
def test_whole_units_where_a_lane_holds_a_row(k, one_lane, dtype):
    """Halves of 256 x 8 cost more than they spread where a lane holds a whole row of
    X, past 512 units (128 x 16 and 128 x 8 items have as many units); past those, a
    named 256 x 8 is what it says."""
    whole, halves = {"block_size": 128, "items_per_thread": 16}, {"block_size": 128, "items_per_thread": 8}
    few, many = 512 * 2048, 512 * 2048 + 1  # merge items
    assert _bytes(100_000, few - 100_000, k, dtype) == _bytes(100_000, few - 100_000, k, dtype, **halves)
    assert _bytes(100_000, many - 100_000, k, dtype) == _bytes(100_000, many - 100_000, k, dtype, **(whole if one_lane else halves))
    named = {"block_size": 256, "items_per_thread": 8}
    assert _bytes(100_000, few - 100_000, k, dtype, **named) == _bytes(100_000, few - 100_000, k, dtype, **halves)
    assert _bytes(100_000, many - 100_000, k, dtype, **named) == _bytes(100_000, many - 100_000, k, dtype, **whole)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("k", [2, 3, 4, 8])
@pytest.mark.parametrize("items", [512 * 2048, 512 * 2048 + 1])
def test_sizes_around_the_rule(items, k, dtype):
    rng = np.random.default_rng(k)
    lengths = rng.integers(0, 9, 150_000)
    lengths[7] = 40_000  # longer than units
    lengths[-1] += items - 150_000 - lengths.sum()
    A, _ = S.csr._from_lengths(5, lengths, 600_000)
    assert A.m + A.nnz == items
    X = S.random_vector(3, A.n * k).reshape(A.n, k)
    if dtype == "bf16":
        A, X = A.with_values(S.to_bf16_bits(A.values)), S.to_bf16_bits(X)
        Xd = torch.from_numpy(X.view("int16")).view(torch.bfloat16).to("cuda:0")
    else:
        Xd = torch.from_numpy(X).to("cuda:0")
    Ad = lb.CSR.from_host(A, "cuda:0")
    want = oracle_spmm(A, X)
    assert_rows_close(lb.spmm(Ad, Xd).cpu().numpy(), *want, what=f"k={k} {dtype}")
    # the workspace of whole units and of the columns of one pass, 8, 4 or 2, as before the one-pass form
    narrow = lb.workspace_size(Ad, "merge_path", k={2: 2, 3: 2, 4: 4, 8: 8}[k], block_size=128, items_per_thread=16)
    ws = torch.empty(narrow, dtype=torch.uint8, device="cuda:0")
    assert_rows_close(lb.spmm(Ad, Xd, workspace=ws).cpu().numpy(), *want, what=f"k={k} {dtype}, workspace of one pass")
    base = lambda n: torch.tensor([0, n], dtype=torch.int64, device="cuda:0")  # noqa: E731
    B = lb.Batch(Ad.row_offsets, Ad.col_idx, Ad.values, base(A.m), base(A.nnz), base(A.n))
    assert_rows_close(lb.batched_spmm(B, Xd).cpu().numpy(), *want, what=f"batched k={k} {dtype}")


@pytest.mark.gpu
@pytest.mark.parametrize("k", [2, 24])
def test_resolved_schedule_gives_the_same_bits(k):
    A, _ = S.powerlaw_csr(7, 30_000, 20_000, 1.7, 9000, 0.1)
    X = S.random_vector(3, A.n * k).reshape(A.n, k)
    Ad, Xd = lb.CSR.from_host(A, "cuda:0"), torch.from_numpy(X).to("cuda:0")
    c = Ad.c_struct()
    Y = lb.spmm(Ad, Xd)
    assert_rows_close(Y.cpu().numpy(), *oracle_spmm(A, X), what=f"k={k}")
    back = _resolved(c, lb.make_schedule("merge_path"), k)
    assert torch.equal(Y, lb.spmm(Ad, Xd, back))
    # units of 256 x 8 items (as many as of 128 x 16) where the workspace is for those
    # only: for all columns, then for eight of them
    for cols in sorted({k, min(k, 8)}, reverse=True):
        n = lb.workspace_size(Ad, "merge_path", k=cols, block_size=128, items_per_thread=16)
        assert n < lb.workspace_size(Ad, "merge_path", k=cols)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda:0")
        for s in (lb.make_schedule("merge_path"), back):
            Z = torch.full_like(Y, 7.0)
            st = lb._lib.lb_spmm(ctypes.byref(c), lb._ptr(Xd), 0, k, k, lb._ptr(Z), k, ctypes.byref(s), lb._ptr(ws), n,
                                 lb._stream(Ad.device))
            assert st == 0
            assert_rows_close(Z.cpu().numpy(), *oracle_spmm(A, X), what=f"k={k}, workspace of {cols} columns")
