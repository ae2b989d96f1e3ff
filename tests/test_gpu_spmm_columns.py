"""SpMM of two and more columns: every lane-group width (k from 2 to 64, the
last lanes overlapping where k is no multiple of a load), both value types, X
and Y rows at any alignment, and the passes of a narrow workspace, against the
oracle at the usual tolerance."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2301_04792_amd as lb
import synthetic as S
from tests.gpu_util import assert_rows_close, oracle_spmm

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _matrix():
    # empty rows, rows of a unit and of many units, ragged short ones
    rng = np.random.default_rng(3)
    lengths = np.concatenate([[0, 7000, 0, 1], rng.integers(0, 40, 900), [0, 0, 2048, 4096, 1], rng.integers(0, 3, 3000), [0]])
    return S.csr._from_lengths(21, lengths, 7001)[0]


def _bf16(A, X):
    return A.with_values(S.to_bf16_bits(A.values)), S.to_bf16_bits(X)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("k", [2, 3, 4, 5, 7, 8, 9, 13, 16, 24, 33, 63, 64])
def test_column_counts(k, dtype):
    A = _matrix()
    ld = k + 3  # an odd stride, and a first column past an aligned one
    X = S.random_vector(5, A.n * ld).reshape(A.n, ld)
    if dtype == "bf16":
        A, Xr = _bf16(A, X)
        Xd = torch.from_numpy(Xr.view(np.int16)).view(torch.bfloat16).to(DEV)
    else:
        Xr, Xd = X, torch.from_numpy(X).to(DEV)
    Ad = lb.CSR.from_host(A, DEV)
    for c0, block, items in ((0, 256, 8), (1, 128, 4), (3, 512, 16)):
        Y = torch.full((A.m, ld), 7.0, device=DEV)
        lb.spmm(Ad, Xd[:, c0:c0 + k], "merge_path", Y=Y[:, c0:c0 + k], block_size=block, items_per_thread=items)
        ref, scale = oracle_spmm(A, np.ascontiguousarray(Xr[:, c0:c0 + k]))
        Yh = Y.cpu().numpy()
        assert_rows_close(Yh[:, c0:c0 + k], ref, scale, what=f"k={k} {dtype} from column {c0}")
        outside = np.delete(Yh, np.s_[c0:c0 + k], axis=1)
        assert np.all(outside == 7.0)


@pytest.mark.parametrize("k", [11, 24])
def test_narrow_workspace_runs_in_passes(k):
    """A workspace with at most eight columns of carries (what a call took
    before the one-pass form) is still enough."""
    A = _matrix()
    X = S.random_vector(6, A.n * k).reshape(A.n, k)
    Ad, Xd = lb.CSR.from_host(A, DEV), torch.from_numpy(X).to(DEV)
    ref, scale = oracle_spmm(A, X)
    small = {"block_size": 128, "items_per_thread": 4}
    old_default = lb.workspace_size(Ad, "merge_path", k=8, block_size=256, items_per_thread=8)
    for units, n8 in ((small, lb.workspace_size(Ad, "merge_path", k=8, **small)), ({}, old_default)):
        s = lb.make_schedule("merge_path", **units)
        assert n8 < lb.workspace_size(Ad, "merge_path", k=k, **units)
        ws = torch.empty(n8, dtype=torch.uint8, device=DEV)
        Y = torch.empty((A.m, k), device=DEV)
        st = lb._lib.lb_spmm(ctypes.byref(Ad.c_struct()), lb._ptr(Xd), 0, k, k, lb._ptr(Y), k, ctypes.byref(s), lb._ptr(ws),
                             n8, lb._stream(Ad.device))
        assert st == 0
        assert_rows_close(Y.cpu().numpy(), ref, scale, what=f"narrow workspace, k={k}, {units}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("k", [2, 6, 8, 11, 17])
def test_batched_column_counts(k, dtype):
    B = S.batched_powerlaw(8, 23, 1, 4000)
    X = S.random_vector(9, B.total_cols * k).reshape(-1, k)
    if dtype == "bf16":
        import dataclasses
        B = dataclasses.replace(B, values=S.to_bf16_bits(B.values))
        X = S.to_bf16_bits(X)
        Xd = torch.from_numpy(X.view(np.int16)).view(torch.bfloat16).to(DEV)
    else:
        Xd = torch.from_numpy(X).to(DEV)
    Y = lb.batched_spmm(lb.Batch.from_host(B, DEV), Xd).cpu().numpy()
    assert_rows_close(Y, oracle.batched_spmm(B, X), oracle.batched_spmm(B, X, abs_terms=True), what=f"batched k={k}")
