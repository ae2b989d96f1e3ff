"""The one-pass products, the scatter by bins and the products form under HIP graph
capture and on a stream of their own: replays on new values, with eager work and
waits between them, equal the eager call (whole numbers: exact in any order)."""
import numpy as np
import pytest
import torch

import paper_2301_04792_amd as lb
import synthetic as S

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _whole(seed, *shape):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return torch.randint(-3, 4, shape, device=DEV, generator=g).float()


def _matrix(name):
    if name == "stencil":
        return lb.CSR.from_host(S.laplacian_5pt(3, 460)[0], DEV)
    return lb.CSR.from_host(S.integer_valued(S.powerlaw_csr(31, 90_000, 50_000, 1.6, 30_000, 0.1)[0], 7)[0], DEV)


def _calls(name):
    """name -> (inputs that a replay changes, the call)"""
    A = _matrix(name)
    m, n = A.shape
    X, x, dy = _whole(1, n, 11), _whole(2, n), _whole(3, m)
    base = lambda v: torch.tensor([0, v], dtype=torch.int64, device=DEV)  # noqa: E731
    B = lb.Batch(A.row_offsets, A.col_idx, A.values, base(m), base(A.nnz), base(n))
    T = lb.CSC(A.row_offsets, A.col_idx, A.values, (n, m))
    tr = lb.transpose_pattern(A.pattern)
    return {
        "spmm": (X, lambda: lb.spmm(A, X)),
        "batched": (X, lambda: lb.batched_spmm(B, X)),
        "csc": (dy, lambda: lb.spmv_csc(T, dy)),
        "scatter": (dy, lambda: lb.spmv_backward(A, x, dy)),
        "transposed": (dy, lambda: lb.spmv_backward(A, x, dy, transposed=tr)),
    }


CALLS = ["spmm", "batched", "csc", "scatter", "transposed"]


def _list(out):
    return list(out) if isinstance(out, tuple) else [out]


@pytest.mark.parametrize("call", CALLS)
@pytest.mark.parametrize("name", ["powerlaw", "stencil"])
def test_capture(name, call):
    changed, f = _calls(name)[call]
    f()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        outs = _list(f())
    for seed in range(4):
        changed.copy_(_whole(10 + seed, *changed.shape))
        want = _list(f())
        for o in outs:
            o.fill_(7.0)
        torch.cuda.synchronize()
        g.replay()
        if seed % 2:
            torch.cuda.synchronize()
        for o, w in zip(outs, want):
            assert torch.equal(o, w), (name, call, seed)


@pytest.mark.parametrize("call", CALLS)
def test_two_streams(call):
    changed, f = _calls("powerlaw")[call]
    want = [w.clone() for w in _list(f())]
    torch.cuda.synchronize()
    streams, outs = [torch.cuda.Stream(), torch.cuda.Stream()], []
    for _ in range(3):
        for s in streams:
            with torch.cuda.stream(s):
                outs.append(_list(f()))
    torch.cuda.synchronize()
    for out in outs:
        for o, w in zip(out, want):
            assert torch.equal(o, w), call
