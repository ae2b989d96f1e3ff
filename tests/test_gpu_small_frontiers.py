"""Merge-path traversal of small frontiers, several iterations a launch: chains
past the iterations of one launch, fans that leave and enter the small regime
after even and odd numbers of them, ends without out-edges, and iteration limits
at every place, against the oracle bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2301_04792_amd as lb
import synthetic as S

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _chain_fan_chain(head, fan, tail, degree):
    """A chain of `head` edges, then `fan` vertices of `degree` edges into the next
    `degree`, all of which enter a chain of `tail` edges; the first chain's edges are also doubled."""
    n = head + 1 + fan + degree + tail + 1
    rows = [[] for _ in range(n)]
    for v in range(head):
        rows[v] = [v + 1, v + 1]
    f0, d0, t0 = head + 1, head + 1 + fan, head + 1 + fan + degree
    rows[head] = list(range(f0, d0))
    for v in range(f0, d0):
        rows[v] = list(range(d0, t0))
    for v in range(d0, t0):
        rows[v] = [t0, 0]
    for v in range(t0, n - 1):
        rows[v] = [v + 1]
    ro = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    ci = np.array([c for r in rows for c in r], np.int32)
    w = np.random.default_rng(head + fan).uniform(2.0 ** -10, 1, ci.size).astype(np.float32)
    return S.CSRHost(ro, ci, w, (n, n))


@pytest.mark.parametrize("params", [{}, {"grid_size": 1}], ids=["resident", "one_block"])
@pytest.mark.parametrize("head,fan,tail,degree", [
    (0, 1, 0, 1), (1, 2048, 0, 1), (2, 2049, 3, 1), (3, 2048, 2, 2), (254, 5000, 7, 1), (255, 5000, 258, 1),
    (256, 700, 1, 3), (257, 683, 255, 3), (1030, 10, 600, 200), (5, 2000, 300, 30)])
def test_chains_and_fans(head, fan, tail, degree, params):
    G = _chain_fan_chain(head, fan, tail, degree)
    Gd = lb.CSR.from_host(G, DEV)
    dref = oracle.bfs(G.row_offsets, G.col_idx, 0)
    depth, levels = lb.bfs(Gd.pattern, 0, "merge_path", **params)
    assert np.array_equal(depth.cpu().numpy(), dref)
    assert levels == int(dref.max()) + 1
    dist, _ = lb.sssp(Gd, 0, "merge_path", **params)
    ref = oracle.sssp(G.row_offsets, G.col_idx, G.values, 0)
    assert np.array_equal(dist.cpu().numpy().view(np.int32), ref.view(np.int32))


@pytest.mark.parametrize("limit", [1, 2, 3, 255, 256, 257, 300, 301, 302, 303, 304, 599, 600, 601, 602])
def test_iteration_limits(limit):
    G = _chain_fan_chain(300, 3000, 297, 1)
    Gd = lb.CSR.from_host(G, DEV)
    dref = oracle.bfs(G.row_offsets, G.col_idx, 0)
    needed = int(dref.max()) + 1  # frontiers, the last one's vertex without out-edges too
    if limit >= needed:
        depth, levels = lb.bfs(Gd.pattern, 0, "merge_path", max_iterations=limit)
        assert levels == needed and np.array_equal(depth.cpu().numpy(), dref)
        return

    depth = torch.full((G.m,), 7, dtype=torch.int32, device=DEV)
    with pytest.raises(lb.LBError, match="max_iterations"):
        lb.bfs(Gd.pattern, 0, "merge_path", depth=depth, max_iterations=limit)
    assert np.array_equal(depth.cpu().numpy(), np.where(dref <= limit, dref, -1))
