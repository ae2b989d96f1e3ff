"""Merge-path traversal at the edges of its units: frontiers of one vertex to
several units of vertices, with degrees of none, one and about a unit, odd and
even slot counts, against the oracle bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_2301_04792_amd as lb
import synthetic as S

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _two_levels(width, degree, empty_every):
    """Vertex 0 -> `width` vertices; each of those -> `degree` of `width + 7` others
    (every empty_every-th of them none)."""
    rng = np.random.default_rng(width * 31 + degree)
    third = width + max(degree, 7)
    n = 1 + width + third
    lengths = np.zeros(n, np.int64)
    lengths[0] = width
    lengths[1:1 + width] = degree
    if empty_every:
        lengths[1:1 + width:empty_every] = 0
    lengths[1 + width::5] = 1  # some go on, to anywhere
    ro = np.zeros(n + 1, np.int32)
    np.cumsum(lengths, out=ro[1:])
    ci = rng.integers(1 + width, n, int(ro[-1])).astype(np.int32)
    ci[:width] = np.arange(1, 1 + width)
    w = rng.uniform(2.0 ** -10, 1, ci.size).astype(np.float32)
    return S.CSRHost(ro, ci, w, (n, n))


@pytest.mark.parametrize("width,degree,empty_every", [
    (1, 1, 0), (1, 2047, 0), (1, 2048, 0), (1, 2049, 0), (2, 1, 0), (2, 5000, 0), (3, 0, 0), (1023, 1, 0), (1024, 2, 0),
    (2047, 1, 0), (2048, 1, 0), (2049, 1, 0), (2050, 1, 2), (4097, 1, 3), (6000, 3, 0), (40_000, 1, 0), (40_001, 7, 4)])
@pytest.mark.parametrize("params", [{}, {"grid_size": 1}, {"grid_size": 7}], ids=["resident", "one_block", "seven_blocks"])
def test_two_levels(width, degree, empty_every, params):
    G = _two_levels(width, degree, empty_every)
    Gd = lb.CSR.from_host(G, DEV)
    dist, _ = lb.sssp(Gd, 0, "merge_path", **params)
    ref = oracle.sssp(G.row_offsets, G.col_idx, G.values, 0)
    assert np.array_equal(dist.cpu().numpy().view(np.int32), ref.view(np.int32))
    depth, levels = lb.bfs(Gd.pattern, 0, "merge_path", **params)
    dref = oracle.bfs(G.row_offsets, G.col_idx, 0)
    assert np.array_equal(depth.cpu().numpy(), dref)
    assert levels == int(dref.max()) + 1
