"""Where the scatter goes by bins, seen from the workspace sizes (on the host):
sizes at which bins measured slower than atomics ask for the split's workspace only."""
import ctypes

import pytest

pytest.importorskip("torch")
lb = pytest.importorskip("paper_2301_04792_amd", reason="liblb.so not built")
from paper_2301_04792_amd import _abi  # noqa: E402

FAKE = 0x10000  # never dereferenced


def _size(fn, A, *args):
    n = ctypes.c_size_t(0)
    assert fn(ctypes.byref(A), ctypes.byref(lb.make_schedule("merge_path")), *args, ctypes.byref(n)) == _abi.OK
    return n.value


def _backward_by_bins(rows, cols, nnz):
    A = _abi.CSR(rows, cols, nnz, FAKE, FAKE, FAKE, _abi.F32)
    return _size(_abi.load().lb_workspace_size, A, 0) >= 6 * nnz


def _csc_by_bins(rows, cols, nnz):
    A = _abi.CSC(rows, cols, nnz, FAKE, FAKE, FAKE, _abi.F32)
    return _size(_abi.load().lb_csc_workspace_size, A) >= 6 * nnz


FASTER = [(100_000, 100_000, 400_000), (20_000, 300_000, 400_000), (1_000_000, 1_000_000, 1_000_000), (1_000_000, 4_194_304, 4_000_000),
          (90_000, 90_000, 448_800), (4_194_304, 4_194_304, 20_963_328), (5_000_000, 10_000, 400_000), (64_000_000, 10_000, 4_000_000),
          (1_000_000, 1000, 32_000_000), (30_000_000, 4_000_000, 16_000_000)]
SLOWER = [(400_000, 400_000, 399_999), (400_000, 400_000, 400_000), (20_000, 1_000_000, 640_000), (200_000, 4_194_304, 400_000),
          (1_000_000, 4_194_304, 2_000_000), (4_000_000, 4_194_304, 400_000), (50_000_000, 10_000, 500_000),
          (200_000_000, 4_000_000, 500_000), (100_000_000, 4_000_000, 16_000_000), (1_000_000, 4_194_305, 40_000_000)]


@pytest.mark.parametrize("rows,cols,nnz", FASTER)
def test_bins_where_they_are_faster(rows, cols, nnz):
    assert _backward_by_bins(rows, cols, nnz)
    assert _csc_by_bins(cols, rows, nnz)  # the same scatter: A^T stored by columns


@pytest.mark.parametrize("rows,cols,nnz", SLOWER)
def test_atomics_where_they_are_faster(rows, cols, nnz):
    assert not _backward_by_bins(rows, cols, nnz)


@pytest.mark.parametrize("tiles,targets,nnz,bins", [(50_000, 4_194_304, 400_000, True), (50_001, 4_194_304, 400_000, False),
                                                    (20_000, 1_000_000, 640_000, True), (1_000_000, 1_000_000, 400_000, False),
                                                    (50_000_000, 1_000_000, 500_000, False)])
def test_csc_of_few_columns(tiles, targets, nnz, bins):
    assert _csc_by_bins(targets, tiles, nnz) == bins


@pytest.mark.parametrize("tiles,targets,nnz,bins", [(20_000, 2, 500_000, False), (300_000, 4, 2_000_000, False), (20_000, 2, 4_000_000, False),
                                                    (20_000, 2, 4_000_001, True), (20_000, 8, 1_000_000, False), (20_000, 9, 500_000, True),
                                                    (20_000, 1, 4_000_000, True), (2_000_000, 4, 500_000, True),
                                                    (2_000_000, 1, 500_000, False), (2_000_001, 1, 500_000, True)])
def test_csc_of_few_rows(tiles, targets, nnz, bins):
    assert _csc_by_bins(targets, tiles, nnz) == bins
