"""Binding a pattern on the device at the sizes where its kernels change shape: bins of one and of several columns,
bitmaps in one and in several pieces, entries that fill their tiles exactly or by one more, bins with more entries than
a work-group holds in registers, more columns than one launch covers.  The mirror is compared bit for bit with a stable
sort by column, and a product through both partitions with plain sums."""
import numpy as np
import pytest

from paper_2407_17437_amd import workloads as wl
from test_gpu_parity import _mirror_check, close

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nb():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2407_17437_amd import binding
    return binding


@pytest.mark.parametrize("rows,cols,nnz", [
    (1, 1, 1), (1, 300, 300), (300, 1, 300), (64, 255, 2048), (64, 257, 2049),   # one tile, two tiles
    (33, 512, 4096), (8192, 513, 40000), (8193, 16384, 40000), (16385, 20000, 50000),   # narrower bins as the rows grow
    (262144, 5, 20000), (262145, 5, 20000), (600000, 3, 9000),                   # bitmap in one, two and three pieces
    (5000, 40, 190000),                                                          # more entries in a bin than its registers hold
    (3, (1 << 25) + 77, 500),                                                    # two launches' worth of columns
])
def test_mirror_where_the_build_changes_shape(nb, rows, cols, nnz):
    import torch
    rng = np.random.default_rng(rows + cols + nnz)
    flat = np.unique(rng.integers(0, rows * cols, size=2 * nnz, dtype=np.int64)) if nnz < rows * cols else np.arange(nnz)
    flat = np.sort(rng.permutation(flat)[:nnz])
    if cols > 1 << 25:
        flat = np.unique(np.concatenate([flat, [(1 << 25) - 1, 1 << 25, cols - 1, cols + (1 << 25) - 1]]))   # either side of the border
    indptr = np.concatenate([[0], np.cumsum(np.bincount(flat // cols, minlength=rows))])
    _mirror_check(nb, torch, rows, cols, indptr, (flat % cols).astype(np.int32))


@pytest.mark.parametrize("rows,cols,lens", [
    (2048, 300, "mixed"),       # short rows, long rows and rows at the 128-entry limit
    (2600, 9000, "huge"),       # rows cut over several work-groups among short ones
    (700, 1300, "staged"),      # a staged plan whose ranges hold split rows
])
def test_products_through_the_partitions(nb, oracle, rows, cols, lens):
    import torch
    rng = np.random.default_rng(rows)
    n = {"mixed": np.where(rng.random(rows) < 0.2, rng.integers(127, 300, rows), rng.integers(0, 40, rows)),
         "huge": np.where(rng.random(rows) < 0.004, rng.integers(4000, 9000, rows), rng.integers(0, 20, rows)),
         "staged": np.where(rng.random(rows) < 0.05, 1300, 200)}[lens]
    indptr, indices = wl.pattern_from_row_nnz(np.minimum(n, cols), cols, seed=rows)
    lay = wl.SparseLayerData(rows, cols, indptr, indices, wl.init_values(indptr, rows + 1), np.zeros(rows, np.float32), False)
    for batch in (100, 256):
        L = nb.SparseLinear(lay, max_batch=batch)
        X = rng.standard_normal((cols, batch)).astype(np.float32); dY = rng.standard_normal((rows, batch)).astype(np.float32)
        Yd, dXd = nb.dense(rows, batch), nb.dense(cols, batch)
        g, db = torch.empty(lay.nnz, device="cuda"), torch.empty(rows, device="cuda")
        nb.sparse_linear_forward(L.handle, nb.to_dense(X), Yd, batch)
        nb.sparse_linear_backward(L.handle, nb.to_dense(X), None, nb.to_dense(dY), dXd, g, db, batch)
        torch.cuda.synchronize()
        Y, S = oracle.spmm(rows, cols, indptr, indices, lay.values, lay.bias, X, False)
        close(Yd.cpu().numpy(), Y, S, what="Y")
        dX, S = oracle.spmm_t(rows, cols, indptr, indices, lay.values, dY)
        close(dXd.cpu().numpy(), dX, S, what="dX")
        gr, Sg, dbr, Sdb = oracle.sddmm(rows, cols, indptr, indices, dY, X)
        close(g.cpu().numpy(), gr, Sg, what="dvalues"); close(db.cpu().numpy(), dbr, Sdb, what="dbias")
        L.close()
