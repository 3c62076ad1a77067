"""Binding a pattern on the device at the sizes where its kernels change shape: bins of one and of several columns,
bitmaps in one and in several pieces, entries that fill their tiles exactly or by one more, bins with more entries than
a work-group holds in registers, more columns than one launch covers.  The mirror is compared bit for bit with a stable
sort by column, and a product through both partitions with plain sums."""
import numpy as np
import pytest

from paper_2407_17437_amd import workloads as wl
from test_gpu_parity import _mirror_check, close, raw_i32

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


def device_tables(nb, torch, layer, side):
    out = []
    for table in range(6):
        p, n = nb.sparse_linear_partition(layer, side, table)
        out.append(raw_i32(nb, torch, p, n) if n else np.zeros(0, np.int32))
    return out


@pytest.mark.parametrize("rows,cols,max_batch,lens", [
    (1, 1, 1, lambda r: [1]), (5, 9, 64, lambda r: np.zeros(5)), (300, 77, 16, lambda r: r.integers(0, 78, 300)),
    (1025, 3072, 100, lambda r: r.integers(250, 360, 1025)),                                        # classes that hand rows up
    (2047, 900, 256, lambda r: r.integers(0, 129, 2047)), (2048, 900, 256, lambda r: r.integers(0, 129, 2048)),   # no packed rows, all packed
    (3000, 5000, 128, lambda r: np.where(r.random(3000) < 0.02, r.integers(1000, 5000, 3000), r.integers(0, 200, 3000))),   # huge rows among packed ones
    (40, 20000, 64, lambda r: r.integers(15000, 20001, 40)),                                        # nothing but huge rows
    (1200, 1500, 512, lambda r: np.where(r.random(1200) < 0.03, 1500, 220)),                        # all rows staged, some of them split
    (9000, 4000, 1024, lambda r: np.where(r.random(9000) < 0.1, r.integers(200, 490, 9000), r.integers(0, 40, 9000))),      # the long rows staged
    (4096, 4096, 1024, lambda r: np.minimum(4096, 2e5 / (1 + np.arange(4096.)))),                   # power law
], ids=str)
def test_tables_equal_the_host_planner(nb, rows, cols, max_batch, lens):
    """Entry for entry, of the matrix and of its mirror, also after a rebind has used the other set of buffers."""
    import torch
    rng = np.random.default_rng(rows)
    n = np.asarray(lens(rng)).astype(np.int64)
    nb.nerva_set_dense_threshold(2.0)
    try:
        for take in (slice(None), slice(None, None, -1)):   # (then the same rows in the other order, by rebinding)
            indptr, indices = wl.pattern_from_row_nnz(n[take], cols, seed=rows + cols)
            values = wl.init_values(indptr, 1)
            if take.step is None:
                L = nb.SparseLinear(wl.SparseLayerData(rows, cols, indptr, indices, values, np.zeros(rows, np.float32), False), max_batch=max_batch)
            else:
                L.rebind(indptr, indices, values)
            row = np.repeat(np.arange(rows), np.diff(indptr))
            order = np.lexsort((row, indices))
            indptr_t = np.concatenate([[0], np.cumsum(np.bincount(indices, minlength=cols))]).astype(np.int32)
            for side, (m, k, ip, ix) in enumerate(((rows, cols, indptr, indices), (cols, rows, indptr_t, row[order].astype(np.int32)))):
                waves, huge, short, long_waves, staged_rows, staged_ends = device_tables(nb, torch, L.handle, side)
                _, _, h_huge, _, h_waves = nb.nerva_plan_rows_host(m, ip)
                h_short, n_short, h_long, _ = nb.nerva_plan_short_rows_host(m, ip)
                assert np.array_equal(huge, h_huge.ravel()), "huge rows"
                assert np.array_equal(short, h_short.ravel()), "short rows"
                for got, ref in ((waves, h_waves), (long_waves, h_long)):
                    got, ref = got.reshape(-1, 4), ref.reshape(-1, 4)
                    assert got.shape == ref.shape and np.array_equal(got[:, :3], ref[:, :3]) and np.array_equal(got[:, 3] & 1023, ref[:, 3])
                    is_huge = (got[:, 3] >> 9 & 1).astype(bool) & (got[:, 0] >= 0)
                    assert np.array_equal(h_huge[got[is_huge, 3] >> 10, 0], got[is_huge, 0])
                # dense rows leave the staged plan to the others, and only a batch below theirs has one of all rows
                lengths = np.diff(ip)
                partial = 0 < n_short < m and int(lengths.max()) * m > 4 * int(ip[-1])
                plans = [nb.nerva_plan_staged_host(m, k, ip, ix, max_batch, e) for e in ((nb.NERVA_PACK_MAX_LEN + 1, 0) if partial else (0,))]
                ref_rows, ref_ends = next(((r, e) for r, e in plans if len(r)), plans[-1])
                dense = side == 0 and cols >= 1024 and max_batch >= 128 and (lengths >= max(cols // 8, 129)).sum() >= 17
                assert len(staged_rows) or side or (rows, cols) not in ((1200, 1500), (9000, 4000))
                if len(staged_rows) or not dense:
                    assert np.array_equal(staged_rows, ref_rows.ravel()), "staged rows"
                    assert np.array_equal(staged_ends, ref_ends.ravel()), "staged ends"
    finally:
        nb.nerva_set_dense_threshold(0.4)
    L.close()


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
