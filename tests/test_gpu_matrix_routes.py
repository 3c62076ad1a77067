"""The routes through the matrix instructions and the column tiles of wide batches, at the sizes where they can go wrong:
edges of tiles, remainders, the ends of their dispatch ranges.  Checked against the CPU oracle."""
import numpy as np
import pytest

from paper_2407_17437_amd import workloads as wl
from test_gpu_parity import close, layer_case, raw_f32, raw_i32

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nb():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2407_17437_amd import binding
    return binding


def routes(nb, lay, batch, max_batch=None):
    """The ways that calls of the layer take, as the library says."""
    L = nb.SparseLinear(lay, max_batch=max_batch or batch)
    taken = nb.sparse_linear_routes(L.handle, batch)
    L.close()
    return taken


def check_layer(nb, oracle, lay, batch, ld=None, max_batch=None, seed=1, backward=True):
    import torch
    rng = np.random.default_rng(seed)
    X = rng.standard_normal((lay.cols, batch)).astype(np.float32); dY = rng.standard_normal((lay.rows, batch)).astype(np.float32)
    L = nb.SparseLinear(lay, max_batch=max_batch or batch)
    Xd, dYd = nb.to_dense(X, ld=ld), nb.to_dense(dY, ld=ld)
    Yd, dXd = nb.dense(lay.rows, batch, ld=ld), nb.dense(lay.cols, batch, ld=ld)
    g, db = torch.full((lay.nnz,), float("nan"), device="cuda"), torch.full((lay.rows,), float("nan"), device="cuda")
    nb.sparse_linear_forward(L.handle, Xd, Yd, batch)
    torch.cuda.synchronize()
    Y, S = oracle.spmm(lay.rows, lay.cols, lay.indptr, lay.indices, lay.values, lay.bias, X, lay.relu)
    close(Yd.cpu().numpy(), Y, S, what="Y")
    if backward:
        nb.sparse_linear_backward(L.handle, Xd, Yd if lay.relu else None, dYd, dXd, g, db, batch)
        torch.cuda.synchronize()
        dZ = oracle.relu_backward(dY, Yd.cpu().numpy()) if lay.relu else dY
        dX, SdX = oracle.spmm_t(lay.rows, lay.cols, lay.indptr, lay.indices, lay.values, dZ)
        close(dXd.cpu().numpy(), dX, SdX, what="dX")
        gr, Sg, dbr, Sdb = oracle.sddmm(lay.rows, lay.cols, lay.indptr, lay.indices, dZ, X)
        close(g.cpu().numpy(), gr, Sg, what="dvalues")
        close(db.cpu().numpy(), dbr, Sdb, what="dbias")
    L.close()


@pytest.mark.parametrize("rows,cols,density,batch,ld", [
    (64, 64, 0.36, 16, None), (65, 127, 0.5, 17, 17), (129, 64, 1.0, 63, 63),      # few tiles: the narrowest batches, ragged tiles
    (100, 300, 0.35, 65, None), (300, 100, 0.38, 128, 129),
    (1500, 1410, 0.16, 100, None), (1473, 1409, 0.15, 67, 67),                     # 552 tiles, the last of them one row and one column
])
def test_sampled_gradient(nb, oracle, rows, cols, density, batch, ld):
    check_layer(nb, oracle, layer_case(rows, cols, density, seed=rows + batch), batch, ld=ld)


@pytest.mark.parametrize("rows,cols,batch,ld", [
    # slices of the sum that are empty, one chunk, whole rounds of chunks and one more; 1, 2 and 4 tiles of 16 columns to a work-group
    (16, 16, 1, None), (17, 33, 5, 5), (48, 80, 16, None), (1041, 129, 33, 33), (1024, 256, 100, None), (1039, 271, 99, 99),
    (1024, 320, 256, None), (1030, 330, 130, None), (1090, 61, 257, 257), (4081, 70, 16, None), (4097, 79, 15, 15),   # (256 work-groups of eight waves, 257 of four)
    # tiles of 64 columns shared by two and four work-groups, and tiles of 32 rows
    (1024, 1536, 65, None), (1041, 1551, 97, 97), (1024, 1792, 33, None), (1009, 1801, 63, 63), (2049, 3073, 200, None),
    # two and four tiles of columns in the transposed product
    (67, 2049, 257, 257), (70, 4100, 511, None), (65, 16384, 33, None), (66, 5500, 100, None), (66, 8192, 64, None),
])
def test_products_of_the_dense_copy(nb, oracle, rows, cols, batch, ld):
    check_layer(nb, oracle, layer_case(rows, cols, 0.6, seed=rows + batch), batch, ld=ld)


@pytest.mark.parametrize("rows,cols,batch", [(1041, 1551, 97), (1009, 1801, 63)])
def test_shared_tiles_of_the_dense_copy_come_out_the_same_again(nb, oracle, rows, cols, batch):
    """... whichever work-group was last, with an infinity in the operand's last row and with its neighbour NaN outside the batch."""
    import torch
    lay = layer_case(rows, cols, 0.6, seed=7, relu=False)
    rng = np.random.default_rng(3)
    X = rng.standard_normal((cols, batch)).astype(np.float32)
    L = nb.SparseLinear(lay, max_batch=batch)
    Xd = torch.full((cols, batch + 3), float("nan"), device="cuda")[:, :batch]
    Xd.copy_(torch.from_numpy(X))
    Ys = [nb.dense(rows, batch) for _ in range(4)]
    for Yd in Ys[:3]:
        nb.sparse_linear_forward(L.handle, Xd, Yd, batch)
    want, S = oracle.spmm(rows, cols, lay.indptr, lay.indices, lay.values, lay.bias, X, False)
    close(Ys[0].cpu().numpy(), want, S, what="Y")
    assert all(torch.equal(Ys[0], Yd) for Yd in Ys[1:3])
    Xd[cols - 1, 5] = float("inf")
    nb.sparse_linear_forward(L.handle, Xd, Ys[3], batch)
    held = np.arange(batch) != 5
    assert np.array_equal(Ys[3].cpu().numpy()[:, held], Ys[0].cpu().numpy()[:, held])
    stored = lay.indices[lay.indptr[1:][np.diff(lay.indptr) > 0] - 1] == cols - 1
    assert not np.isfinite(Ys[3].cpu().numpy()[np.diff(lay.indptr) > 0][stored, 5]).any()
    L.close()


def mixed_rows(rows, cols, n_dense, density, seed, relu=False):
    """n_dense rows that store `density` of their columns among short, empty and middling ones."""
    rng = np.random.default_rng(seed)
    lens = np.where(rng.random(rows) < 0.05, rng.integers(125, 137, rows), rng.integers(0, 30, rows))
    lens[rng.permutation(rows)[:n_dense]] = (density * cols + rng.integers(-20, 20, n_dense)).clip(1, cols).astype(np.int64)
    indptr, indices = wl.pattern_from_row_nnz(lens, cols, seed=seed)
    return wl.SparseLayerData(rows, cols, indptr, indices, wl.init_values(indptr, seed), rng.standard_normal(rows).astype(np.float32), relu)


@pytest.fixture
def dense_rows_at_any_batch(nb):
    nb.nerva_set_partition_mode(nb.NERVA_PARTITION_PREFER_DENSE_ROWS)
    yield
    nb.nerva_set_partition_mode(nb.NERVA_PARTITION_BALANCED)


@pytest.mark.usefixtures("dense_rows_at_any_batch")
@pytest.mark.parametrize("rows,cols,n_dense,density,batch,ld,relu", [
    (2300, 1300, 129, 0.6, 128, None, True),    # short rows packed; a row tile with one row
    (2300, 1345, 128, 1.0, 131, 131, False),    # full row tiles, full rows, a last step of one column
    (600, 1407, 200, 0.5, 300, 301, True),      # too few short rows to be packed
    (1000, 2049, 64, 0.9, 513, None, False),    # a batch that leaves one column over
    (130, 1500, 130, 0.7, 192, None, False),    # nothing but dense rows
    (20000, 1100, 300, 0.4, 129, 129, True),
])
def test_dense_rows(nb, oracle, rows, cols, n_dense, density, batch, ld, relu):
    # (bound for batches up to 4096, at which the dense rows are worth a launch of their own)
    check_layer(nb, oracle, mixed_rows(rows, cols, n_dense, density, rows + cols, relu), batch, ld=ld, max_batch=4096)


@pytest.mark.parametrize("batch", [130, 320, 448])
def test_dense_rows_on_either_side_of_their_batch(nb, oracle, batch):
    """550 thousand entries in dense rows, bound for 1024 columns: up to 366 columns they are staged with all the others, or
    gathered, from there on they go apart and the others are staged alone."""
    rng = np.random.default_rng(8)
    lens = rng.integers(180, 220, 16384)
    lens[rng.permutation(16384)[:500]] = 1100
    indptr, indices = wl.pattern_from_row_nnz(lens, 2048, seed=9)
    check_layer(nb, oracle, wl.SparseLayerData(16384, 2048, indptr, indices, wl.init_values(indptr, 7), np.zeros(16384, np.float32), False), batch, max_batch=1024)


@pytest.mark.usefixtures("dense_rows_at_any_batch")
def test_dense_rows_keep_a_non_finite_operand_row_to_the_rows_that_read_it(nb, oracle):
    import torch
    lay, batch = mixed_rows(900, 1300, 150, 0.5, 3), 256
    X = np.random.default_rng(4).standard_normal((lay.cols, batch)).astype(np.float32)
    Xf = X.copy()
    odd = (0, 63, 64, 700, 1299)
    X[odd, :] = np.inf
    X[700, :] = np.nan
    Xf[odd, :] = 0.0
    L = nb.SparseLinear(lay, max_batch=4096)
    Yd = nb.dense(lay.rows, batch)
    nb.sparse_linear_forward(L.handle, nb.to_dense(X), Yd, batch)
    torch.cuda.synchronize()
    Y = Yd.cpu().numpy()
    touched = np.zeros(lay.rows, dtype=bool)
    touched[np.repeat(np.arange(lay.rows), np.diff(lay.indptr))[np.isin(lay.indices, odd)]] = True
    Yr, S = oracle.spmm(lay.rows, lay.cols, lay.indptr, lay.indices, lay.values, lay.bias, Xf, False)
    close(Y[~touched], Yr[~touched], S[~touched], what="rows that do not reference the odd rows")
    assert (~touched & (np.diff(lay.indptr) > 500)).any() and not np.isfinite(Y[touched]).all(axis=1).any()
    L.close()


SPLIT_SHAPES = [   # rows, columns, dense rows, their density, batch, leading dimension, ReLU: on the bf16 units (test_host_memory)
    (2500, 1057, 1030, 0.6, 1024, None, True),    # a row tile of six rows, a last chunk of one column, slices, short rows besides
    (5000, 1030, 5000, 0.36, 193, 193, False),     # nothing but dense rows; a column tile of 193 of 256 columns
    (1400, 2310, 1281, 0.42, 771, 773, False),     # row and column tiles of one row and of three columns
    (4000, 1060, 4000, 0.35, 2000, None, True),   # as many tiles as compute units: no slices
]


@pytest.mark.usefixtures("dense_rows_at_any_batch")
@pytest.mark.parametrize("rows,cols,n_dense,density,batch,ld,relu", SPLIT_SHAPES)
def test_dense_rows_on_the_bf16_units(nb, oracle, rows, cols, n_dense, density, batch, ld, relu):
    check_layer(nb, oracle, mixed_rows(rows, cols, n_dense, density, rows + cols, relu), batch, ld=ld, backward=False)


@pytest.mark.usefixtures("dense_rows_at_any_batch")
def test_dense_rows_on_the_bf16_units_with_infinities(nb, oracle):
    """Numbers that are not finite, or that round to an infinity in bf16, in the operand and among the weights: entries that are
    not stored do not meet them, and what is stored gives what fp32 gives."""
    import torch
    lay, batch = mixed_rows(2500, 1057, 1030, 0.6, 3), 1024
    X = np.random.default_rng(4).standard_normal((lay.cols, batch)).astype(np.float32)
    X[(0, 31, 32, 700, 1056), :] = np.array([np.inf, -np.inf, 3.4e38, np.nan, np.inf], np.float32)[:, None]
    X[500, 77] = np.inf
    dense = np.flatnonzero(np.diff(lay.indptr) > 500)
    for row, v in zip(dense[[0, 5, 200, 1029]], (np.inf, np.nan, -3.4e38, -np.inf)):
        lay.values[(lay.indptr[row] + lay.indptr[row + 1]) // 2] = v
    L = nb.SparseLinear(lay, max_batch=batch)
    Yd = nb.dense(lay.rows, batch)
    nb.sparse_linear_forward(L.handle, nb.to_dense(X), Yd, batch)
    torch.cuda.synchronize()
    Y = Yd.cpu().numpy()
    with np.errstate(all="ignore"):
        for row in range(lay.rows):
            at = slice(lay.indptr[row], lay.indptr[row + 1])
            terms = lay.values[at, None].astype(np.float64) * X[lay.indices[at]]
            terms = np.where(np.abs(terms) > np.finfo(np.float32).max, np.sign(terms) * np.inf, terms)
            ref, S = terms.sum(0) + lay.bias[row], np.abs(terms).sum(0) + abs(lay.bias[row])
            large = S > 1e37   # (sums of numbers near the end of the range may pass it in one order and not in another)
            fine = np.isfinite(S) & ~large
            np.testing.assert_allclose(Y[row, fine], ref[fine], rtol=0, atol=float((1e-5 * S[fine]).max(initial=0.0)))
            assert not np.isfinite(Y[row, ~np.isfinite(S)]).any(), row
            gone = np.isnan(ref) & ~large
            assert np.isnan(Y[row, gone]).all(), row
    assert np.isfinite(Y).any() and not np.isfinite(Y).all()
    L.close()


@pytest.mark.usefixtures("dense_rows_at_any_batch")
@pytest.mark.parametrize("small", ["operand", "weights"])
def test_dense_rows_on_the_bf16_units_with_small_numbers(nb, oracle, small):
    """Numbers down to the end of the normal range, of which three bf16 numbers do not hold all bits: columns of the operand, or rows of
    the matrix, of very different scales.  Relative to the terms of each result, as everywhere."""
    import torch
    lay, batch = mixed_rows(2500, 1057, 1030, 0.6, 3), 1024
    lay.bias[:] = 0
    rng = np.random.default_rng(4)
    X = rng.standard_normal((lay.cols, batch)).astype(np.float32)
    scale = np.float32(10.0) ** -np.array([0, 30, 32, 33, 34, 35, 36], np.float32)
    if small == "operand":
        X *= scale[np.arange(batch) * 7 // batch][None, :]
        X[:, :5] *= scale[2:7]   # (and next to the ordinary ones)
    else:
        lay.values *= np.repeat(scale[rng.integers(0, 7, lay.rows)], np.diff(lay.indptr))
    L = nb.SparseLinear(lay, max_batch=batch)
    Yd = nb.dense(lay.rows, batch)
    nb.sparse_linear_forward(L.handle, nb.to_dense(X), Yd, batch)
    torch.cuda.synchronize()
    Y, S = oracle.spmm(lay.rows, lay.cols, lay.indptr, lay.indices, lay.values, lay.bias, X, False)
    close(Yd.cpu().numpy(), Y, S, what="Y", tol=1e-6)   # (fp32 sums of 640 terms; the parts alone are off by 1e-3 at 1e-36)
    L.close()


@pytest.mark.usefixtures("dense_rows_at_any_batch")
@pytest.mark.parametrize("kind", ["normal", "one sign", "one term"])
def test_dense_rows_on_the_bf16_units_are_no_further_off_than_fp32_sums(nb, kind):
    """Against 64 bits, beside a chain of fp32 sums: ordinary numbers, numbers of one sign (a biased rounding would show) and results of a
    single product, which fp32 rounds once: 2^-24, and the product left out adds 2^-32 to it."""
    import torch
    lay, batch = mixed_rows(2500, 1057, 1030, 0.6, 3), 1024
    lay.bias[:] = 0
    X = np.random.default_rng(4).standard_normal((lay.cols, batch)).astype(np.float32)
    if kind == "one sign":
        X, lay.values[:] = np.abs(X), np.abs(lay.values)
    elif kind == "one term":
        X *= np.arange(lay.cols)[:, None] == np.arange(batch)[None, :]
    L = nb.SparseLinear(lay, max_batch=batch)
    Yd = nb.dense(lay.rows, batch)
    nb.sparse_linear_forward(L.handle, nb.to_dense(X), Yd, batch)
    torch.cuda.synchronize()
    Y = Yd.cpu().numpy().astype(np.float64)
    mine = chain = norm = worst = 0.0
    for row in np.flatnonzero(np.diff(lay.indptr) > 500)[::40]:
        at = slice(lay.indptr[row], lay.indptr[row + 1])
        w, x = lay.values[at], X[lay.indices[at]]
        want, s = w.astype(np.float64) @ x.astype(np.float64), np.zeros(batch, np.float32)
        for k in range(w.size):
            s += w[k] * x[k]
        mine, chain, norm = mine + ((Y[row] - want) ** 2).sum(), chain + ((s - want) ** 2).sum(), norm + (want ** 2).sum()
        worst = max(worst, float((np.abs(Y[row] - want) / np.maximum(np.abs(want), 1e-30)).max()))
    if kind == "one term":
        assert mine <= chain * 1.01 and worst <= 2.0 ** -24 * (1 + 2.0 ** -6), (np.sqrt(mine / norm), np.sqrt(chain / norm), worst)
    else:
        assert mine <= chain, (np.sqrt(mine / norm), np.sqrt(chain / norm))
    L.close()


@pytest.mark.parametrize("low,high,batches", [
    (560, 609, (300, 600)),   # 28 % of 2100 columns, bound for 600: gathered at 300, on the bf16 units at 600 (test_host_memory)
    (390, 450, (300, 470)),   # 20 %, bound for 470: long enough rows, but no batch pays
])
def test_uniform_rows_on_the_bf16_units(nb, oracle, low, high, batches):
    rng = np.random.default_rng(12)
    indptr, indices = wl.pattern_from_row_nnz(rng.integers(low, high, 2050), 2100, seed=9)
    lay = wl.SparseLayerData(2050, 2100, indptr, indices, wl.init_values(indptr, 7), rng.standard_normal(2050).astype(np.float32), True)
    for batch in batches:
        check_layer(nb, oracle, lay, batch, max_batch=batches[1])


@pytest.mark.parametrize("batch", [16, 32, 64, 128])
def test_both_gradients_in_one_tile_of_more_waves_than_fit_at_once(nb, oracle, batch):
    """2125, 4250 and 8500 waves: two or three gathers in flight (test_host_memory)."""
    check_layer(nb, oracle, layer_case(60, 17000, 0.01, seed=batch), batch)


@pytest.mark.parametrize("batch", [64, 128])
@pytest.mark.parametrize("rows,cols,lens", [(900, 301, range(3, 60)), (700, 640, [21]), (640, 1200, [33, 20, 31]), (2500, 77, [390, 400, 65]), (500, 2, [399, 401]), (5000, 8200, [21, 24]),
                                            (1000, 900, [20]), (5000, 500, [401])])
def test_both_gradients_in_chunks_of_sixteen(nb, oracle, rows, cols, lens, batch):
    """One tile in groups of 16 or 32 lanes, mirror rows of 1 to 25 chunks and every remainder, alone in a wave and shared by groups; the last two and the longest matrix lie beyond the rule.
    Infinities in dZ reach the entries that read them as infinities also where a row's number of entries is odd."""
    import torch
    lens = np.resize(np.asarray(list(lens)), cols)
    tp, ti = wl.pattern_from_row_nnz(lens, rows, seed=cols)   # the mirror's rows
    order = np.lexsort((np.repeat(np.arange(cols), lens), ti))
    indptr = np.concatenate([[0], np.cumsum(np.bincount(ti, minlength=rows))]).astype(tp.dtype)
    lay = wl.SparseLayerData(rows, cols, indptr, np.repeat(np.arange(cols), lens)[order].astype(ti.dtype), wl.init_values(indptr, 5), np.zeros(rows, np.float32), False)
    check_layer(nb, oracle, lay, batch)
    rng = np.random.default_rng(1)
    dY, X = (rng.standard_normal((n, batch)).astype(np.float32) for n in (rows, cols))
    dY[np.argmax(np.diff(indptr)), 5] = np.inf
    ref, S = oracle.spmm_t(rows, cols, lay.indptr, lay.indices, lay.values, np.where(np.isinf(dY), 0, dY))
    L = nb.SparseLinear(lay, max_batch=batch)
    dX, g, db = nb.dense(cols, batch), torch.empty(lay.nnz, device="cuda"), torch.empty(rows, device="cuda")
    nb.sparse_linear_backward(L.handle, nb.to_dense(X), None, nb.to_dense(dY), dX, g, db, batch)
    torch.cuda.synchronize()
    hit = np.zeros(ref.shape, dtype=bool)
    bad = np.nonzero(np.isinf(dY))[0][0]
    hit[lay.indices[indptr[bad]:indptr[bad + 1]], 5] = True
    got = dX.cpu().numpy()
    assert not np.isfinite(got[hit]).any()
    if len(set(lens.tolist())) == 1:   # (rows side by side in a wave are as long)
        assert np.isinf(got[hit]).all()
    close(np.where(hit, 0, got), np.where(hit, 0, ref), np.where(hit, 1, S), what="dX beside infinities")
    L.close()


def test_huge_rows_after_products_that_overlapped(nb, oracle):
    """Products of one layer on several streams at once may spoil one another (their results are not looked at), but no product
    that is ordered after them: the shares of its huge rows are counted from 0 again, in both orientations."""
    import torch
    rng = np.random.default_rng(3)
    rows, cols, batch = 5000, 6000, 100
    lens = np.full(rows, 3)
    lens[::125] = rng.integers(2000, 5900, 40)
    indptr, indices = wl.pattern_from_row_nnz(lens, cols, seed=4)
    for i in np.nonzero(lens == 3)[0]:
        indices[indptr[i]:indptr[i + 1]] = np.sort(rng.choice(10, 3, replace=False))   # ten columns of 1500 entries
    lay = wl.SparseLayerData(rows, cols, indptr, indices, wl.init_values(indptr, 5), np.zeros(rows, np.float32), False)
    L = nb.SparseLinear(lay, max_batch=batch)
    X, dY = (rng.standard_normal((n, batch)).astype(np.float32) for n in (cols, rows))
    Xd, dYd = nb.to_dense(X), nb.to_dense(dY)
    Ys, dXs = [nb.dense(rows, batch) for _ in range(3)], [nb.dense(cols, batch) for _ in range(3)]
    streams = [torch.cuda.Stream() for _ in Ys]
    torch.cuda.synchronize()
    for _ in range(100):
        for s, Y, dX in zip(streams, Ys, dXs):
            nb.sparse_linear_forward(L.handle, Xd, Y, batch, s)
            nb.sparse_linear_backward(L.handle, None, None, dYd, dX, None, None, batch, s)
    torch.cuda.synchronize()
    nb.sparse_linear_forward(L.handle, Xd, Ys[0], batch)
    nb.sparse_linear_backward(L.handle, None, None, dYd, dXs[0], None, None, batch)
    torch.cuda.synchronize()
    Y, S = oracle.spmm(rows, cols, indptr, indices, lay.values, lay.bias, X, False)
    close(Ys[0].cpu().numpy(), Y, S, what="Y")
    dX, S = oracle.spmm_t(rows, cols, indptr, indices, lay.values, dY)
    close(dXs[0].cpu().numpy(), dX, S, what="dX")
    L.close()


def test_shared_tiles_after_products_that_overlapped(nb, oracle):
    """The same of tiles of the dense copy that work-groups share, two at some batches and four at others, all of them in flight at once."""
    import torch
    rows, cols, batches = 1024, 1801, (100, 64, 97, 33)
    lay = layer_case(rows, cols, 0.6, seed=8, relu=False)
    rng = np.random.default_rng(9)
    L = nb.SparseLinear(lay, max_batch=100)
    Xs = [rng.standard_normal((cols, batch)).astype(np.float32) for batch in batches]
    Xd, Yd = [nb.to_dense(X) for X in Xs], [nb.dense(rows, batch) for batch in batches]
    streams = [torch.cuda.Stream() for _ in batches]
    torch.cuda.synchronize()
    for _ in range(200):
        for s, X, Y, batch in zip(streams, Xd, Yd, batches):
            nb.sparse_linear_forward(L.handle, X, Y, batch, s)
    torch.cuda.synchronize()
    for X, x, Y, batch in zip(Xs, Xd, Yd, batches):
        Y.fill_(float("nan"))
        nb.sparse_linear_forward(L.handle, x, Y, batch)
        torch.cuda.synchronize()
        want, S = oracle.spmm(rows, cols, lay.indptr, lay.indices, lay.values, lay.bias, X, False)
        close(Y.cpu().numpy(), want, S, what=f"Y at batch {batch}")
    L.close()


def with_infinities(rng, features, batch):
    """Every third row holds an infinity: in the first column, which idle lanes re-read, or in one of the last four, which the lanes
    of a ragged batch share."""
    M = rng.standard_normal((features, batch)).astype(np.float32)
    at = np.arange(0, features, 3)
    M[at, np.where(at % 2 == 0, 0, np.maximum(batch - 1 - at % 4, 0))] = np.where(at % 5 == 0, -np.inf, np.inf)
    return M


@pytest.mark.parametrize("rows,cols,density,batch,relu,dx", [
    # gathered entry by entry: every number of lanes per entry and of columns per lane
    *[(150, 260, 0.1, batch, False, False) for batch in (5, 16, 21, 33, 50, 63, 77, 97, 100, 129, 150, 193, 257, 385, 513, 769, 1023)],
    (700, 9000, 0.002, 101, False, False), (2100, 13000, 0.001, 650, False, False),   # column tiles
    (600, 700, 0.4, 67, False, False), (600, 700, 0.4, 130, False, True),    # sampled from the matrix units' tiles
    (10, 400, 1.0, 70, False, False), (10, 400, 1.0, 301, False, False),     # a full matrix of few rows
    # with the other gradient, on one gather stream: a single tile, rows through all tiles, several tiles; masked by the output
    (300, 500, 0.05, 6, False, True), (300, 500, 0.05, 41, True, True), (300, 500, 0.05, 101, False, True), (300, 500, 0.05, 203, True, True),
    (700, 1000, 0.04, 301, False, True), (700, 1000, 0.02, 302, True, True), (3000, 700, 0.02, 999, False, True),
    (900, 2000, "staged", 259, False, False), (900, 2000, "staged", 449, False, False),
])
def test_infinities_reach_the_gradients_of_their_own_columns(nb, rows, cols, density, batch, relu, dx):
    """An entry's gradient is the sum over the batch's columns, whatever the lanes that have none of them re-read: infinite where
    one product is, and NaN only where two of them cancel or one is 0 times infinity."""
    import torch
    staged = density == "staged"
    lay = layer_case(rows, cols, 0.02 if staged else density, seed=rows + batch, relu=relu)
    rng = np.random.default_rng(batch)
    X, dY = with_infinities(rng, cols, batch), with_infinities(rng, rows, batch)
    Y = rng.standard_normal((rows, batch)).astype(np.float32)
    if staged:
        nb.nerva_set_partition_mode(nb.NERVA_PARTITION_PREFER_STAGED)
    try:
        L = nb.SparseLinear(lay, max_batch=batch)
    finally:
        nb.nerva_set_partition_mode(nb.NERVA_PARTITION_BALANCED)
    g, db = torch.full((lay.nnz,), 7.0, device="cuda"), torch.full((rows,), 7.0, device="cuda")
    nb.sparse_linear_backward(L.handle, nb.to_dense(X, ld=batch), nb.to_dense(Y, ld=batch) if relu else None, nb.to_dense(dY, ld=batch),
                              nb.dense(cols, batch, ld=batch) if dx else None, g, db, batch)
    torch.cuda.synchronize()
    dZ = np.where(Y > 0, dY, np.float32(0)).astype(np.float64) if relu else dY.astype(np.float64)
    with np.errstate(invalid="ignore"):
        products = dZ[np.repeat(np.arange(rows), np.diff(lay.indptr))] * X[lay.indices].astype(np.float64)
        for what, got, ref, S in (("dvalues", g, products.sum(1), np.abs(products).sum(1)), ("dbias", db, dZ.sum(1), np.abs(dZ).sum(1))):
            got, fine = got.cpu().numpy(), np.isfinite(ref)
            assert fine.any() and np.isinf(ref).any()
            close(got[fine], ref[fine], S[fine], what=what)
            assert np.array_equal(got[~fine], ref[~fine].astype(np.float32), equal_nan=True), what
    L.close()


@pytest.mark.parametrize("rows,batch", [(2600, 1024), (2600, 1001), (700, 1024)])
def test_huge_rows_in_column_tiles(nb, oracle, rows, batch):
    """Rows cut into 3, 4, 5, 6, 9, ... 36 work-groups per tile, the shares added by one wave; beside packed rows and without."""
    rng = np.random.default_rng(batch)
    lens = rng.integers(0, 20, rows)
    lens[rng.permutation(rows)[:11]] = [513, 768, 769, 1024, 1025, 1280, 1281, 2049, 4000, 8999, 9000]
    indptr, indices = wl.pattern_from_row_nnz(lens, 9000, seed=rows)
    lay = wl.SparseLayerData(rows, 9000, indptr, indices, wl.init_values(indptr, 1), rng.standard_normal(rows).astype(np.float32), True)
    check_layer(nb, oracle, lay, batch, ld=batch)


@pytest.mark.parametrize("batch", [257, 300, 320, 385, 511, 512, 513, 640, 1023, 1024, 1025])
def test_wide_batches_in_column_tiles(nb, oracle, batch):
    # (operands of 300 rows, which no rule tiles; rows cut over several waves and several work-groups)
    rng = np.random.default_rng(batch)
    lens = np.where(rng.random(120) < 0.1, 300, rng.integers(0, 40, 120))
    indptr, indices = wl.pattern_from_row_nnz(lens, 300, seed=batch)
    lay = wl.SparseLayerData(120, 300, indptr, indices, wl.init_values(indptr, 1), rng.standard_normal(120).astype(np.float32), True)
    check_layer(nb, oracle, lay, batch, ld=batch if batch % 2 else None)


@pytest.mark.parametrize("rows,cols,density,batch,ld,relu", [
    (40, 3000, 0.02, 5, 5, False), (40, 3000, 0.02, 32, None, True), (3000, 40, 0.02, 33, 33, False),     # lane groups of 8 and 16
    (900, 500, 0.05, 64, None, True), (900, 500, 0.3, 65, 65, False), (500, 900, 0.01, 128, None, False),  # one tile of 64 and 128 columns
    (700, 1000, 0.04, 129, 129, False), (700, 1000, 0.04, 256, None, True),                                # one tile of 256
    (6000, 700, 0.01, 200, None, False), (700, 1000, 0.04, 257, 257, True), (600, 9000, 0.005, 700, None, False),   # several tiles
    (700, 1000, 0.03, 300, None, True), (300, 2000, 0.02, 1025, 1025, False), (300, 2000, 0.02, 513, None, True),   # rows through all tiles
    (9000, 400, 0.02, 16, None, False), (3, 1500, 0.5, 100, None, False),   # rows shared by lane groups; hardly any rows to sum
])
def test_both_gradients_in_one_pass(nb, oracle, rows, cols, density, batch, ld, relu):
    lay = layer_case(rows, cols, density, seed=rows + cols + batch, relu=relu)
    check_layer(nb, oracle, lay, batch, ld=ld)
    # the mirror's values follow values[] in the same call
    import torch
    L = nb.SparseLinear(lay, max_batch=batch)
    L.values.mul_(3.0)
    X, Y, dY, dX = (nb.dense(n, batch) for n in (cols, rows, rows, cols))
    for t in (X, Y, dY):
        t.normal_()
    g, db = torch.empty(lay.nnz, device="cuda"), torch.empty(rows, device="cuda")
    nb.sparse_linear_backward(L.handle, X, Y if relu else None, dY, dX, g, db, batch)
    torch.cuda.synchronize()
    _, _, v_t, perm = nb.sparse_linear_mirror(L.handle)
    assert np.array_equal(raw_f32(nb, torch, v_t, lay.nnz), L.values.cpu().numpy()[raw_i32(nb, torch, perm, lay.nnz)])
    L.close()


@pytest.mark.parametrize("relu", [False, True])
@pytest.mark.parametrize("nnz", [1, 2048, 2049, 70001, (1 << 20) - 1, 1 << 20, (1 << 20) + 1025])
def test_mirror_values_follow_the_weights(nb, nnz, relu):
    """Weights changed by the caller reach every mirror entry before the transposed product: numbers of entries about whole turns of the
    launch's work-groups, and about where a thread begins to bring four."""
    import torch
    rows, cols, batch = 3001, 2000, 12
    indptr, indices = wl.uniform_pattern(rows, cols, nnz, nnz)
    lay = wl.SparseLayerData(rows, cols, indptr, indices, wl.init_values(indptr, 1), np.zeros(rows, np.float32), relu)
    L = nb.SparseLinear(lay, max_batch=batch)
    L.values.normal_()
    X, Y, dY, dX = nb.dense(cols, batch), nb.dense(rows, batch), nb.dense(rows, batch), nb.dense(cols, batch)
    for t in (X, dY):
        t.normal_()
    nb.sparse_linear_forward(L.handle, X, Y, batch)
    nb.sparse_linear_backward(L.handle, X, Y if relu else None, dY, dX, None, None, batch)
    torch.cuda.synchronize()
    _, _, v_t, perm = nb.sparse_linear_mirror(L.handle)
    assert np.array_equal(raw_f32(nb, torch, v_t, nnz), L.values.cpu().numpy()[raw_i32(nb, torch, perm, nnz)])
    L.close()


@pytest.mark.parametrize("batch,hidden", [(60, (2000, 1500)), (64, (2000, 3000)), (200, (900, 1300)), (300, (1100, 1000))])
def test_training_step_with_both_gradients_in_one_pass(nb, batch, hidden):
    """Against the same step by separate products: one and several column tiles, momentum applied inside the pass and after it."""
    import torch
    data = wl.make_mlp((300,) + hidden + (10,), sparsity=0.9)
    X, labels = nb.dense(300, batch), torch.randint(10, (batch,), device="cuda", dtype=torch.int32)
    X.normal_()
    out = []
    for flags in (nb.NERVA_MLP_DEFAULT, nb.NERVA_MLP_UNFUSED):
        m = nb.MLP(data, batch, flags)
        for _ in range(3):
            m.train_step(X, labels, batch, 0.05, 0.9)
        torch.cuda.synchronize()
        out.append([t.clone() for l in m.layers for t in (l.values, l.velocity, l.bias, l.bias_velocity)] + [m.loss.clone()])
        m.close()
    for a, b in zip(*out):
        assert torch.allclose(a, b, rtol=1e-3, atol=2e-6 * max(1.0, float(b.abs().max())))


@pytest.mark.parametrize("flags", ["plain", "nesterov"])
@pytest.mark.parametrize("batch,max_batch", [(640, 640), (577, 640)])
def test_training_step_with_dense_rows_above_the_first_layer(nb, batch, max_batch, flags):
    """Their gradients, the momentum step and the new weights' places in the mirror come from the matrix units' launch, the other
    rows' from theirs: against the same step by separate products."""
    import types
    import torch
    upper = mixed_rows(3000, 1500, 420, 0.6, 11, relu=True)
    first, last = layer_case(1500, 200, 0.1, 12, relu=True), layer_case(10, 3000, 0.2, 13)
    data = types.SimpleNamespace(layers=[first, upper, last])
    X, labels = nb.dense(200, batch), torch.randint(10, (batch,), device="cuda", dtype=torch.int32)
    X.normal_()
    extra = nb.NERVA_MLP_NESTEROV if flags == "nesterov" else 0
    out = []
    for how in (nb.NERVA_MLP_DEFAULT, nb.NERVA_MLP_UNFUSED):
        m = nb.MLP(data, max_batch, how | extra)
        for _ in range(3):
            m.train_step(X, labels, batch, 0.05, 0.9)
        torch.cuda.synchronize()
        out.append([t.clone() for l in m.layers for t in (l.values, l.velocity, l.bias, l.bias_velocity)] + [m.loss.clone()])
        L = m.layers[1]
        _, _, v_t, perm = nb.sparse_linear_mirror(L.handle)
        assert np.array_equal(raw_f32(nb, torch, v_t, L.nnz), L.values.cpu().numpy()[raw_i32(nb, torch, perm, L.nnz)])
        if how == nb.NERVA_MLP_DEFAULT:   # (not the launch that forms both gradients on one gather stream)
            nb.mlp_profile_enable(m.handle, 1)
            m.train_step(X, labels, batch, 0.0, 0.0)
            names = [name for name, _ in nb.mlp_profile_read(m.handle)[1]]
            assert "sddmm_update[1]" in names and "spmm_transposed[1]" in names, names
        m.close()
    for a, b in zip(*out):
        assert torch.allclose(a, b, rtol=1e-3, atol=2e-6 * max(1.0, float(b.abs().max())))


@pytest.mark.parametrize("classes,batch", [(16, 65), (17, 1), (17, 64), (33, 129), (128, 63), (129, 512), (300, 513), (100, 1025)])
def test_softmax_of_many_classes(nb, oracle, classes, batch):
    import torch
    rng = np.random.default_rng(classes)
    Z = (rng.standard_normal((classes, batch)) * 3).astype(np.float32)
    labels = rng.integers(0, classes, size=batch).astype(np.int32)
    ref, Sl, dZr, SdZ = oracle.softmax_ce(Z, labels)
    lab = torch.as_tensor(labels).cuda()
    Zd, dZd = nb.to_dense(Z), nb.dense(classes, batch)
    for out in (dZd, Zd):   # apart, in place
        loss = torch.zeros(1, device="cuda")
        nb.softmax_cross_entropy(Zd, lab, classes, batch, out, loss)
        torch.cuda.synchronize()
        close(out.cpu().numpy(), dZr, SdZ, what="dZ")
        assert abs(float(loss.item()) - ref) <= 1e-5 * Sl


@pytest.mark.parametrize("batch", [5, 15, 16, 17, 31, 32, 33, 48, 49, 77, 96, 97, 129, 192, 193, 257, 384, 385, 513, 768, 769])
def test_lane_groups_of_every_batch(nb, oracle, batch):
    # rows of every class: shared by 1 to 16 waves, and cut into work-groups
    lens = np.concatenate([np.arange(0, 300, 7), [1, 63, 64, 65, 900, 1400, 1400]])
    indptr, indices = wl.pattern_from_row_nnz(lens, 1400, seed=batch)
    lay = wl.SparseLayerData(len(lens), 1400, indptr, indices, wl.init_values(indptr, 1), np.ones(len(lens), np.float32), batch % 2 == 0)
    check_layer(nb, oracle, lay, batch, ld=batch)


@pytest.mark.parametrize("rows,cols,density,batch,relu", [
    (1000, 1000, 0.53, 1, True), (9000, 700, 0.09, 3, False), (700, 9000, 0.09, 4, True), (33, 70000, 0.25, 2, False),
])
def test_one_to_four_examples_on_many_entries(nb, oracle, rows, cols, density, batch, relu):
    nb.nerva_set_dense_threshold(2.0)
    try:
        check_layer(nb, oracle, layer_case(rows, cols, density, seed=rows, relu=relu), batch, ld=batch)
    finally:
        nb.nerva_set_dense_threshold(0.4)


def strips_case(rows, cols, lens, seed):
    """A layer whose row i has lens(i) entries, at most `cols`."""
    rng = np.random.default_rng(seed)
    per_row = [np.sort(rng.choice(cols, min(cols, int(lens(i))), replace=False)) for i in range(rows)]
    indptr = np.concatenate([[0], np.cumsum([len(r) for r in per_row])]).astype(np.int32)
    indices = np.concatenate(per_row).astype(np.int32)
    return wl.SparseLayerData(rows, cols, indptr, indices, rng.standard_normal(len(indices)).astype(np.float32), rng.standard_normal(rows).astype(np.float32), bool(seed % 2))


@pytest.fixture()
def prefer_strips(nb):
    nb.nerva_set_partition_mode(nb.NERVA_PARTITION_PREFER_STRIPS)
    yield
    nb.nerva_set_partition_mode(nb.NERVA_PARTITION_BALANCED)


@pytest.mark.parametrize("rows,cols,lens,batch,ld", [
    (1, 256, lambda i: 3, 193, None), (17, 257, lambda i: i, 194, 195), (16, 300, lambda i: 0 if i else 1, 200, None),     # the fewest; empty rows; one entry
    (300, 2048, lambda i: i % 41, 208, None), (255, 2049, lambda i: i % 75, 207, 207),                                    # one block and two; every length of a chunk's rest
    (2049, 4097, lambda i: 20 + i % 7, 193, 193), (700, 3072, lambda i: 40 if i % 3 else 90, 321, None),                  # three blocks; a set more than a range of a single one
    (130, 9001, lambda i: 1200 - i, 195, 199), (4500, 700, lambda i: 12, 1023, None), (900, 1500, lambda i: 30, 1026, 1027),   # long segments; batches beyond 1024
])
def test_product_in_strips(nb, oracle, prefer_strips, rows, cols, lens, batch, ld):
    check_layer(nb, oracle, strips_case(rows, cols, lens, rows + batch), batch, ld=ld, backward=False)


@pytest.mark.parametrize("rows,cols,lens,batch", [case[:4] for case in test_product_in_strips.pytestmark[0].args[1]])
def test_matrices_of_the_strips_tests_take_strips(nb, prefer_strips, rows, cols, lens, batch):
    assert routes(nb, strips_case(rows, cols, lens, rows + batch), batch) & nb.NERVA_ROUTE_FORWARD_STRIPS


def test_product_in_strips_where_the_rule_takes_it(nb, oracle):
    """The layer sizes at which strips are the library's own choice, bound for a wider batch than it is called with; then another pattern, and the weights of that changed."""
    rows, cols, batch = 6001, 2999, 811
    lay = layer_case(rows, cols, 0.014, seed=3, relu=True)
    check_layer(nb, oracle, lay, batch, ld=813, max_batch=1024, backward=False)
    check_layer(nb, oracle, lay, 64, max_batch=1024, backward=False)


def test_product_in_strips_through_changed_weights_and_patterns(nb, oracle):
    """The layer sizes at which strips are the library's own choice, bound for a wider batch than it is called with: one handle through weights that change in place, a pattern of more entries, whose
    stream is longer, one of fewer, and one of so few that the product goes another way; and narrower batches between."""
    import torch
    rows, cols, ld = 6001, 2999, 813
    X = np.random.default_rng(2).standard_normal((cols, 811)).astype(np.float32)
    Xd = nb.to_dense(X, ld=ld)
    lay = layer_case(rows, cols, 0.014, seed=3, relu=True)
    L = nb.SparseLinear(lay, max_batch=1024)

    def check(indptr, indices, what, strips=True):
        values = L.values.cpu().numpy()
        for batch in (811, 64):
            assert nb.sparse_linear_routes(L.handle, batch) & nb.NERVA_ROUTE_FORWARD_STRIPS == (strips and batch == 811), what
            Yd = nb.dense(rows, batch, ld=ld)
            Yd.fill_(float("nan"))
            nb.sparse_linear_forward(L.handle, Xd, Yd, batch)
            torch.cuda.synchronize()
            Y, S = oracle.spmm(rows, cols, indptr, indices, values, lay.bias, np.ascontiguousarray(X[:, :batch]), True)
            close(Yd[:, :batch].cpu().numpy(), Y, S, what=f"{what}, batch {batch}")

    check(lay.indptr, lay.indices, "as created")
    L.values.mul_(-0.5)
    check(lay.indptr, lay.indices, "weights changed in place")
    for density in (0.022, 0.012, 0.002):
        new = layer_case(rows, cols, density, seed=int(1000 * density))
        L.rebind(new.indptr, new.indices, new.values)
        check(new.indptr, new.indices, f"rebound at {density}", strips=density > 0.002)
    L.values.add_(0.25)
    check(new.indptr, new.indices, "weights of the last pattern changed", strips=False)
    L.rebind(lay.indptr, lay.indices, lay.values)
    check(lay.indptr, lay.indices, "rebound as created")
    L.close()


def test_product_in_strips_keeps_a_non_finite_operand_row_to_the_rows_that_read_it(nb, oracle, prefer_strips):
    """As of the staged product: lanes without an entry gather a row of zeros and not the first operand row of a block (0; 4608 - 1536, where the last block starts; 1536)."""
    import torch
    rows, cols, batch, bad = 500, 4600, 200, (0, 1536, 3064, 3072, 4599)
    lay = strips_case(rows, cols, lambda i: i % 50, 8)
    X = np.random.default_rng(5).standard_normal((cols, batch)).astype(np.float32)
    X[list(bad)] = np.inf
    L = nb.SparseLinear(lay, max_batch=batch)
    Yd = nb.dense(rows, batch)
    nb.sparse_linear_forward(L.handle, nb.to_dense(X), Yd, batch)
    torch.cuda.synchronize()
    Y = Yd.cpu().numpy()
    touched = np.zeros(rows, dtype=bool)
    touched[np.repeat(np.arange(rows), np.diff(lay.indptr))[np.isin(lay.indices, bad)]] = True
    assert touched.any() and np.isfinite(Y[~touched]).all() and not np.isfinite(Y[touched]).all(axis=1).any()
    X[list(bad)] = 0
    Yr, S = oracle.spmm(rows, cols, lay.indptr, lay.indices, lay.values, lay.bias, X, False)
    close(Y[~touched], Yr[~touched], S[~touched], what="rows that do not read them")
    L.close()


def test_training_step_in_strips_on_new_patterns(nb, oracle, prefer_strips):
    """Both hidden layers in strips from one launch of streams, fused and apart, then on other patterns: steps of either pipeline stay close, and replays of a graph give what eager steps give."""
    import torch
    sizes, batch = [400, 600, 520, 10], 200
    rng = np.random.default_rng(0)
    labels = torch.from_numpy(rng.integers(0, 10, batch).astype(np.int32)).cuda()
    X = nb.to_dense(rng.standard_normal((sizes[0], batch)).astype(np.float32))
    data = wl.make_mlp(sizes, sparsity=0.7)
    mlps = [nb.MLP(data, batch, f) for f in (nb.NERVA_MLP_DEFAULT, nb.NERVA_MLP_UNFUSED)]
    for density in (None, 0.2):
        if density:
            for l in (0, 1):
                new = strips_case(sizes[l + 1], sizes[l], lambda i: int(density * sizes[l]) + i % 9, l)
                for m in mlps:
                    L = m.layers[l]
                    L.indptr, L.indices, L.values = (torch.from_numpy(np.array(a)).cuda() for a in (new.indptr, new.indices, new.values))
                    L.velocity = torch.zeros_like(L.values)
                    nb.sparse_linear_rebind(L.handle, L.values.numel(), L.indptr, L.indices, L.values)
                    nb.mlp_rebind_velocity(m.handle, l, L.velocity)
        for _ in range(3):
            for m in mlps:
                m.train_step(X, labels, batch, 0.01, 0.9)
        torch.cuda.synchronize()
        assert np.isclose(mlps[0].loss.item(), mlps[1].loss.item(), rtol=1e-5)
        for a, b in zip(mlps[0].layers, mlps[1].layers):
            close(a.values.cpu().numpy(), b.values.cpu().numpy(), np.full(b.values.numel(), 10 * b.values.abs().max().item()), what="weights")
    m = mlps[0]
    m.forward(X, batch)
    torch.cuda.synchronize()
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        m.forward(X, batch)
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            out = m.forward(X, batch)
    for k in range(3):
        m.layers[0].values.mul_(1.1)
        want = m.forward(X, batch).clone()
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out[:, :batch], want[:, :batch]), k
    m.close(); mlps[1].close()


def hot_rows_layer(rows, cols, n_long, long_share, short, seed, relu=False):
    """`n_long` rows that store `long_share` of their columns among rows of `short` entries: the backward pass keeps dZ of the 512 longest in LDS.  Column 0 is only in rows of the
    latter kind, column 1 only in the long ones, column 2 in none."""
    rng = np.random.default_rng(seed)
    long_rows = set(rng.choice(rows, n_long, replace=False).tolist())
    per_row = []
    for i in range(rows):
        n = int(long_share * cols) if i in long_rows else short
        j = rng.choice(np.arange(3, cols), n, replace=False)
        if i in long_rows and i % 2 or i not in long_rows and i % 50 == 0:
            j[0] = 1 if i in long_rows else 0
        per_row.append(np.unique(j))
    indptr = np.concatenate([[0], np.cumsum([len(r) for r in per_row])]).astype(np.int32)
    indices = np.concatenate(per_row).astype(np.int32)
    values = (rng.standard_normal(len(indices)) * 0.1).astype(np.float32)
    return wl.SparseLayerData(rows, cols, indptr, indices, values, np.zeros(rows, dtype=np.float32), relu), sorted(long_rows)


@pytest.mark.parametrize("rows,cols,n_long,batch,ld,relu", [
    (1100, 2600, 400, 512, None, False),    # whole tiles; some of the 512 rows in LDS are short ones
    (1531, 2599, 500, 509, 509, False),     # ragged columns, rows in sets of four with one left over
    (1300, 2603, 600, 500, None, True),     # long rows outside LDS; a batch of a multiple of 4 that fills no tile
    (6200, 2501, 512, 576, 577, False),     # more rows of dZ than an L2 holds two tiles of: two rounds of work-groups
])
def test_both_gradients_with_hot_rows_in_lds(nb, oracle, rows, cols, n_long, batch, ld, relu):
    lay, _ = hot_rows_layer(rows, cols, n_long, 0.28 if rows < 6000 else 0.25, 20, rows + batch, relu)
    check_layer(nb, oracle, lay, batch, ld=ld)


@pytest.mark.parametrize("rows,cols,n_long,batch,relu", [(*case[:4], case[5]) for case in test_both_gradients_with_hot_rows_in_lds.pytestmark[0].args[1]])
def test_matrices_of_the_hot_rows_tests_take_them_from_lds(nb, rows, cols, n_long, batch, relu):
    assert routes(nb, hot_rows_layer(rows, cols, n_long, 0.28 if rows < 6000 else 0.25, 20, rows + batch, relu)[0], batch) & nb.NERVA_ROUTE_BACKWARD_HOT_ROWS


@pytest.mark.parametrize("rows,cols,density,batch,hot", [(1100, 2600, 0.1, 1000, True), (1201, 9001, 0.06, 319, True), (1500, 1500, 0.05, 1024, False), (1500, 8000, 0.05, 256, False)])
def test_both_gradients_of_even_rows_with_the_first_512_in_lds(nb, oracle, rows, cols, density, batch, hot):
    """Half of the gathers, or fewer, are from LDS: where the mirror's rows are long that still pays."""
    lay = layer_case(rows, cols, density, seed=rows + batch)
    assert bool(routes(nb, lay, batch) & nb.NERVA_ROUTE_BACKWARD_HOT_ROWS) == hot
    check_layer(nb, oracle, lay, batch)


def test_order_of_hot_rows_is_made_by_the_call_that_takes_it(nb, oracle):
    """Of a pattern bound to a layer that has not taken it: the first such call may be one that is recorded into a graph, which has not run when an eager one follows.  Then a new pattern, with
    which the order is made as it is bound, and one more without a call between."""
    import torch
    rows, cols, batch = 1100, 2600, 500
    lay = hot_rows_layer(rows, cols, 400, 0.28, 20, 11)[0]
    other = hot_rows_layer(rows, cols, 380, 0.29, 21, 12)[0]
    rng = np.random.default_rng(7)
    X = rng.standard_normal((cols, batch)).astype(np.float32); dY = rng.standard_normal((rows, batch)).astype(np.float32)
    Xd, dYd, dXd = nb.to_dense(X), nb.to_dense(dY), nb.dense(cols, batch)
    db = torch.empty(rows, device="cuda")

    def call(L, g):
        nb.sparse_linear_backward(L.handle, Xd, None, dYd, dXd, g, db, batch)

    def check(L, pattern, g, what):
        torch.cuda.synchronize()
        values = L.values.cpu().numpy()
        dX, S = oracle.spmm_t(rows, cols, pattern.indptr, pattern.indices, values, dY)
        close(dXd.cpu().numpy(), dX, S, what=f"dX, {what}")
        gr, Sg, dbr, Sdb = oracle.sddmm(rows, cols, pattern.indptr, pattern.indices, dY, X)
        close(g.cpu().numpy(), gr, Sg, what=f"g, {what}")
        close(db.cpu().numpy(), dbr, Sdb, what=f"db, {what}")

    warm, g = nb.SparseLinear(lay, max_batch=batch), torch.empty(lay.nnz, device="cuda")
    call(warm, g)   # (the kernels are loaded)
    torch.cuda.synchronize()
    warm.close()
    L = nb.SparseLinear(lay, max_batch=batch)
    assert nb.sparse_linear_routes(L.handle, batch) & nb.NERVA_ROUTE_BACKWARD_HOT_ROWS
    L.rebind(lay.indptr, lay.indices, lay.values)
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        call(L, g)
    for k in range(3):
        L.values.mul_(-1.1)
        dXd.fill_(float("nan")); g.fill_(float("nan"))
        if k == 1:
            call(L, g)
            check(L, lay, g, "eager")
            dXd.fill_(float("nan")); g.fill_(float("nan"))
        graph.replay()
        check(L, lay, g, f"replay {k}")
    del graph
    L.rebind(other.indptr, other.indices, other.values)
    g = torch.full((other.nnz,), float("nan"), device="cuda")
    dXd.fill_(float("nan"))
    call(L, g)
    check(L, other, g, "rebound")
    for pattern in (other, lay):
        L.rebind(pattern.indptr, pattern.indices, pattern.values)
    g = torch.full((lay.nnz,), float("nan"), device="cuda")
    dXd.fill_(float("nan"))
    call(L, g)
    check(L, lay, g, "rebound twice")
    L.close()


def test_hot_rows_in_lds_keep_infinities_to_the_rows_that_read_them(nb, oracle):
    """A row of dZ of infinities, one of those in LDS and one that is not: they reach the gradients of the inputs that reference them, and their own entries' and biases', and nothing else."""
    import torch
    rows, cols, batch = 1100, 2600, 500
    lay, long_rows = hot_rows_layer(rows, cols, 400, 0.28, 20, 11)
    short_rows = [i for i in range(rows) if i not in set(long_rows)]
    rng = np.random.default_rng(3)
    X = rng.standard_normal((cols, batch)).astype(np.float32); dY = rng.standard_normal((rows, batch)).astype(np.float32)
    bad = [long_rows[7], short_rows[-3]]
    dY[bad] = np.inf
    L = nb.SparseLinear(lay, max_batch=batch)
    dXd, g, db = nb.dense(cols, batch), torch.empty(lay.nnz, device="cuda"), torch.empty(rows, device="cuda")
    nb.sparse_linear_backward(L.handle, nb.to_dense(X), None, nb.to_dense(dY), dXd, g, db, batch)
    torch.cuda.synchronize()
    row_of = np.repeat(np.arange(rows), np.diff(lay.indptr))
    hit = np.zeros(cols, dtype=bool); hit[lay.indices[np.isin(row_of, bad)]] = True
    dX, gh = dXd.cpu().numpy(), g.cpu().numpy()
    assert np.isfinite(dX[~hit]).all() and not np.isfinite(dX[hit]).all(axis=1).any()
    own = np.isin(row_of, bad)
    assert np.isfinite(gh[~own]).all() and not np.isfinite(gh[own]).any()
    assert np.array_equal(np.isfinite(db.cpu().numpy()), ~np.isin(np.arange(rows), bad))
    dY[bad] = 0
    ref, S = oracle.spmm_t(rows, cols, lay.indptr, lay.indices, lay.values, dY)
    close(dX[~hit], ref[~hit], S[~hit], what="dX beside infinities")
    L.close()


@pytest.mark.parametrize("batch", [512, 449])
def test_training_step_with_hot_rows_in_lds(nb, oracle, batch):
    """The layer's update behind the same pass: every stage against the oracle, over steps whose weights each find changed."""
    import torch
    from test_gpu_mlp_step import snapshot, stage_parity
    sizes = (60, 2600, 1100, 10)
    mlp = wl.make_mlp(sizes, layer_nnz=(5200, 2600, 2000), pattern_seed=1, value_seed=2)
    mlp.layers[1] = hot_rows_layer(1100, 2600, 400, 0.28, 20, 5, relu=True)[0]
    Xs, Ts = wl.make_batches(sizes[0], sizes[-1], batch, 2, seed=3)
    M = nb.MLP(mlp, batch)
    for t in range(2):
        before = snapshot(M)
        M.train_step(nb.to_dense(Xs[t]), torch.as_tensor(Ts[t]).cuda(), batch, 0.05, 0.9)
        torch.cuda.synchronize()
        stage_parity(nb, torch, oracle, M, mlp, before, Xs[t], Ts[t], batch, 0.05, 0.9, False)
    M.close()


@pytest.mark.parametrize("batch", [512, 449])
def test_training_step_takes_hot_rows_from_lds(nb, batch):
    """The network of the test above."""
    import torch
    from test_gpu_mlp_step import _launch_names
    sizes = (60, 2600, 1100, 10)
    mlp = wl.make_mlp(sizes, layer_nnz=(5200, 2600, 2000), pattern_seed=1, value_seed=2)
    mlp.layers[1] = hot_rows_layer(1100, 2600, 400, 0.28, 20, 5, relu=True)[0]
    Xs, Ts = wl.make_batches(sizes[0], sizes[-1], batch, 1, seed=3)
    M = nb.MLP(mlp, batch)
    assert nb.sparse_linear_routes(M.layers[1].handle, batch) & nb.NERVA_ROUTE_BACKWARD_HOT_ROWS
    assert "backward_fused[1]" in _launch_names(nb, torch, M, Xs[0], Ts[0], batch)   # (whose kernels the route says)
    M.close()
