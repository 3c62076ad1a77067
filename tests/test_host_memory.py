"""Device memory that a layer owns, from the host's side: what it holds when a call of the runtime fails.  The library runs on
a HIP runtime without a GPU (fake_hip.cpp), each test in a process of its own, where any allocation can be made to fail."""
import ctypes
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2407_17437_amd", "libnerva_sparse.so")


class Library:
    """The library on the runtime at `fake`, and one layer whose pattern is whatever `counts` makes of it."""

    def __init__(self, fake):
        self.hip = ctypes.CDLL(fake, mode=ctypes.RTLD_GLOBAL)   # (before the library, which then binds to it)
        self.hip.fake_launched.restype = ctypes.c_char_p
        self.hip.fake_live_bytes.restype = ctypes.c_size_t
        self.hip.fake_fail_after.argtypes = [ctypes.c_long]
        self.hip.fake_fail_after_left.restype = ctypes.c_long
        self.lib = ctypes.CDLL(LIB)
        self.lib.nerva_last_error.restype = ctypes.c_char_p
        self.host = [(ctypes.c_float * (1 << 20))() for _ in range(4)]   # (never read: no kernel runs)
        self.layer = ctypes.c_void_p()

    def counts(self, side, **values):
        for name, value in values.items():
            assert self.hip.fake_set(side, name.encode(), value) == 0, name

    def create(self, rows, cols, nnz, max_batch, relu=False):
        self.rows, self.cols = rows, cols
        a = [ctypes.addressof(h) for h in self.host]
        return self.lib.sparse_linear_create(ctypes.byref(self.layer), rows, cols, nnz, ctypes.c_void_p(a[0]), ctypes.c_void_p(a[1]), ctypes.c_void_p(a[2]),
                                             None, 1 if relu else 0, max_batch, None)

    def rebind(self, nnz):
        a = [ctypes.addressof(h) for h in self.host]
        return self.lib.sparse_linear_rebind(self.layer, nnz, ctypes.c_void_p(a[0]), ctypes.c_void_p(a[1]), ctypes.c_void_p(a[2]), None)

    def destroy(self):
        self.lib.sparse_linear_destroy(self.layer)
        self.layer = ctypes.c_void_p()

    def forward(self, batch):
        p = ctypes.c_void_p(ctypes.addressof(self.host[3]))
        return self.lib.sparse_linear_forward(self.layer, p, batch, p, batch, batch, None)

    def backward(self, batch, dx=True, dvalues=True):
        p = ctypes.c_void_p(ctypes.addressof(self.host[3]))
        return self.lib.sparse_linear_backward(self.layer, p, batch, p, batch, p, batch, p if dx else None, batch, p if dvalues else None, p, batch, None)

    def routes(self, batch):
        out = ctypes.c_int32(-1)
        assert self.lib.sparse_linear_routes(self.layer, batch, ctypes.byref(out)) == 0
        return out.value

    def launched(self):
        return self.hip.fake_launched().decode().split()


def a_failed_call_is_reported_once(L):
    L.counts(0, n_blocks=8, longest_row=40)
    L.counts(1, n_blocks=8, longest_row=40)
    assert L.create(64, 512, 2000, 32) == 0
    L.hip.fake_fail_after(0)
    assert L.rebind(4000) == -5
    assert L.forward(32) == 0 and L.backward(32) == 0, L.lib.nerva_last_error()   # (their launches are in order)


def a_failed_rebind_leaves_nothing_freed_in_use(L):
    """Whichever of its allocations, fills and waits fails, the layer goes on with the old pattern (few rows cut into many
    work-groups, then many rows cut into few, and back)."""
    few, many = dict(n_blocks=60, n_huge_rows=2, n_huge_blocks=50, longest_row=400), dict(n_blocks=400, n_huge_rows=150, n_huge_blocks=300, longest_row=400)
    for old, new in ((few, many), (many, few)):
        for k in range(100):
            for side in (0, 1):
                L.counts(side, **old)
            assert L.create(256, 512, 2000, 128, relu=True) == 0
            for side in (0, 1):
                L.counts(side, **new)
            L.hip.fake_fail_after(k)
            rc = L.rebind(9000)
            L.hip.fake_fail_after(-1)
            for batch in (1, 100, 128):
                assert L.forward(batch) == 0 and L.backward(batch) == 0, L.lib.nerva_last_error()
            L.destroy()
            assert L.hip.fake_bad_pointers() == 0 and L.hip.fake_dirty_tickets() == 0, k
            if rc == 0:
                break
            assert rc == -5
        assert 3 < k < 99


def dense_rows_go_apart_by_the_batch_of_the_call(L):
    """500 dense rows of 1100 entries: the work that pays for their launch is there from 367 columns on, whatever the layer is bound for."""
    for max_batch in (367, 1024, 4096):
        L.counts(0, n_blocks=600, n_dense=500, dense_nnz=550000, longest_row=1100)
        L.counts(1, n_blocks=600, longest_row=2000)
        assert L.create(16384, 2048, 3700000, max_batch) == 0
        for batch in (128, 366, 367, max_batch):
            L.launched()
            assert L.forward(batch) == 0
            assert any("dense_rows_kernel" in k for k in L.launched()) == (batch >= 367), (max_batch, batch)
            assert L.backward(batch, dx=False) == 0
            assert any("sampled_update_kernel" in k for k in L.launched()) == (batch >= 367), (max_batch, batch)
        L.destroy()


def wide_products_of_dense_rows_take_the_bf16_units(L):
    """By the estimates of both; a narrow batch of the same layer, and few rows, stay on the fp32 ones."""
    for rows, cols, n, nnz, batch, split in ((2500, 1057, 1030, 653000, 1024, True), (5000, 1030, 5000, 1854000, 193, True), (1400, 2310, 1281, 1243000, 771, True),
                                            (4000, 1060, 4000, 1484000, 2000, True), (2500, 1057, 1030, 653000, 322, False), (3000, 16384, 205, 1680000, 1024, False)):
        for max_batch in (batch, 2048):
            L.counts(0, n_blocks=600, n_dense=n, dense_nnz=nnz, longest_row=2000)
            L.counts(1, n_blocks=600, longest_row=2000)
            assert L.create(rows, cols, nnz + 9000, max_batch) == 0
            L.launched()
            assert L.forward(batch) == 0
            launched = L.launched()
            assert any("split_dense_rows_kernel" in k for k in launched) == split, (rows, cols, batch, launched)
            assert any("dense_rows_kernel" in k for k in launched)
            L.destroy()


def a_ticket_of_a_shared_tile_counts_to_one_number(L):
    """1024 x 3072 on the dense route: tiles in four slices up to 64 columns of the batch, in two from there to 192.  The calls of both
    may overlap, and a ticket that both counted on, modulo 4 and modulo 2, would not be back at 0 after them."""
    L.counts(0, n_blocks=64, longest_row=1600)
    L.counts(1, n_blocks=64, longest_row=600)
    assert L.create(1024, 3072, 1600000, 200) == 0
    for batch in (64, 100, 33, 192, 200, 64):
        assert L.forward(batch) == 0
    assert any("dense_nn_kernel" in k for k in L.launched())
    assert L.hip.fake_bad_pointers() == 0 and L.hip.fake_dirty_tickets() == 0 and L.hip.fake_mixed_tickets() == 0
    L.destroy()


def a_thin_matrix_takes_the_bf16_units_where_they_pay(L):
    """A matrix of 17 to 30 %: by the estimates of gathering (staged where the batch fills its tiles) and of the split product, never on the
    fp32 units.  Bound for the batch, as those were measured; where the operand's parts have no room it is gathered."""
    def bound(rows, cols, density, max_batch):
        nnz = int(rows * cols * density)
        L.counts(0, n_blocks=600, longest_row=cols // 3)
        L.counts(1, n_blocks=600, longest_row=2000)
        return L.create(rows, cols, nnz, max_batch)

    def forward(batch):
        L.launched()
        assert L.forward(batch) == 0
        launched = L.launched()
        assert not any("dense_rows_kernelILi" in k for k in launched), launched
        return any("split_dense_rows_kernel" in k for k in launched)

    for rows, cols, density, max_batch, batch, split in (
            (9019, 2137, 0.26, 288, 288, False), (9019, 2137, 0.26, 768, 768, True), (873, 11642, 0.27, 270, 270, True), (8192, 4096, 0.2, 257, 257, False),
            (8192, 4096, 0.2, 512, 512, True), (8192, 4096, 0.2, 1024, 1024, True), (8192, 4096, 0.2, 1024, 520, True), (8192, 4096, 0.2, 520, 520, False), (2600, 16384, 0.2, 256, 256, True),
            (2600, 16384, 0.175, 320, 320, False), (3935, 8046, 0.2243, 384, 384, False), (2916, 2321, 0.2311, 500, 500, False), (1000, 8000, 0.175, 320, 320, True),
            (2050, 2100, 0.278, 600, 600, True), (2050, 2100, 0.278, 600, 300, False), (2050, 2100, 0.2, 470, 470, False), (600, 38138, 0.25, 10474, 10474, False), (600, 38138, 0.25, 10474, 1024, True)):
        L.launched()
        assert bound(rows, cols, density, max_batch) == 0
        names = L.launched()
        assert sum("11plan_kernel" in k for k in names) == 1 and sum("pattern_table_kernel" in k for k in names) == 1, names
        assert forward(batch) == split, (rows, cols, density, max_batch, batch)
        L.destroy()
    for k in range(100):
        L.hip.fake_fail_after(k)
        rc = bound(8192, 4096, 0.2, 512)
        failed = L.hip.fake_fail_after_left() < 0
        L.hip.fake_fail_after(-1)
        if rc == 0:
            for batch in (128, 300, 512):
                forward(batch)
            L.destroy()
            if not failed:
                break
    assert k < 99 and L.hip.fake_bad_pointers() == 0


def slices_of_dense_rows_stay_where_their_parts_have_no_room(L):
    """Whichever allocation fails: a wide product of dense rows that does not get the bf16 units still has its sum cut into slices."""
    seen = set()
    for k in range(100):
        L.counts(0, n_blocks=600, n_dense=1030, dense_nnz=653000, longest_row=800)
        L.counts(1, n_blocks=600, longest_row=2000)
        L.hip.fake_fail_after(k)
        rc = L.create(2500, 1057, 662000, 1024)
        failed = L.hip.fake_fail_after_left() < 0
        L.hip.fake_fail_after(-1)
        if rc == 0:
            L.launched()
            assert L.forward(1024) == 0
            launched = L.launched()
            if any("dense_rows" in name for name in launched):   # (else the row table is the one without room)
                assert any("dense_rows_finish_kernel" in name for name in launched), (k, launched)
                seen.add(any("split_dense_rows_kernel" in name for name in launched))
            L.destroy()
            if not failed:
                break
    assert seen == {True, False}


def a_layer_is_created_without_what_it_can_do_without(L):
    """Dense rows with sliced results, a staged plan for the batches below theirs, partial products, dZ of a ReLU layer: each of them
    fails once.  (The calls fail one after another; those whose failure the create survives are these.)"""
    survived = 0
    for k in range(100):
        L.counts(0, n_blocks=600, n_dense=500, dense_nnz=550000, longest_row=1100, staged_ranges=48, staged_rows=16000, staged_nnz=3000000)
        L.counts(1, n_blocks=600, longest_row=2000)
        L.hip.fake_fail_after(k)
        rc = L.create(16384, 2048, 3700000, 1024, relu=True)
        failed = L.hip.fake_fail_after_left() < 0
        L.hip.fake_fail_after(-1)
        if rc == 0:
            for batch in (1, 100, 128, 320, 700, 1024):
                assert L.forward(batch) == 0 and L.backward(batch) == 0 and L.backward(batch, dx=False) == 0, L.lib.nerva_last_error()
            L.destroy()
            if not failed:
                break
            survived += 1
        assert rc in (0, -5) and L.hip.fake_bad_pointers() == 0
        assert L.hip.fake_live_bytes() == 0, "a failed create, or a destroyed layer, holds memory"
    assert survived == 5


def a_single_tile_needs_no_partial_products(L):
    held = []
    for max_batch in (64, 100):
        L.counts(0, n_blocks=600, longest_row=400)
        L.counts(1, n_blocks=600, longest_row=150)
        assert L.create(1024, 3072, 315000, max_batch, relu=True) == 0
        held.append(L.hip.fake_live_bytes())
        L.launched()
        assert L.backward(max_batch) == 0
        assert any("backward_fused_kernel" in k for k in L.launched())
        L.destroy()
    assert held[1] - held[0] == 1024 * (128 - 64) * 4, held   # (dZ, whose rows are 128 and 64 columns apart)


def gathers_of_a_backward_tile_are_all_in_flight_where_its_waves_fit(L):
    for cols, entries, batch, apart in ((17000, 10200, 16, False), (17000, 10200, 32, False), (17000, 10200, 64, False), (17000, 700000, 128, False), (17000, 10200, 128, True),
                                        (17000, 10200, 256, True), (16000, 10200, 16, True), (16000, 10200, 32, True), (16000, 10200, 64, True), (6100, 10200, 128, True), (6200, 10200, 128, True),
                                        (6200, 310000, 128, False), (4600, 200000, 128, True), (25000, 10200, 64, True), (33000, 10200, 128, True)):
        L.counts(0, n_blocks=600, longest_row=300)
        L.counts(1, n_blocks=600, longest_row=10)
        assert L.create(60, cols, entries, 256) == 0
        L.launched()
        assert L.backward(batch) == 0
        names = [k for k in L.launched() if "backward_fused_kernel" in k]
        assert len(names) == 1 and ("BackwardPassE1" in names[0]) and ("SpareE%dELb%dEE" % (2 if batch == 16 else 0, apart) in names[0]), (cols, entries, batch, names)
        L.destroy()


def few_column_tiles_serve_where_they_pay(L):
    """Rows, columns, entries, longest row, batch; whether the forward product and the gradient alone run in column tiles (fewer than eight)."""
    for rows, cols, nnz, longest, batch, product, gradient in (
            (9106, 9383, 85441, 30, 400, True, False),       # even rows, an operand of 14 MiB gathered rarely
            (9106, 9383, 85441, 30, 256, False, False),      # the same at 9 MiB
            (9106, 9383, 256323, 60, 256, True, True),       # 27 entries an operand row
            (8192, 8192, 402653, 2000, 256, True, True),     # rows of very different lengths, 49 entries a row
            (8192, 8192, 402653, 2000, 128, False, False),
            (5000, 5000, 300000, 2000, 700, False, True),    # tiles of 2.4 MiB
            (12000, 3000, 108000, 2000, 850, False, False),  # nine entries a row
            (9106, 9383, 1024320, 4000, 768, True, True),
            (9106, 9383, 1024320, 4000, 850, False, True)):  # the seventh tile partly empty, a tile beyond an L2
        L.counts(0, n_blocks=600, longest_row=longest)
        L.counts(1, n_blocks=600, longest_row=60)
        assert L.create(rows, cols, nnz, batch) == 0
        L.launched()
        assert L.forward(batch) == 0
        assert any("spmm_tiled" in k or "spmm_packed" in k for k in L.launched()) == product, (rows, cols, nnz, batch)
        assert L.backward(batch, dx=False) == 0
        assert any("sddmm_tiled" in k for k in L.launched()) == gradient, (rows, cols, nnz, batch)
        L.destroy()


def short_segments_are_staged_by_the_work_of_the_plan(L):
    """Beside dense rows the plan covers a part of the matrix, and its entries, not the matrix's, are the work that shorter segments take; neither do
    they pay where copying the operand weighs more than serving them."""
    for rows, cols, nnz, n_dense, dense_nnz, plan, batch, product, gradient in (
            (5000, 5000, 2500000, 600, 1700000, (64, 4000, 726000), 256, True, False),       # segments of 18, 186 M of 640 M entries times columns
            (5000, 5000, 3600000, 600, 1700000, (64, 9000, 1730000), 256, True, True),       # of 19, 443 M
            (16384, 5000, 2500000, 600, 1700000, (64, 8000, 726000), 256, False, False),     # of 9, 186 M
            (16384, 5000, 3900000, 600, 1700000, (64, 15000, 1350000), 256, True, False),    # of 9, 346 M
            (7278, 12626, 1788000, 0, 0, (64, 7278, 1788000), 256, False, False),            # of 9.8, 458 M, 2.2 entries per copied row
            (7278, 12626, 1788000, 0, 0, (56, 7278, 1788000), 256, True, False)):            # 2.53
        L.counts(0, n_blocks=600, n_dense=n_dense, dense_nnz=dense_nnz, longest_row=300, staged_ranges=plan[0], staged_rows=plan[1], staged_nnz=plan[2])
        L.counts(1, n_blocks=600, longest_row=2000)
        assert L.create(rows, cols, nnz, batch) == 0
        L.launched()
        assert L.forward(batch) == 0
        launched = L.launched()
        assert any("dense_rows" in k for k in launched) == (n_dense > 0)
        assert any("spmm_staged_kernel" in k for k in launched) == product, (rows, cols, plan, launched)
        assert L.backward(batch, dx=False) == 0
        assert any("sddmm_staged_kernel" in k for k in L.launched()) == gradient, (rows, cols, plan)
        L.destroy()


def both_gradients_go_apart_where_that_is_faster(L):
    """rows, columns, entries, batch, ranges of W's plan and of its mirror's; dense rows, their entries, rows and entries of the plan beside them.  As measured,
    us, on one stream of gathers and apart (with the mirror's values ahead)."""
    for rows, cols, nnz, batch, ranges, dense, apart in (
            (9877, 13217, 11592349, 192, (85, 85), None, True),      # 636 / 545
            (7626, 7351, 5448993, 640, (25, 25), None, True),        # 647 / 598
            (13983, 2818, 4562994, 768, (21, 21), (2648, 3245624, 3477, 718494), True),    # 825 / 593
            (14473, 2876, 3000000, 1024, (48, 16), None, True),
            (1896, 8041, 5070586, 300, (29, 51), None, True),        # 360 / 225, the gradient by matrix instructions
            (2064, 1450, 459694, 640, (25, 22), None, False),        # 68 / 83, as well
            (3336, 14187, 4368363, 640, (25, 51), None, False),      # 483 / 546
            (6304, 10132, 5812395, 256, (64, 64), None, False),      # 306 / 334
            (11649, 4703, 2969360, 512, (32, 32), (925, 1891006, 2354, 606578), False),    # 310 / 346
            (9535, 4605, 5576402, 256, (64, 64), (2012, 4030623, 4998, 1277028), False),   # 284 / 324
            (11458, 1073, 944212, 1024, (32, 16), None, False),      # 198 / 222
            (1525, 1453, 334363, 900, (17, 17), None, False)):       # 69 / 89: 301 M entries times columns
        n_dense, dense_nnz, plan_rows, plan_nnz = dense or (0, 0, rows, nnz)
        L.counts(0, n_blocks=600, n_dense=n_dense, dense_nnz=dense_nnz, longest_row=cols // 3, staged_ranges=ranges[0], staged_rows=plan_rows, staged_nnz=plan_nnz)
        L.counts(1, n_blocks=600, longest_row=rows // 5, staged_ranges=ranges[1], staged_rows=cols, staged_nnz=nnz)
        assert L.create(rows, cols, nnz, batch) == 0
        L.launched()
        assert L.backward(batch) == 0
        names = L.launched()
        assert any("backward_fused_kernel" in k for k in names) != apart, (rows, cols, batch, names)
        gradient = "sampled_update_kernel" if nnz >= 0.15 * rows * cols else "sddmm_staged_kernel"
        assert (any("spmm_staged_kernel" in k for k in names) and any(gradient in k for k in names)) == apart, (rows, cols, batch, names)
        L.destroy()


def both_gradients_go_apart_where_that_beats_hot_rows_in_lds(L):
    """rows, columns, entries, batch, ranges of W's plan and of its mirror's; dense rows, their entries, rows and entries of the plan beside them; shares of the 1024 and of the 512 longest rows.  Power-law
    matrices as measured, us, apart and with hot rows in LDS (one stream from the L2s takes longer than either)."""
    for rows, cols, nnz, batch, ranges, dense, most, share, hot in (
            (12085, 6193, 9677122, 656, (23, 23), (2602, 7015440, 9483, 2661682), 0.51, 0.33, False),     # 951 / 1329
            (8782, 15534, 13505539, 768, (21, 42), (1384, 9356951, 7398, 4148588), 0.63, 0.47, False),    # 1449 / 1837
            (8164, 11068, 10400338, 666, (23, 46), (1533, 7386461, 6631, 3013877), 0.62, 0.46, False),    # 1066 / 1255
            (8119, 5813, 5177373, 450, (32, 32), (1443, 3648530, 6676, 1528843), 0.63, 0.47, False),      # 445 / 488
            (4089, 5120, 2018199, 856, (18, 18), (625, 1392036, 3464, 626163), 0.78, 0.65, True),         # 304 / 273
            (9349, 10144, 4580591, 1024, (32, 32), (651, 2874377, 8698, 1706214), 0.71, 0.58, True),      # 835 / 733
            (9341, 4974, 2169781, 967, (32, 16), (628, 1357123, 8713, 812658), 0.71, 0.59, True),         # 423 / 354
            (2128, 4636, 1253893, 901, (17, 17), (450, 906259, 1678, 347634), 0.88, 0.75, True)):         # 228 / 181
        n_dense, dense_nnz, plan_rows, plan_nnz = dense
        L.counts(0, n_blocks=600, n_dense=n_dense, dense_nnz=dense_nnz, longest_row=int(0.9 * cols), hot_nnz=int(most * nnz), hot_lds_nnz=int(share * nnz),
                 staged_ranges=ranges[0], staged_rows=plan_rows, staged_nnz=plan_nnz)
        L.counts(1, n_blocks=600, longest_row=2 * nnz // cols, hot_nnz=nnz // 8, staged_ranges=ranges[1], staged_rows=cols, staged_nnz=nnz)
        assert L.create(rows, cols, nnz, batch) == 0
        L.launched()
        assert L.backward(batch) == 0
        names = L.launched()
        assert any("backward_hot_kernel" in k for k in names) == hot and any("spmm_staged_kernel" in k for k in names) != hot, (rows, cols, batch, names)
        L.destroy()


def an_order_of_hot_rows_is_made_when_a_call_takes_it(L):
    """As a layer is created, and for a new pattern by the first that does or where one has; not where the layer's wide batches go by its dense copy, nor where at every batch the hot rows would be slower than both gradients apart."""
    for rows, cols, nnz, max_batch, dense, ranges, most, share, made in (
            (2000, 4000, 4000000, 1024, None, 0, 0.52, 0.26, False),         # half of its entries stored: the dense route
            (2000, 4000, 1000000, 1024, None, 0, 0.52, 0.26, True),
            (12085, 6193, 9677122, 512, (2602, 7015440, 9483, 2661682), 32, 0.51, 0.33, False),
            (9341, 4974, 2169781, 1024, (628, 1357123, 8713, 812658), 24, 0.71, 0.59, True)):
        n_dense, dense_nnz, plan_rows, plan_nnz = dense or (0, 0, 0, 0)
        L.counts(0, n_blocks=600, n_dense=n_dense, dense_nnz=dense_nnz, longest_row=int(0.9 * cols), hot_nnz=int(most * nnz), hot_lds_nnz=int(share * nnz),
                 staged_ranges=ranges, staged_rows=plan_rows, staged_nnz=plan_nnz)
        L.counts(1, n_blocks=600, longest_row=2 * nnz // cols, hot_nnz=nnz // 8, staged_ranges=ranges, staged_rows=cols if ranges else 0, staged_nnz=nnz if ranges else 0)
        L.launched()
        before = L.hip.fake_live_bytes()
        assert L.create(rows, cols, nnz, max_batch) == 0
        took = [batch for batch in range(1, max_batch + 1) if L.routes(batch) & 2]
        assert bool(took) == made, (rows, cols, nnz)
        assert any("hot_order_kernel" in k for k in L.launched()) == made, (rows, cols, nnz)

        def ordered():
            return sum("hot_order_kernel" in k for k in L.launched())

        # for a new pattern by the first call that takes it, where none has: nothing else of the layer pays for it
        assert L.forward(max_batch) == 0 and L.backward(max_batch, dx=False) == 0 and L.backward(64) == 0 and L.rebind(nnz) == 0
        assert ordered() == 0
        if made:
            # (a call that is recorded into a graph has not run)
            L.hip.fake_set_capturing(1)
            assert L.backward(took[-1]) == 0 and L.backward(took[0]) == 0 and ordered() == 2
            L.hip.fake_set_capturing(0)
            waits = L.hip.fake_waits()
            L.hip.fake_set_pending(1)
            assert L.backward(took[-1]) == 0 and ordered() == 1
            # (while it has not come through, calls that may be on other streams wait for it, recorded ones make their own)
            assert L.backward(took[-1]) == 0 and L.backward(took[0]) == 0 and ordered() == 0 and L.hip.fake_waits() == waits + 2
            L.hip.fake_set_capturing(1)
            assert L.backward(took[-1]) == 0 and ordered() == 1
            L.hip.fake_set_capturing(0)
            L.hip.fake_set_pending(0)
            assert L.backward(took[-1]) == 0 and L.backward(took[0]) == 0 and ordered() == 0 and L.hip.fake_waits() == waits + 2
            # a layer that has taken it has it made as a pattern is bound
            for _ in range(2):
                assert L.rebind(nnz) == 0 and ordered() == 1
                assert L.backward(took[-1]) == 0 and ordered() == 0
            assert L.rebind(nnz) == 0 and ordered() == 1 and L.rebind(nnz) == 0 and ordered() == 0
            assert L.backward(took[0]) == 0 and ordered() == 1
        L.destroy()
        assert L.hip.fake_live_bytes() == before and L.hip.fake_events() == 0 and L.hip.fake_bad_pointers() == 0


def a_failed_rebind_leaves_strips_and_hot_rows_in_place(L):
    """As above, of patterns whose forward product runs in strips, or whose gradients keep hot rows in LDS, and which grow or shrink."""
    def strips(nnz):
        L.counts(0, n_blocks=600, longest_row=2 * nnz // 8192, hot_nnz=nnz // 8, hot_lds_nnz=nnz // 16, n_short=8192)
        L.counts(1, n_blocks=600, longest_row=2 * nnz // 3072, hot_nnz=nnz // 3)
        L.hip.fake_set_strips(int(nnz / 16 / 8 / 0.9) + 600, int(nnz / 16 / 0.9))

    def hot(nnz):
        L.counts(0, n_blocks=600, longest_row=3000, hot_nnz=int(0.76 * nnz), hot_lds_nnz=int(0.67 * nnz))
        L.counts(1, n_blocks=600, longest_row=600, hot_nnz=nnz // 8)
        L.hip.fake_set_strips(0, 0)

    for rows, cols, counts, old, new, route in ((8192, 3072, strips, 342893, 500000, 1), (8192, 3072, strips, 500000, 342893, 1), (16384, 16384, hot, 2000000, 2684354, 2), (16384, 16384, hot, 2684354, 2000000, 2)):
        for k in range(100):
            counts(old)
            assert L.create(rows, cols, old, 1024, relu=True) == 0
            assert L.routes(1024) & route == route
            counts(new)
            L.hip.fake_fail_after(k)
            rc = L.rebind(new)
            L.hip.fake_fail_after(-1)
            L.launched()
            assert L.forward(1024) == 0 and L.backward(1024) == 0, L.lib.nerva_last_error()
            assert L.hip.fake_bad_pointers() == 0, k
            names = L.launched()
            if rc != 0:   # (else it may have gone on without what there was no room for)
                assert any(("spmm_strip_kernel", "backward_hot_kernel")[route - 1] in n for n in names), (k, names)
            L.destroy()
            assert rc in (0, -5)
            if rc == 0 and k > 30:
                break
        assert 3 < k < 99


def hot_rows_are_done_without_where_something_for_them_fails(L):
    """Whichever of a layer's allocations fails: it is not created, or its calls are in order, and their first launches report nothing that went before."""
    L.counts(0, n_blocks=600, longest_row=3000, hot_nnz=int(0.76 * 2684354), hot_lds_nnz=int(0.67 * 2684354))
    L.counts(1, n_blocks=600, longest_row=600, hot_nnz=300000)
    took = set()
    for k in range(60):
        L.hip.fake_fail_after(k)
        rc = L.create(16384, 16384, 2684354, 1024)
        left = L.hip.fake_fail_after_left()
        L.hip.fake_fail_after(-1)
        assert rc in (0, -5), k
        if rc == 0:
            took.add(L.routes(1024) & 2)
            assert L.backward(1024) == 0 and L.forward(1024) == 0, (k, L.lib.nerva_last_error())
            L.destroy()
        assert L.hip.fake_events() == 0 and L.hip.fake_bad_pointers() == 0, k
        if left >= 0:
            break
    assert took == {0, 2} and 3 < k < 59


def a_grid_has_no_more_work_groups_than_a_launch_can(L):
    """The gradient in column tiles comes in quarters of the partition's work-groups: where these are too many for a grid, the rows go through all columns at once."""
    for n_blocks, tiled in ((30_000_000, True), (60_000_000, False)):
        L.counts(0, n_blocks=n_blocks, longest_row=2000)
        L.counts(1, n_blocks=600, longest_row=60)
        assert L.create(5000, 5000, 300000, 700) == 0
        L.launched()
        assert L.backward(700, dx=False) == 0
        assert any("sddmm_tiled" in k for k in L.launched()) == tiled
        assert L.hip.fake_bad_grids() == 0, n_blocks
        L.destroy()


def products_of_very_many_entries_are_staged(L):
    """On either side of 2^30 entries, whose byte offsets do not fit in 32 bits."""
    for nnz, many in (((1 << 30) - 4, "0"), (1 << 30, "1")):
        L.counts(0, n_blocks=600, longest_row=17000, staged_ranges=147, staged_rows=65536, staged_nnz=nnz)
        L.counts(1, n_blocks=600, longest_row=10000, staged_ranges=293, staged_rows=131072, staged_nnz=nnz)
        assert L.create(65536, 131072, nnz, 128) == 0
        L.launched()
        assert L.forward(128) == 0 and L.backward(128, dvalues=False) == 0
        names = [k for k in L.launched() if "spmm_staged_kernel" in k]
        assert len(names) == 2 and all(f"ELb{many}E" in k for k in names), names
        L.destroy()


def the_first_layers_gradient_takes_a_second_pass_of_other_partial_products_only(L):
    """Layer 1's second pass rides in the launch of layer 0's column-tiled gradient, which writes partial products of its own: not where an MLP holds one handle twice.  Nor where it strews more over more
    rows than the L2s keep beside the gathers: as measured, us, apart and in one launch."""
    def layer(rows, cols, nnz, relu, batch):
        L.counts(0, n_blocks=600, longest_row=90, hot_nnz=nnz // 2 - 9)
        L.counts(1, n_blocks=600, longest_row=90, hot_nnz=nnz // 2 - 9)
        assert L.create(rows, cols, nnz, batch, relu=relu) == 0
        handle, L.layer = L.layer, ctypes.c_void_p()
        return handle

    p = ctypes.addressof(L.host[3])
    L.lib.mlp_workspace_bytes.restype = ctypes.c_size_t
    for cols, first, second, twice, batch, together in (
            (2600, (2600, 94640), (2600, 94640), False, 700, True), (2600, (2600, 94640), (2600, 94640), True, 700, False),
            (3072, (8192, 342893), (8192, 498753), False, 1024, True),       # 322 / 318
            (1879, (1879, 62000), (8144, 459000), False, 1024, False),       # 230 / 241
            (5871, (5373, 900000), (4349, 660000), False, 492, False),       # 274 / 288
            (2000, (5000, 200000), (4097, 99000), False, 1000, True), (2000, (5000, 200000), (4097, 310000), False, 1000, False), (2000, (5000, 200000), (4096, 310000), False, 1000, True)):
        below = layer(first[0], cols, first[1], True, batch)
        above = below if twice else layer(second[0], first[0], second[1], True, batch)
        handles, mlp, three = (below, above, layer(40, second[0], 1456, False, batch)), ctypes.c_void_p(), ctypes.c_void_p * 3
        assert L.lib.mlp_create(ctypes.byref(mlp), 3, three(*handles), three(p, p, p), three(p, p, p), batch, 0) == 0
        room = L.lib.mlp_workspace_bytes(mlp, batch)
        held = (ctypes.c_char * (room + 256))()
        work = ctypes.c_void_p(ctypes.addressof(held) + -ctypes.addressof(held) % 256)
        L.launched()
        assert L.lib.mlp_train_step(mlp, ctypes.c_void_p(p), batch, ctypes.c_void_p(p), batch, ctypes.c_float(0.1), ctypes.c_float(0.9), work, ctypes.c_size_t(room), None, None) == 0, L.lib.nerva_last_error()
        names = L.launched()
        assert any("sddmm_tiled_finish_kernel" in k for k in names) == together and any("backward_finish_kernel" in k for k in names) != together, (first, second, names)
        assert sum("sddmm_tiled" in k for k in names) == 1 and sum("backward_fused_kernel" in k for k in names) == 1, names
        L.lib.mlp_destroy(mlp)
        for handle in {h.value: h for h in handles}.values():
            L.lib.sparse_linear_destroy(handle)


def hot_rows_are_kept_in_lds_where_that_is_faster(L):
    """rows, columns, entries of a mirror row, batch, shares of the 1024 longest rows and of the 512 that fit in LDS; as measured, us, from the L2s and from LDS."""
    for rows, cols, entries, batch, most, share, hot in (
            (16384, 16384, 164, 1024, 0.76, 0.67, True),    # 541 / 446
            (16384, 16384, 164, 256, 0.76, 0.67, True),     # 146 / 133
            (4000, 8000, 160, 256, 0.84, 0.75, True),       # 77.7 / 65.5
            (5197, 6386, 62, 632, 0.87, 0.80, True),        # 57.3 / 52.2
            (1100, 2600, 110, 1024, 0.96, 0.49, True),      # even rows: 62.5 / 53.1
            (1200, 16384, 72, 320, 0.87, 0.44, True),       # 91.8 / 75.3
            (1500, 1500, 75, 1024, 0.71, 0.38, False),      # 32.4 / 34.8
            (1500, 8000, 75, 256, 0.71, 0.36, False),       # 37.6 / 44.5: one tile, no second pass
            (3000, 6000, 90, 256, 0.89, 0.81, False),       # power-law rows: 33.7 / 40.5
            (2000, 8000, 60, 256, 0.93, 0.86, False),       # 31.5 / 35.3
            (2000, 8000, 60, 384, 0.93, 0.86, True),        # 44.2 / 43.0
            (8192, 8192, 164, 1024, 0.13, 0.07, False)):    # 270 / 284
        nnz = cols * entries
        L.counts(0, n_blocks=600, longest_row=3000, hot_nnz=int(most * nnz), hot_lds_nnz=int(share * nnz))
        L.counts(1, n_blocks=600, longest_row=2 * entries, hot_nnz=nnz // 8, hot_lds_nnz=nnz // 16)
        for max_batch in (batch, 1024):
            assert L.create(rows, cols, nnz, max_batch) == 0
            L.launched()
            assert L.backward(batch) == 0
            names = L.launched()
            assert any("backward_hot_kernel" in k for k in names) == hot and any("backward_fused_kernel" in k for k in names) != hot, (rows, cols, batch, names)
            assert L.routes(batch) & 2 == 2 * hot
            L.destroy()


def strips_are_planned_where_a_batch_takes_them(L):
    """rows, columns, entries, share of the steps that carry an entry; widest batch; batches, and whether they take strips (None: no plan is made).  As measured, us, by the other kernel and in strips."""
    for rows, cols, nnz, full, max_batch, batches in (
            (8192, 3072, 342893, 0.97, 300, None),                                  # 20 / 25: nor any narrower one
            (8192, 8192, 498753, 0.82, 300, None),
            (8192, 3072, 342893, 0.97, 1024, ((208, False), (1024, True))),         # 59 / 41
            (8192, 8192, 498753, 0.82, 1024, ((208, False), (1024, True))),         # 93 / 58
            (3101, 2026, 381630, 0.99, 329, ((329, False),)),                       # 24.9 / 31.4: staged, the best such a plan can come to would pay
            (2622, 4783, 128466, 0.93, 1020, None),                                 # 23.8 / 29.3
            (16384, 16384, 2684355, 0.77, 1024, ((1024, True),)),                   # 456 / 245
            (8192, 8192, 498753, 0.3, 1024, ((1024, False),))):                     # segments of many lengths: no room is held for a stream
        blocks = (cols + 2047) // 2048
        steps = int(nnz / 16 / full)
        L.counts(0, n_blocks=600, longest_row=int(1.6 * nnz / rows), hot_nnz=nnz // 8, n_short=rows if nnz < 100 * rows else 0)
        L.counts(1, n_blocks=600, longest_row=int(1.6 * nnz / cols), hot_nnz=nnz * 1024 // cols)
        ranges = {16384: 48, 3101: 42}.get(rows, 0)
        L.counts(0, staged_ranges=ranges, staged_rows=rows * (ranges > 0), staged_nnz=nnz * (ranges > 0))
        L.hip.fake_set_strips(int(steps / 8 + rows / 16 * blocks / 2), steps)
        assert L.create(rows, cols, nnz, max_batch) == 0
        assert (L.hip.fake_strip_blocks() > 0) == (batches is not None), (rows, cols, max_batch)
        for batch, strips in batches or ((max_batch, False),):
            L.launched()
            assert L.forward(batch) == 0
            names = L.launched()
            assert any("spmm_strip_kernel" in k for k in names) == any("strip_stream_kernel" in k for k in names) == strips, (rows, cols, batch, names)
            assert L.routes(batch) & 1 == strips
        L.destroy()


CASES = [hot_rows_are_done_without_where_something_for_them_fails, a_failed_rebind_leaves_strips_and_hot_rows_in_place, an_order_of_hot_rows_is_made_when_a_call_takes_it, both_gradients_go_apart_where_that_beats_hot_rows_in_lds, strips_are_planned_where_a_batch_takes_them, hot_rows_are_kept_in_lds_where_that_is_faster, the_first_layers_gradient_takes_a_second_pass_of_other_partial_products_only, products_of_very_many_entries_are_staged, a_grid_has_no_more_work_groups_than_a_launch_can, both_gradients_go_apart_where_that_is_faster, short_segments_are_staged_by_the_work_of_the_plan, few_column_tiles_serve_where_they_pay, gathers_of_a_backward_tile_are_all_in_flight_where_its_waves_fit, a_thin_matrix_takes_the_bf16_units_where_they_pay, slices_of_dense_rows_stay_where_their_parts_have_no_room, a_ticket_of_a_shared_tile_counts_to_one_number, wide_products_of_dense_rows_take_the_bf16_units, a_layer_is_created_without_what_it_can_do_without, a_single_tile_needs_no_partial_products, a_failed_call_is_reported_once, a_failed_rebind_leaves_nothing_freed_in_use, dense_rows_go_apart_by_the_batch_of_the_call]


@pytest.fixture(scope="module")
def fake_hip(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("hip") / "fake_hip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__=1", "-isystem", "/opt/rocm/include",
                    os.path.join(HERE, "fake_hip.cpp"), "-o", out], check=True)
    return out


@pytest.mark.parametrize("case", [c.__name__ for c in CASES])
def test_host_memory(fake_hip, case):
    run = subprocess.run([sys.executable, os.path.abspath(__file__), fake_hip, case], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout + run.stderr


if __name__ == "__main__":
    globals()[sys.argv[2]](Library(sys.argv[1]))
