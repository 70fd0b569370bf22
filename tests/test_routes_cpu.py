"""Which kernels a public call launches, and what device memory it takes, without a GPU: the library's objects linked with
a HIP runtime that records (tests/route_recorder.cpp)."""
import ctypes as C
import os

import numpy as np
import pytest

from paper_2505_11076_amd import binding as B
from paper_2505_11076_amd import build as _build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


class Recorder:
    """The recording library; layers and stacks are plain handles."""

    def __init__(self):
        self.lib = C.CDLL(_build.build_route_recorder(os.path.join(ROOT, "tests", "route_recorder.cpp")))
        for name in ("rec_take", "rec_last_block", "rec_held", "rec_memset_bytes", "dbf_gemm_workspace_bytes", "dbf_tiled_bytes"):
            getattr(self.lib, name).restype = C.c_size_t
        self.lib.dbf_gemm.argtypes = [C.c_void_p, C.c_void_p, C.c_void_p, C.c_int, C.c_void_p, C.c_size_t, C.c_void_p]
        self.lib.rec_take.argtypes = [C.c_void_p, C.c_size_t]
        self.lib.dbf_free.restype = self.lib.dbf_stack_free.restype = self.lib.dbf_tuning_reset.restype = None

    def launches(self):
        """[(kernel, grid, threads, dynamic LDS bytes)] since the last call."""
        self.full_names = []
        buf = C.create_string_buffer(self.lib.rec_take(None, 0) + 1)
        self.lib.rec_take(buf, len(buf))
        out = []
        for line in buf.value.decode().splitlines():
            name, gx, gy, gz, threads, lds = line.split()
            name = name[name.index("dbf_"):]
            self.full_names.append(name)
            out.append((name[:name.index("_kernel")], (int(gx), int(gy), int(gz)), int(threads), int(lds)))
        return out

    def layer(self, n_in, n_out, k):
        """A layer with all signs -1 and zero scales: only its shape matters here."""
        A = np.zeros((n_out, (k + 31) // 32), np.uint32)
        Bw = np.zeros((k, (n_in + 31) // 32), np.uint32)
        v = [np.zeros(n, np.uint16) for n in (n_out, k, n_in)]
        h = C.c_void_p()
        assert self.lib.dbf_pack_bits(n_in, n_out, k, *[C.c_void_p(a.ctypes.data) for a in (A, Bw, *v)], C.byref(h)) == 0
        return h

    def stack(self, layers):
        h = C.c_void_p()
        assert self.lib.dbf_stack_create((C.c_void_p * len(layers))(*[l.value for l in layers]), len(layers), C.byref(h)) == 0
        return h

    def gemv(self, layer, batch, offset=0, kind=B.GEMV_AUTO):
        self.launches()
        assert self.lib.dbf_gemv_kind(layer, C.c_void_p(4096 + offset), C.c_void_p(1 << 20), batch, kind, None) == 0
        return self.launches()

    def gemm(self, layer, T, offset=0):
        self.launches()
        n = self.lib.dbf_gemm_workspace_bytes(layer, T)
        assert self.lib.dbf_gemm(layer, C.c_void_p(4096 + offset), C.c_void_p(1 << 20), T, C.c_void_p(1 << 21), C.c_size_t(n), None) == 0
        return self.launches()

    def stack_gemv(self, stack, batch, kind=B.GEMV_AUTO):
        self.launches()
        assert self.lib.dbf_stack_gemv(stack, C.c_void_p(4096), C.c_void_p(1 << 20), batch, kind, None) == 0
        return self.launches()


@pytest.fixture(scope="module")
def rec():
    r = Recorder()
    yield r
    r.lib.dbf_tuning_reset()


def _names(launches):
    return [l[0] for l in launches]


FEW = {"dbf_few", "dbf_small_layer"}


@pytest.mark.parametrize("when,knob,value", [
    ("plan", B.TUNE_COL_PIECES, 0), ("plan", B.TUNE_COL_PIECES, 3), ("plan", B.TUNE_PIECE_TARGET, 4096), ("plan", B.TUNE_PIECE_MIN_TILES, 2),
    ("plan", B.TUNE_PIECE_NEVER_TILES, 0), ("plan", B.TUNE_PIECE_MAX_ROW_TILES, 16), ("plan", B.TUNE_STACK_SPAN_B, 3), ("plan", B.TUNE_STACK_SPAN_A, 2),
    ("plan", B.TUNE_LONG_ROWS, 0),
    ("launch", B.TUNE_SHARED_Q, 2), ("launch", B.TUNE_SHARED_MIN_BATCH, 1), ("launch", B.TUNE_SHARED_MIN_BATCH, 17), ("launch", B.TUNE_SHARED_LDS_KB, 40),
    ("launch", B.TUNE_FUSED_MIN_B_ITEMS, 0), ("launch", B.TUNE_WIDE_WG_MAX_ITEMS, 0), ("launch", B.TUNE_FP4_MAX_ITEMS, 0)])
def test_a_decode_knob_off_its_default_takes_the_forms_that_the_knobs_steer(rec, when, knob, value):
    """Every knob of the decode cuts and forms is one of the item lists' (dbf.h): where one of them is set, a default call of
    few workgroups -- a layer alone, a group, at any batch -- goes through those lists, and PLAN knobs stay with the plan that
    was built under them."""
    shapes = [(6000, 300, 520), (520, 700, 6000), (300, 200, 100)]
    lib = rec.lib
    lib.dbf_tuning_reset()
    before = [rec.layer(*s) for s in shapes]
    assert lib.dbf_tuning_set(knob, value) == 0
    layers = [rec.layer(*s) for s in shapes]
    stack = rec.stack(layers)
    if when == "plan":
        lib.dbf_tuning_reset()
    try:
        for batch in (1, 2, 7, 16):
            for call, h in [(rec.gemv, l) for l in layers] + [(rec.stack_gemv, stack)]:
                assert not FEW & set(_names(call(h, batch))), (batch, _names(call(h, batch)))
        lib.dbf_tuning_reset()
        for l in before:                       # (plans built at the defaults are not affected)
            assert set(_names(rec.gemv(l, 1))) <= FEW
        if when == "launch":
            for l in layers:
                assert set(_names(rec.gemv(l, 1))) <= FEW
    finally:
        lib.dbf_tuning_reset()
        lib.dbf_stack_free(stack)
        for l in layers + before:
            lib.dbf_free(l)


def test_knobs_steer_what_the_header_says(rec):
    """Of the forms behind the knobs: no column piece with COL_PIECES = 0 (one workgroup per row tile), N pieces with N, once-per-call
    quantisation from SHARED_MIN_BATCH on, eight wavefronts and the fp4 form by their item limits."""
    lib = rec.lib
    lib.dbf_tuning_reset()

    def routes(plan, launch, batch, shape=(6000, 300, 520)):
        for knob, value in plan + launch:
            assert lib.dbf_tuning_set(knob, value) == 0
        l = rec.layer(*shape)
        try:
            return rec.gemv(l, batch)
        finally:
            lib.dbf_tuning_reset()
            lib.dbf_free(l)

    k_tiles, out_tiles = 5, 3          # row tiles of the two stages
    assert [l[1][0] for l in routes([(B.TUNE_COL_PIECES, 0)], [], 1)] == [k_tiles, out_tiles]
    assert [l[1][0] for l in routes([(B.TUNE_COL_PIECES, 3)], [], 1)] == [3 * k_tiles, out_tiles]   # (8 tiles a piece: the short rows stay whole)
    assert _names(routes([(B.TUNE_COL_PIECES, 0)], [(B.TUNE_SHARED_MIN_BATCH, 1)], 1)) == ["dbf_quantise_inputs", "dbf_items_mfma"] * 2
    assert _names(routes([(B.TUNE_COL_PIECES, 0)], [(B.TUNE_SHARED_MIN_BATCH, 17)], 16)) == ["dbf_items_mfma"] * 2
    square = (4096, 4096, 2048)
    threads = lambda **kw: [l[2] for l in routes([], [(getattr(B, n), v) for n, v in kw.items()], 1, square)]   # noqa: E731
    assert threads(TUNE_FP4_MAX_ITEMS=0) == [512, 512] and threads(TUNE_FP4_MAX_ITEMS=0, TUNE_WIDE_WG_MAX_ITEMS=0) == [256, 256]
    lds = lambda **kw: [l[3] for l in routes([], [(getattr(B, n), v) for n, v in kw.items()], 1, square)]       # noqa: E731
    assert lds(TUNE_WIDE_WG_MAX_ITEMS=1) != lds(TUNE_WIDE_WG_MAX_ITEMS=1, TUNE_FP4_MAX_ITEMS=0)                 # (its operand rows are the larger)


@pytest.mark.parametrize("shape,T,offset,quantiser", [
    ((4096, 4096, 3072), 2048, 0, "rows_held"), ((11008, 4096, 4477), 2048, 0, "rows_held"), ((16384, 128, 300), 1500, 0, "rows_block"),
    ((16384, 128, 300), 1536, 0, "rows_twice"), ((28672, 128, 300), 1279, 0, "rows_block"),
    ((28672, 128, 300), 4096, 0, "rows_twice"), ((4095, 4097, 3071), 4096, 0, "rows_twice"),
    ((4096, 4096, 3072), 2048, 2, "rows_twice"), ((11007, 4096, 4477), 1500, 0, "rows_twice"), ((11007, 4096, 4477), 384, 0, "rows_twice"),
    ((11007, 4096, 4477), 200, 0, "rows_block"), ((1001, 2000, 700), 4096, 0, "rows")])
def test_long_and_ragged_rows_of_many_tokens_are_not_written_in_pieces_of_cache_lines(rec, shape, T, offset, quantiser):
    """A prompt's rows go to the quantiser whose stores fit the operand layout: with a workgroup per token a cache line of it is
    written in eight pieces, which took up to 2.4 times as long (178 us against 73 for 4096 tokens of 16384 columns)."""
    l = rec.layer(*shape)
    try:
        assert _names(rec.gemm(l, T, offset))[0] == "dbf_quantise_" + quantiser
    finally:
        rec.lib.dbf_free(l)


def _layer_bytes(n_in, n_out, k):
    """Signs, vectors and scratch of a layer, each section a multiple of 256 bytes: what its calls read and write."""
    up = lambda v, a: (v + a - 1) // a * a   # noqa: E731
    rows = lambda v: up(v, 128)              # noqa: E731
    cols = lambda v: up(v, 64)               # noqa: E731
    parts = [rows(n_out) * cols(k) // 8, rows(k) * cols(n_in) // 8, 2 * rows(n_out), 2 * rows(k), 2 * cols(n_in),
             4 * 16 * rows(k), 128 + 32 * cols(n_in), 128 + 32 * cols(k)]
    return sum(up(v, 256) for v in parts)


def _tables_bound(n_in, n_out, k):
    # counters, and per row tile the records of the item lists and two rows of sums of their column pieces
    return 8192 + 3072 * ((n_out + 127) // 128 + (k + 127) // 128)


@pytest.mark.parametrize("shape", [(64, 64, 32), (512, 512, 256), (4096, 4096, 2048), (4096, 11008, 4477), (5056, 4096, 3000), (4096, 28672, 2730)])
def test_layers_and_stacks_whose_rows_are_never_cut_hold_no_sums_of_column_pieces(rec, shape):
    """Sums of column pieces take 8.1 KiB per row tile (260 KiB beside the 2 MiB of a 4096 x 4096 layer of k = 2048): only a plan with
    a stage that a call can cut -- 80 column tiles and more, 128 row tiles at most -- holds and clears them."""
    rec.lib.dbf_tuning_reset()
    cleared = rec.lib.rec_memset_bytes()
    layers = [rec.layer(*shape) for _ in range(2)]
    held, cleared = rec.lib.rec_last_block(), rec.lib.rec_memset_bytes() - cleared
    stack = rec.stack(layers)
    in_stack = rec.lib.rec_last_block()
    try:
        assert held <= _layer_bytes(*shape) + _tables_bound(*shape)
        assert cleared <= 2 * (held - rec.lib.dbf_tiled_bytes(shape[1], shape[2]) - rec.lib.dbf_tiled_bytes(shape[2], shape[0]))
        assert in_stack <= 2 * _tables_bound(*shape)
        for batch in (1, 2, 16):
            assert all(l[1][2] == 1 for l in rec.gemv(layers[0], batch) + rec.stack_gemv(stack, batch) if l[0] == "dbf_few")
    finally:
        rec.lib.dbf_stack_free(stack)
        for l in layers:
            rec.lib.dbf_free(l)


@pytest.mark.parametrize("shape,cut", [((11008, 4096, 4477), (True, False)), ((28672, 8192, 12743), (True, True)), ((5120, 300, 100), (True, False)),
                                       ((100, 300, 5120), (False, True))])
def test_layers_whose_rows_can_be_cut_hold_the_sums(rec, shape, cut):
    l = rec.layer(*shape)
    try:
        tiles = max(((v + 127) // 128) for v, c in zip((shape[2], shape[1]), cut) if c)
        assert rec.lib.rec_last_block() >= _layer_bytes(*shape) + 8320 * tiles
        assert tuple(x[1][2] > 1 for x in rec.gemv(l, 1)) == cut
    finally:
        rec.lib.dbf_free(l)


@pytest.mark.parametrize("shape,kept", [((64, 64, 32), 1), ((512, 300, 256), 200), ((4096, 4096, 2048), 1536), ((100, 300, 5120), 5119)])
def test_a_pruned_layer_holds_what_a_packed_one_of_its_shape_holds(rec, shape, kept):
    """The kept indices are there while the layer is made, not for its life."""
    n_in, n_out, k = shape
    rec.lib.dbf_tuning_reset()
    l, same = rec.layer(*shape), rec.layer(n_in, n_out, kept)
    want, held = rec.lib.rec_last_block(), rec.lib.rec_held()
    keep = np.sort(np.random.default_rng(1).choice(k, kept, replace=False)).astype(np.int32)
    pruned = C.c_void_p()
    try:
        assert rec.lib.dbf_prune_middle(l, C.c_void_p(keep.ctypes.data), kept, C.byref(pruned)) == 0
        assert rec.lib.rec_held() - held == want
    finally:
        for h in (l, same, pruned):
            rec.lib.dbf_free(h)


@pytest.mark.parametrize("shape", [(1, 1, 1), (512, 512, 256), (4096, 4096, 2048), (11008, 4096, 4477)])
def test_dims_reports_all_the_device_memory_a_layer_holds(rec, shape):
    """Launch plan and sums of column pieces included: they live in the layer's block."""
    rec.lib.dbf_tuning_reset()
    l = rec.layer(*shape)
    try:
        n = C.c_size_t()
        assert rec.lib.dbf_dims(l, None, None, None, C.byref(n)) == 0
        assert n.value == rec.lib.rec_last_block()
    finally:
        rec.lib.dbf_free(l)


@pytest.mark.parametrize("n,shape", [(1, (64, 64, 32)), (4, (4096, 4096, 2048)), (12, (512, 512, 256)), (1, (4096, 11008, 4477))])
def test_a_short_stack_is_made_by_one_upload(rec, n, shape):
    """The little memory that must start at zero goes up with the tables: a memset takes 12 us, as much as all the rest of making a
    stack of four layers.  (All of it is zero: the recorder's memory is not to begin with, and calls check the tables on the GPU.)"""
    rec.lib.dbf_tuning_reset()
    layers = [rec.layer(*shape) for _ in range(n)]
    before = rec.lib.rec_memset_bytes()
    stack = rec.stack(layers)
    try:
        assert rec.lib.rec_memset_bytes() == before
        waits = C.c_int(-1)
        assert rec.lib.dbf_stack_sync_timeouts(stack, C.byref(waits)) == 0 and waits.value == 0   # (a counter in that memory)
    finally:
        rec.lib.dbf_stack_free(stack)
        for l in layers:
            rec.lib.dbf_free(l)


@pytest.mark.parametrize("shape", [(64, 64, 32), (65, 129, 63), (300, 100, 200), (128, 640, 64), (512, 512, 256)])
def test_sections_of_a_small_layers_lds_are_read_where_they_are_aligned(rec, shape):
    """The middle activations are the last section of the small-layer kernel's LDS and are read in 16-byte pieces; they and what lies
    before the sums are multiples of 16 bytes, so they start on one if the whole is one (sums of an odd number of row tiles
    for one token are not)."""
    rec.lib.dbf_tuning_reset()
    l = rec.layer(*shape)
    try:
        for batch in (1, 2, 3, 16):
            (name, _, _, lds), = rec.gemv(l, batch)
            assert name == "dbf_small_layer" and lds % 16 == 0, (batch, lds)
    finally:
        rec.lib.dbf_free(l)


@pytest.mark.parametrize("shape,offset,any_rows", [((4096, 4096, 2048), 0, False), ((4096, 4096, 2048), 2, True), ((4095, 4097, 2047), 0, True),
                                                   ((512, 512, 256), 0, False), ((512, 512, 256), 2, True), ((5, 40, 9), 0, True)])
def test_rows_that_cannot_be_read_in_16_byte_pieces_have_kernels_of_their_own(rec, shape, offset, any_rows):
    """... which read them in as few loads and hold them as the others do (calls of 768-1024 columns with a misaligned x had become 8 %
    slower than the launches before them), and the others do without the code for it."""
    rec.lib.dbf_tuning_reset()
    l = rec.layer(*shape)
    try:
        for batch in (1, 8):
            first = rec.gemv(l, batch, offset)[0][0]
            assert first in FEW and rec.full_names[0].split("EEv")[0].rstrip("E").endswith("Lb1" if any_rows else "Lb0"), rec.full_names
    finally:
        rec.lib.dbf_free(l)


@pytest.mark.parametrize("n,shape,batch,few", [(4, (14336, 4096, 3185), 10, False), (6, (6144, 4096, 3000), 8, False), (2, (9216, 4096, 2000), 16, True),
                                               (6, (5120, 2048, 3000), 8, True), (4, (8192, 2048, 2000), 16, True), (4, (14336, 4096, 3185), 4, True),
                                               (2, (14336, 2048, 1000), 8, True), (1, (14336, 4096, 3185), 16, True)])
def test_groups_of_layers_with_many_tokens_of_long_rows_round_them_once(rec, n, shape, batch, few):
    """A group of layers whose workgroups would each round more than four whole long rows goes to the launches that round every layer's
    input once (in the others calls were up to 22 % slower)."""
    rec.lib.dbf_tuning_reset()
    layers = [rec.layer(*shape) for _ in range(n)]
    stack = rec.stack(layers)
    try:
        assert set(_names(rec.stack_gemv(stack, batch))) == ({"dbf_few"} if few else {"dbf_quantise_inputs", "dbf_items_mfma"})
    finally:
        rec.lib.dbf_stack_free(stack)
        for l in layers:
            rec.lib.dbf_free(l)


@pytest.mark.parametrize("shapes,batch,stage", [([(9000, 300, 16700)], 8, 0), ([(12000, 300, 16520)], 6, 0), ([(300, 16700, 14100)], 5, 1),
                                                ([(10301, 256, 16520)], 7, 0), ([(18000, 64, 3000)] * 3, 8, 0), ([(64, 16500, 17300), (64, 64, 64)], 4, 1)])
def test_rows_of_several_lds_chunks_go_to_the_few_workgroup_kernels(rec, shapes, batch, stage):
    """The calls of test_few_workgroups_with_rows_of_several_lds_chunks: with less LDS than the whole rows of their tokens would take."""
    rec.lib.dbf_tuning_reset()
    layers = [rec.layer(*s) for s in shapes]
    stack = rec.stack(layers)
    try:
        launches = rec.gemv(layers[0], batch) if len(layers) == 1 else rec.stack_gemv(stack, batch)
        assert _names(launches) == ["dbf_few"] * 2
        _, (_, groups, pieces), _, lds = launches[stage]
        tokens = -(-batch // groups)
        planes = lds - 656 - 2 * tokens * 129 * 4          # (LDS before and behind the operand planes)
        assert pieces == 1 and planes < (shapes[0][0 if stage == 0 else 2] + 63) // 64 * (2 * tokens + 1) * 64
    finally:
        rec.lib.dbf_stack_free(stack)
        for l in layers:
            rec.lib.dbf_free(l)


@pytest.mark.parametrize("shape", [(256, 33000, 4200), (9000, 200, 33100), (4200, 40000, 5000)])
def test_plans_of_257_to_768_row_tiles_keep_their_column_pieces(rec, shape):
    rec.lib.dbf_tuning_reset()
    l = rec.layer(*shape)
    try:
        launches = rec.gemv(l, 1)
        assert _names(launches) == ["dbf_items_mfma"] * 2
        assert sum(x[1][0] for x in launches) > (shape[1] + 127) // 128 + (shape[2] + 127) // 128
    finally:
        rec.lib.dbf_free(l)


@pytest.mark.parametrize("n,shape,batch,grids", [
    (1, (4096, 4096, 2048), 1, [(16, 4, 1), (32, 4, 1)]), (3, (4096, 4096, 3072), 1, [(72, 2, 1), (96, 2, 1)]),
    (1, (4096, 4096, 3072), 8, [(24, 8, 1), (32, 8, 1)]), (1, (4096, 4096, 3072), 16, [(24, 8, 1), (32, 8, 1)]),
    (3, (4096, 4096, 3072), 8, [(72, 2, 1), (96, 2, 1)]), (1, (28672, 8192, 12743), 1, [(100, 1, 2), (64, 1, 4)]),
    (3, (18000, 64, 3000), 8, [(72, 2, 1), (3, 16, 1)])])
def test_bit_planes_of_a_row_tile_are_dealt_to_idle_compute_units(rec, n, shape, batch, grids):
    """Grids (row tiles, groups of tokens times groups of bit planes, column pieces): at most one workgroup per compute unit; rows of several
    LDS chunks keep all eight bit planes in one workgroup."""
    rec.lib.dbf_tuning_reset()
    layers = [rec.layer(*shape) for _ in range(n)]
    stack = rec.stack(layers)
    try:
        launches = rec.gemv(layers[0], batch) if n == 1 else rec.stack_gemv(stack, batch)
        assert _names(launches) == ["dbf_few"] * 2
        assert [l[1] for l in launches] == grids
    finally:
        rec.lib.dbf_stack_free(stack)
        for l in layers:
            rec.lib.dbf_free(l)


@pytest.mark.parametrize("shape,one_launch_from", [
    ((4096, 4096), 3), ((11008, 4096), None), ((768, 768), 6), ((2048, 10240), 3), ((1240, 10240), 4), ((128, 1024), 6), ((768, 10240), 6),
    ((512, 8192), 8), ((384, 4096), 12), ((128, 2048), 12), ((256, 6144), None), ((128, 8192), None), ((4096, 4095), None), ((64, 1000), None)])
def test_the_projection_is_one_launch_where_that_is_the_faster(rec, shape, one_launch_from):
    """All rounds in one launch from a number of rounds on that depends on the size, never where few workgroups would add up the columns of long rows in
    more than two turns (128 x 8192: eight); a launch a round with a workspace that has no room for what the one launch needs."""
    rows, cols = shape
    rec.lib.dbf_svid_workspace_bytes.restype = C.c_size_t
    ws = rec.lib.dbf_svid_workspace_bytes(rows, cols)

    def names(iters, less=0):
        rec.launches()
        p = C.c_void_p
        assert rec.lib.dbf_svid(p(4096), rows, cols, iters, p(1 << 30), p(1 << 31), p(1 << 32), p(1 << 20), C.c_size_t(ws - less), None) == 0
        return _names(rec.launches())

    one = ["dbf_svid_clear", "dbf_svid_held"]
    for iters in (1, 2, 3, 4, 5, 6, 7, 8, 11, 12, 100):
        got = names(iters)
        assert (got == one) == (one_launch_from is not None and iters >= one_launch_from), (iters, got)
        if got == one:
            assert "dbf_svid_held" not in names(iters, 2304) and len(names(iters, 2304)) >= 2 * iters + 1


def test_the_benchmark_counts_the_passes_over_Z_that_the_projection_makes(rec):
    """bench.py's own statement of the rules against the launches of the calls: one kernel that reads Z is one pass."""
    import importlib.util
    spec = importlib.util.spec_from_file_location("bench_under_test", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    rec.lib.dbf_svid_workspace_bytes.restype = C.c_size_t
    rng = np.random.default_rng(3)
    shapes = [(4096, 4096), (11008, 4096), (16384, 1024), (8192, 2500), (6144, 4096), (10240, 2048), (12288, 2048), (77, 24580), (50, 12288), (50, 12289)]
    shapes += [tuple(int(np.exp(rng.uniform(0, np.log(n)))) for n in (40000, 30000)) for _ in range(150)]
    shapes += [(128 * int(rng.integers(1, 100)) - int(rng.integers(0, 2)), 4 * int(rng.integers(1, 3000))) for _ in range(300)]
    one = 0
    for rows, cols in shapes:
        ws = rec.lib.dbf_svid_workspace_bytes(rows, cols)
        for iters in (1, 2, 3, 4, 6, 8, 12):
            rec.launches()
            p = C.c_void_p
            assert rec.lib.dbf_svid(p(4096), rows, cols, iters, p(1 << 40), p(2 << 40), p(3 << 40), p(4 << 40), C.c_size_t(ws), None) == 0
            reads = [n for n in _names(rec.launches()) if n in ("dbf_svid_held", "dbf_svid_round", "dbf_svid_row_dots", "dbf_svid_col_dots", "dbf_svid_signs")]
            assert bench.svid_passes(rows, cols, iters) == len(reads), (rows, cols, iters, reads)
            one += reads == ["dbf_svid_held"]
    assert one > 300


@pytest.mark.parametrize("p,q,r", [(4096, 2048, 4096), (768, 768, 768), (11008, 1500, 4096), (300, 130, 200), (4096, 4096, 4096), (1024, 2830, 9000),
                                   (2100, 300, 1000), (1100, 200, 16600), (8192, 2880, 16384)])
def test_all_parts_of_C_are_made_and_none_beside_a_row_that_is_there(rec, p, q, r):
    """The elimination's launches have a workgroup per block below a row and, up to 256 in all, one per part of C = B^T W; rows of more blocks are made in a launch of
    their own and have no parts beside them.  All parts of the blocks that the contraction's launch leaves out are among them."""
    P = C.c_void_p
    rec.lib.dbf_admm_prepare_workspace_bytes.restype = C.c_size_t
    ws = rec.lib.dbf_admm_prepare_workspace_bytes(p, q, r)
    rec.launches()
    assert rec.lib.dbf_admm_prepare(*[P(n << 32) for n in (1, 2, 3, 4)], p, q, r, C.c_float(1.0), P(5 << 32), P(6 << 32), P(7 << 32), C.c_size_t(ws), P(8 << 32), None) == 0
    launches = rec.launches()
    n, columns = (q + 127) // 128, (r + 127) // 128
    chunks = (p + 127) // 128
    parts_made = blocks_of_row = 0
    row = 0
    for (name, grid, _, _), full in zip(launches, rec.full_names):
        if name == "dbf_chol_first":
            parts_made += grid[0] - 1
            assert grid[0] <= 256
        elif name == "dbf_chol_row":
            below = n - 1 - row
            blocks = below * (below + 1) // 2 + below * (row + 1)
            made = "ILb1E" in full
            assert made == (blocks > 256)
            assert grid[0] == blocks if made else blocks <= grid[0] <= 256
            parts_made += grid[0] - blocks
            row += 1
    assert row == n - 1
    gemms = [grid for name, grid, _, _ in launches if name == "dbf_split_gemm"]
    beside = columns - (gemms[1][1] if len(gemms) == 3 else 0)   # (B^T B, C, Y^T Y)
    assert len(gemms) in (2, 3) and parts_made == beside * n * ((chunks + 7) // 8)
