"""What a call launches, on what sizes: shapes, occupancy bounds and where the neighbour rows are drawn.
The GPU tests record calls into a HIP graph, read the launches back and never run the graph, so that plans
of any size are looked at without their memory."""
import ctypes

import numpy as np
import pytest

from paper_1909_09010_amd import binding as B

SAMPLER_THREADS = 64                       # the sampler's launches have so many threads, the fused kernel's more


class _Dim3(ctypes.Structure):
    _fields_ = [("x", ctypes.c_uint32), ("y", ctypes.c_uint32), ("z", ctypes.c_uint32)]


class _KernelNodeParams(ctypes.Structure):
    _fields_ = [("block", _Dim3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", _Dim3),
                ("params", ctypes.c_void_p), ("shared", ctypes.c_uint32)]


class _CopyArgs(ctypes.Structure):
    """The argument of the copy kernel (CopyArgs)."""
    _fields_ = [("arrays", ctypes.c_void_p * 6), ("placements", ctypes.c_int64 * 6), ("P", ctypes.c_int64), ("K", ctypes.c_int32),
                ("run_len", ctypes.c_uint32), ("fold", ctypes.c_uint32)]


class _SyncArgs(ctypes.Structure):
    """The beginning of the argument of the fused kernel (SyncArgs)."""
    _fields_ = [("arrays", ctypes.c_void_p * 6), ("stride", ctypes.c_int64), ("block_extra", ctypes.c_int64), ("logB", ctypes.c_int32),
                ("reserved", ctypes.c_int32), ("K", ctypes.c_int32), ("q", ctypes.c_int32), ("logT", ctypes.c_int32), ("xcd_log", ctypes.c_int32),
                ("mode", ctypes.c_int32), ("eta", ctypes.c_float), ("zeta", ctypes.c_float), ("inv", ctypes.c_float), ("flags", ctypes.c_int32)]


ROTATE = 64                                # in _SyncArgs.flags


def launches(call, kernels=False, args=None):
    """[(blocks, threads, LDS bytes)] of what ``call(stream)`` enqueues, or which kernels, or their one argument; nothing runs."""
    import torch
    hip = ctypes.CDLL(B.LIB_PATH)          # the HIP runtime that the library itself is bound to
    stream = torch.cuda.Stream()
    graph, count = ctypes.c_void_p(), ctypes.c_size_t()
    assert hip.hipStreamBeginCapture(ctypes.c_void_p(stream.cuda_stream), 1) == 0        # thread-local mode
    try:
        call(stream.cuda_stream)
    finally:
        assert hip.hipStreamEndCapture(ctypes.c_void_p(stream.cuda_stream), ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(count)) == 0
    nodes = (ctypes.c_void_p * max(1, count.value))()
    assert hip.hipGraphGetNodes(graph, nodes, ctypes.byref(count)) == 0
    out = []
    for node in nodes[:count.value]:
        kind, p = ctypes.c_int(-1), _KernelNodeParams()
        assert hip.hipGraphNodeGetType(ctypes.c_void_p(node), ctypes.byref(kind)) == 0 and kind.value == 0   # a kernel
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
        if args is not None:
            first = ctypes.cast(p.params, ctypes.POINTER(ctypes.c_void_p))[0]
            out.append(args.from_buffer_copy(ctypes.string_at(first, ctypes.sizeof(args))))
            continue
        out.append(p.func if kernels else (p.grid.x * p.grid.y * p.grid.z, p.block.x, p.shared))
    assert hip.hipGraphDestroy(graph) == 0
    return out


def fused_args(call):
    """The argument of the fused kernel that ``call(stream)`` launches after the sampler."""
    return launches(call, args=_SyncArgs)[-1]


def tile_kinds(call):
    """How many tiles of the launch lie side by side, in stretches spread over 64 tiles' worth of a row, over 64 KB (TileDesc)."""
    (blocks, _, _), node = launches(call)[-1], fused_args(call)
    tiles = np.zeros((blocks, 8), dtype=np.uint16)
    hip = ctypes.CDLL(B.LIB_PATH)
    assert hip.hipMemcpy(tiles.ctypes.data_as(ctypes.c_void_p), ctypes.c_void_p(node.arrays[0]), ctypes.c_size_t(tiles.nbytes), 2) == 0      # device to host
    return np.bincount(tiles[:, 5] >> 14, minlength=3).tolist()


def fake_state(plan, place="blocked", aligned=True):
    """A state of the plan's size at addresses that nothing may touch."""
    K, P, base = plan.info.K, plan.info.P, 1 << 40
    if place == "blocked":
        lay = B.recommend_layout(P, K, plan=plan)
        at = [base, base + 4 * lay.omega_offset, base + 4 * lay.delta_offset]
        return B.make_state(*at, lay.worker_stride, lay.block_floats, lay.block_stride)
    stride = -(-P // 1024) * 1024 if aligned else P | 1
    return B.make_state(*[base + 4 * a * (-(-K * stride // 1024) * 1024) for a in range(3)], stride)


def need_gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# Kernels for tiles in stretches are theirs alone: 40 workers' blocks and 12 workers' aligned rows both take 512 x 4 in gossip-MA, and
# blocks waited for their neighbour table before the first load of theta while the kernel was one (40 x 22 M 1102 us, 1068).
@pytest.mark.gpu
@pytest.mark.parametrize("values", [150_000_000, 600_000_000])
def test_blocks_take_no_kernel_of_tiles_in_stretches(values):
    need_gpu()
    seen = []
    for K, place in ((40, "blocked"), (12, "rows")):
        pl = B.Plan([0, values // K], K, 2, 0)
        call = lambda s: pl.sync_state(fake_state(pl, place), 0.9, 1.0, B.MODE_GOSSIP_MA, 0, s)
        seen.append((launches(call)[-1][1], launches(call, kernels=True)[-1]))
        pl.destroy()
    assert seen[0][0] == seen[1][0] == 512 and seen[0][1] != seen[1][1]


def cut(values, K, size):
    """Components of `size` floats, the last one what is left; 0: one component."""
    P = values // K
    return [*range(0, P, size or P), P]


# Aligned rows in short components: shapes of their own, (threads, columns), next to those of the same rows in long ones.  In the latter
# 2 x 150 M 14 % longer, 4 x 175 M 14, 6 x 117 M 7, 8 x 87 M 11, 12 x 58 M 14, 32 x 0.9 M 5.
@pytest.mark.parametrize("values", [30_000_000, 300_000_000])
def test_rows_in_short_components_take_shapes_of_their_own(values):
    wide = {1: (256, 512), 2: (256, 256), 3: (512, 128), 4: (256, 128), 5: (1024, 256), 6: (1024, 256), 7: (1024, 256), 8: (1024, 256), 9: (1024, 256), 12: (1024, 256),
            13: (1024, 128), 16: (1024, 128), 17: (1024, 128), 32: (1024, 128), 33: (512, 128), 39: (512, 128), 48: (512, 128), 64: (512, 128), 65: (512, 64)}
    fine = {1: (256, 256), 2: (256, 128), 3: (256, 64), 4: (256, 64), 5: (512, 64), 6: (512, 64), 7: (256, 64), 8: (256, 64), 9: (1024, 128), 12: (1024, 128),
            13: (1024, 128), 16: (1024, 128), 17: (1024, 64), 32: (1024, 64), 33: (512, 128), 39: (512, 128), 48: (1024, 64), 64: (1024, 64), 65: (512, 64)}
    for K in wide:
        for size, expect in ((0, wide), (5120, fine), (32512, fine), (320_000, wide), (16384, wide), (49152, wide), (16385, fine)):
            pl = B.Plan(cut(values, K, size), K, min(K - 1, 2), 0)
            assert (pl.info.threads, pl.info.tile_columns) == expect[K], (K, size)
            pl.destroy()


# How long a component has to be: 8 x 19 M of 75 K floats 3 % longer as if it were short, 8 x 87 M 5 % less.
@pytest.mark.parametrize("K,values,size,wide", [(3, 300_000_000, 48_000, False), (3, 300_000_000, 50_001, True), (4, 600_000_000, 50_001, True), (8, 150_000_000, 48_000, False),
                                                (8, 150_000_000, 75_001, True), (8, 600_000_000, 75_001, False), (8, 600_000_000, 164_001, True), (10, 150_000_000, 75_001, False),
                                                (10, 150_000_000, 164_001, True), (2, 150_000_000, 75_001, False), (2, 150_000_000, 132_001, True), (32, 150_000_000, 33_001, True)])
def test_how_long_a_long_component_is(K, values, size, wide):
    shapes = []
    for n in (size, 0):
        pl = B.Plan(cut(values, K, n), K, 1, 0)
        shapes.append((pl.info.threads, pl.info.tile_columns))
        pl.destroy()
    assert (shapes[0] == shapes[1]) == wide


# Which of them have tiles in stretches 32 KB apart: none of 32 columns, and components of less than 64 KB no group of them.
@pytest.mark.gpu
@pytest.mark.parametrize("mode", [B.MODE_PAPER, B.MODE_GOSSIP_MA])
@pytest.mark.parametrize("K", [1, 2, 3, 4, 5, 8, 10, 16, 24, 32, 33, 48, 64, 65, 128, 200])
def test_which_rows_have_tiles_in_stretches(K, mode):
    need_gpu()
    ma = mode == B.MODE_GOSSIP_MA
    for values in (4_000_000, 10_000_000, 30_000_000, 600_000_000):
        for size in (0, 5120, 20_480):
            pl = B.Plan(cut(values, K, size), K, min(K - 1, 2), 0)
            call = lambda s: pl.sync_state(fake_state(pl, "rows"), 0.9, 1.0, mode, 0, s)
            kinds, log = tile_kinds(call), fused_args(call).logT
            if values < 20_000_000:
                expect = values > 5_000_000 and log > 5 and size != 5120 and (ma or K <= 16)
            else:
                expect = K <= 128 and size != 5120 and not (ma and K == 3) and not (size and K <= 32 and (K != 3 or values < 500_000_000))
            assert sum(kinds[1:]) >= sum(kinds) * (0.6 if size else 0.9) if expect else kinds[1:] == [0, 0], (values, size, kinds)
            assert kinds[2] == 0 or log > 6                      # else 64 tiles are 64 KB
            pl.destroy()


# Gossip-MA of more than 4 neighbours: (threads, columns, stretches).  In the shapes of few neighbours 64 x 0.9 M 17 % longer, 48 x 0.9 M 24, 20 x 30 M 8.
@pytest.mark.gpu
@pytest.mark.parametrize("values", [30_000_000, 600_000_000])
def test_gossip_ma_of_long_averages_takes_smaller_tiles(values):
    need_gpu()
    wide = {6: (512, 256, 1), 8: (512, 128, 1), 12: (512, 128, 1), 16: (512, 128, 1), 20: (512, 64, 1), 24: (512, 64, 1), 28: (1024, 128, 1), 32: (1024, 128, 1),
            33: (512, 128, 1), 64: (512, 128, 1), 65: (512, 64, 1)}
    small = {8: (256, 64, 1), 12: (256, 64, 1), 16: (256, 64, 1), 20: (256, 32, 0), 24: (256, 32, 0), 33: (1024, 64, 0), 64: (1024, 64, 0)}
    many = {**small, 12: (256, 64, 0), 16: (256, 64, 0), 28: (1024, 128, 0), 32: (1024, 128, 0), 65: (1024, 32, 0)}
    for K in wide:
        for q, expect in ((4, wide), ([2, 4], wide), (5, small), ([1, 5], small), (9, many), ([9, 1], many)):
            if np.max(q) >= K:
                continue
            pl = B.Plan([0, values // K // 2, values // K] if np.ndim(q) else [0, values // K], K, q, 5, sampling=B.SAMPLING_SEPARATE)
            call = lambda s: pl.sync_state(fake_state(pl, "rows"), 0.9, 1.0, B.MODE_GOSSIP_MA, 0, s)
            assert (launches(call)[-1][1], 1 << fused_args(call).logT, int(sum(tile_kinds(call)[1:]) > 0)) == expect.get(K, wide[K]), (K, q)
            pl.destroy()


# Rows far from each other, in tiles of 64 columns: side by side (65 x 77 M in stretches 17 % longer, 32 x 0.33 M of rows of 53 M 30 %).
@pytest.mark.gpu
@pytest.mark.parametrize("mode", [B.MODE_PAPER, B.MODE_GOSSIP_MA])
def test_rows_far_from_each_other_have_no_narrow_tiles_in_stretches(mode):
    need_gpu()
    ma = mode == B.MODE_GOSSIP_MA
    def look(K, P, due):                                     # `due` values of rows of P floats
        n = min(due // K, P)
        pl = B.Plan([0, n, P], K, 2, 0, periods=[1, 2])
        call = lambda s: pl.sync_step_state(fake_state(pl, "rows"), 0.9, 1.0, mode, 1, s)
        got = launches(call)[-1][1], 1 << fused_args(call).logT, sum(tile_kinds(call)[1:]) > 0
        pl.destroy()
        return got
    for K in (17, 32, 33, 48, 64, 65, 100, 128):
        for P in (21_000_000, 23_000_000, 60_000_000):
            for due in (12_000_000, 50_000_000, K * P):
                threads, columns, apart = look(K, P, due)
                assert not (apart and columns == 64 and P > 22_000_000) or (ma and K <= 24)
                assert apart == (due > 20_000_000 and (K <= 64 or P < 22_000_000))
                if K > 64 and due == 50_000_000 and not ma:
                    assert (threads, columns) == ((512, 64) if P < 22_000_000 else (512, 16))
    for K in (40, 64):                                       # short components
        for P, expect in ((4_000_000, (1024, 64, True)), (30_000_000, (512, 32, False))):
            pl = B.Plan([*cut(100_000_000, K, 20_480), P], K, 2, 0, periods=[1] * (len(cut(100_000_000, K, 20_480)) - 1) + [2])
            call = lambda s: pl.sync_step_state(fake_state(pl, "rows"), 0.9, 1.0, B.MODE_PAPER, 1, s)
            assert (launches(call)[-1][1], 1 << fused_args(call).logT, sum(tile_kinds(call)[1:]) > 0) == expect
            pl.destroy()


# With sync periods it depends on what is due.
@pytest.mark.gpu
@pytest.mark.parametrize("mode", [B.MODE_PAPER, B.MODE_GOSSIP_MA])
@pytest.mark.parametrize("K", [2, 8, 13, 16, 32])
def test_a_step_of_short_components_runs_like_a_sync_of_them(K, mode):
    need_gpu()
    short = cut(150_000_000, K, 15_872)
    n, long = len(short) - 1, 200_000_000 // K
    off = [0, *(long + np.asarray(short))]
    pl, whole, part = B.Plan(off, K, 1, 0, periods=[2] + [1] * n), B.Plan(off, K, 1, 0), B.Plan(short, K, 1, 0)
    look = lambda p, call, r: (lambda c: (launches(c)[-1], launches(c, kernels=True)[-1], tile_kinds(c)))(lambda s: call(fake_state(p, "rows"), 0.9, 1.0, mode, r, s))
    everything, shorts = look(whole, whole.sync_state, 0), look(part, part.sync_state, 0)
    assert everything[2][1] > 0 and shorts[2][1:] == [0, 0]
    assert look(pl, pl.sync_state, 0) == look(pl, pl.sync_step_state, 2) == everything
    step = look(pl, pl.sync_step_state, 1)
    assert step[0][1:] == shorts[0][1:] and step[1] == shorts[1] and step[2][1:] == [0, 0]
    assert abs(step[0][0] - shorts[0][0]) <= n               # the components begin elsewhere in the row


# Whatever is due, the tiles of a launch are those of its own width: lists of components of all lengths, some of them empty, under periods.
@pytest.mark.gpu
@pytest.mark.parametrize("seed", range(40))
def test_a_launch_takes_the_tile_list_of_its_width(seed):
    need_gpu()
    rng = np.random.default_rng(seed)
    K = int(rng.choice([1, 2, 3, 4, 6, 8, 12, 16, 20, 32, 36, 48, 64, 100, 200]))
    values = 10 ** rng.uniform(6, 9)
    sizes = [rng.integers(0, 3, n) * rng.integers(1, 2 * m, n) for n, m in ((30, 300), (200, 15_000), (50, 60_000), (10, 400_000), (3, 5_000_000)) if rng.random() < 0.6]
    sizes = np.concatenate([*sizes, [1 + int(values) // K // 2]])
    rng.shuffle(sizes)
    off = np.concatenate([[0], np.cumsum(sizes[: 1 + int(np.searchsorted(np.cumsum(sizes), values / K))])]).astype(np.int64)
    m = len(off) - 1
    periods = rng.choice([1, 2, 3], m) if rng.random() < 0.5 else np.where(np.diff(off) < 40_000, 2, 3)
    pl = B.Plan(off, K, [int(x) for x in rng.integers(0, min(K, 4), m)], 3, periods=[int(h) for h in periods], sampling=B.SAMPLING_SEPARATE)
    for place, aligned in (("rows", True), ("rows", False), ("blocked", True)):
        for mode in (B.MODE_PAPER, B.MODE_GOSSIP_MA):
            for step in (1, 2, 3, 6):
                call = lambda s: pl.sync_step_state(fake_state(pl, place, aligned), 0.9, 1.0, mode, step, s)
                due = np.flatnonzero((step % periods == 0) & (np.diff(off) > 0))
                got = launches(call)
                if due.size == 0:
                    assert got == []
                    continue
                T = 4 << fused_args(call).logT
                tiles = np.where(np.diff(off) > 0, -(-off[1:] // T) - off[:-1] // T, 0)
                between = np.diff(off)[due[0]:due[-1] + 1] > 0
                one_run = not np.any(between & (step % periods[due[0]:due[-1] + 1] != 0))
                assert got[-1][0] == (tiles[due[0]:due[-1] + 1].sum() if one_run else tiles.sum()), (K, place, mode, step)
    pl.destroy()


# The component that syncs most often is a bias, or empty; all the others sync every 16th time.  A sync of everything
# has to run like that of a plan without periods.
RARE = [83_070_000 // 8] * 8


@pytest.mark.parametrize("often", [0, 512])
@pytest.mark.parametrize("K", [8, 16, 32, 64])
def test_the_rate_of_syncs_does_not_change_how_all_components_are_synced(K, often):
    off = np.concatenate([[0], np.cumsum([often] + RARE)])
    with_periods, without = B.Plan(off, K, 2, 0, periods=[1] + [16] * 8).info, B.Plan(off, K, 2, 0).info
    for name in ("n_tiles", "tile_columns", "threads", "tile_columns_blocked", "threads_blocked", "workgroups_per_cu_blocked",
                 "tile_columns_blocked_ma", "min_block_floats", "in_kernel_sampling"):
        assert getattr(with_periods, name) == getattr(without, name), name


@pytest.mark.gpu
@pytest.mark.parametrize("place", ["blocked", "rows"])
@pytest.mark.parametrize("mode", [B.MODE_PAPER, B.MODE_GOSSIP_MA])
def test_a_step_runs_like_a_sync_of_what_is_due(place, mode):
    need_gpu()
    K, often = 16, 30_000_000
    off = np.concatenate([[0], np.cumsum([often] + RARE)])
    pl = B.Plan(off, K, 2, 0, periods=[1] + [16] * 8)
    whole, part = B.Plan(off, K, 2, 0), B.Plan([0, often], K, 2, 0)
    run = lambda p, call: launches(lambda s: call(fake_state(p, place), 0.9, 1.0, mode, 16, s))
    everything, frequent = run(whole, whole.sync_state), run(part, part.sync_state)
    # 1.8 G values: the rows are drawn by a kernel of their own; 480 M: in the fused kernel (gossip-MA moves a third)
    assert len(everything) == 2 and len(frequent) == (2 if mode == B.MODE_GOSSIP_MA else 1)
    assert run(pl, pl.sync_state) == everything and run(pl, pl.sync_step_state) == everything
    got = launches(lambda s: pl.sync_step_state(fake_state(pl, place), 0.9, 1.0, mode, 17, s))
    assert got[-1] == frequent[-1] and len(got) == len(frequent)
    assert pl.info.in_kernel_sampling == 0                              # not all of its calls draw that way


@pytest.mark.gpu
@pytest.mark.parametrize("often", [[0], [512]])
def test_a_tiny_frequent_component_does_not_unbound_the_rest(often):
    need_gpu()
    off = np.concatenate([[0], np.cumsum(often + RARE)])
    pl, without = B.Plan(off, 16, 2, 0, periods=[1] + [16] * 8), B.Plan(off, 16, 2, 0)
    for place in ("blocked", "rows"):
        st = fake_state(pl, place)
        everything = launches(lambda s: without.sync_state(st, 0.9, 1.0, 1, 0, s))
        assert launches(lambda s: pl.sync_state(st, 0.9, 1.0, 1, 0, s)) == everything
        step = launches(lambda s: pl.sync_step_state(st, 0.9, 1.0, 1, 0, s))
        assert len(step) == len(everything) == 2 and step[-1] == everything[-1]        # an empty component is not sampled
        rare = launches(lambda s: pl.sync_step_state(st, 0.9, 1.0, 1, 1, s))
        assert rare == [] if often == [0] else len(rare) == 1 and rare[0][0] <= 8


def shape(K, values, place, aligned=True, mode=B.MODE_PAPER):
    """(threads, columns of a tile, LDS bytes, floats of a row that one XCD takes, whether these move on) of a sync."""
    pl = B.Plan([0, values // K], K, min(2, K - 1), 0, sampling=B.SAMPLING_SEPARATE)
    call = lambda s: pl.sync_state(fake_state(pl, place, aligned), 0.9, 1.0, mode, 0, s)
    _, threads, lds = launches(call)[-1]
    node = fused_args(call)
    pl.destroy()
    return threads, 1 << node.logT, lds, 4 << node.logT + node.xcd_log, bool(node.flags & ROTATE)


# Aligned rows of 33 to 128 workers beyond the caches: the XCDs take tiles one by one (4 KB of a row each: 64 x 4.7 M 15 % longer).
@pytest.mark.gpu
@pytest.mark.parametrize("K", [33, 48, 64, 96, 128])
@pytest.mark.parametrize("values", [25_000_000, 150_000_000, 480_000_000])
def test_aligned_rows_go_to_the_xcds_tile_by_tile(K, values):
    need_gpu()
    threads, columns, _, run, rotate = shape(K, values, "rows")
    assert threads == 512 and run == 4 * columns and not rotate
    assert shape(160, values, "rows")[3] == shape(K, 15_000_000, "rows")[3] == 1024


# Rows that share cache lines: an XCD takes 32 KB of a row, or so much less that 4 groups of 8 such runs are whole: tiles beyond the last
# go to the XCDs one by one (128 x 47 K, gossip-MA: all of them, 40 % longer).
@pytest.mark.gpu
@pytest.mark.parametrize("mode", [B.MODE_PAPER, B.MODE_GOSSIP_MA])
@pytest.mark.parametrize("K", [2, 8, 16, 64, 128, 300, 1024])
def test_runs_of_tiles_are_whole_where_rows_share_lines(K, mode):
    need_gpu()
    for values in (200_000, 1_500_000, 6_000_000, 20_000_000, 100_000_000, 1_000_000_000):
        _, columns, _, run, rotate = shape(K, values, "rows", False, mode)
        groups = lambda run: -(-(values // K) // (4 * columns)) // (8 * run // (4 * columns))
        assert not rotate and run <= 8192 and (groups(run) >= 4 or run == 4 * columns)
        assert run == 8192 or groups(2 * run) < 4


# Gossip-MA of 2 and 4 workers' rows that share cache lines: (threads, columns, workgroups per CU).  In 512 x 2 3 to 8 % longer.
@pytest.mark.gpu
@pytest.mark.parametrize("values,two,three,four", [(65_000_000, (256, 512, 3), (512, 256, 0), (256, 256, 3)), (145_000_000, (256, 512, 3), (512, 256, 0), (256, 256, 3)),
                                                   (155_000_000, (512, 2048, 2), (1024, 1024, 0), (1024, 1024, 0)),
                                                   (600_000_000, (512, 2048, 2), (1024, 1024, 0), (1024, 1024, 0))])
def test_shapes_of_gossip_ma_of_few_odd_rows(values, two, three, four):
    need_gpu()
    for K, (threads, columns, bound) in ((2, two), (3, three), (4, four)):
        got = shape(K, values, "rows", False, B.MODE_GOSSIP_MA)
        assert got[:2] == (threads, columns)
        assert bound == 0 or got[2] == 160 * 1024 // bound - 2048


# Gossip-MA of few blocks (5 x 140 M 18 % longer in 256 x 4, 4 x 175 M 6 % in 256 x 2).
@pytest.mark.gpu
@pytest.mark.parametrize("values", [30_000_000, 300_000_000, 700_000_000])
def test_shapes_of_gossip_ma_of_few_blocks(values):
    need_gpu()
    got = {K: shape(K, values, "blocked", mode=B.MODE_GOSSIP_MA) for K in (2, 3, 4, 5, 6, 7, 8)}
    assert {K for K in got if got[K][0] == 512} == ({2, 4} if values > 500_000_000 else {4})
    assert got[4][1] == 256 and got[4][2] < 24 * 1024
    assert [got[K][1] for K in (3, 5, 6, 7, 8)] == [256, 64, 64, 64, 64]


# Gossip-MA of 7 and more blocks in 256 x 2: six workgroups per CU (7 x 271 M unbounded 3 % longer), of 5 and 6 all that fit (5 x 380 M six 3 % longer).
@pytest.mark.gpu
@pytest.mark.parametrize("values", [30_000_000, 1_900_000_000])
def test_bounds_of_gossip_ma_of_blocks(values):
    need_gpu()
    for K, bound in ((5, 0), (6, 0), (7, 6), (8, 6), (12, 0), (14, 6), (15, 6), (16, 6), (24, 0)):
        for q in (1, 4, [2, 1]):
            pl = B.Plan([0, values // K // 2, values // K] if np.ndim(q) else [0, values // K], K, q, 3)
            lds = launches(lambda s: pl.sync_state(fake_state(pl), 0.9, 1.0, B.MODE_GOSSIP_MA, 0, s))[-1][2]
            assert lds == 160 * 1024 // bound - 2048 if bound else lds < 20 * 1024, (K, q)
            pl.destroy()


# Components that draw different numbers of neighbours, whose 1/(q+1) no tile waits for: fewer workgroups per CU for 3 and 4 blocks and for 17 to 32.
@pytest.mark.parametrize("values", [6_000_000, 100_000_000, 900_000_000])
def test_bounds_of_mixed_neighbours_on_blocks(values):
    def bounds(K):
        P = values // K
        return [B.Plan([0, P // 2, P], K, q, 0).info.workgroups_per_cu_blocked for q in (1, [1, 2])]
    assert [bounds(K) for K in (3, 4, 5, 16, 17, 32, 33)] == [[6, 5], [6, 5], [0, 0], [0, 0], [0, 2], [0, 2], [0, 0]]


# Blocked state beyond the caches: the XCDs' tiles move on from block to block, but for 257 to 512 workers, whose tiles hold 256 bytes of a
# row and who take 1 KB of it in one run (one tile each, moving on, 5 % longer).
@pytest.mark.gpu
@pytest.mark.parametrize("values", [30_000_000, 300_000_000, 1_000_000_000])
def test_which_xcd_takes_which_blocks(values):
    need_gpu()
    for K in (129, 200, 256, 257, 300, 400, 480, 481, 512, 513, 1000):
        _, columns, _, run, rotate = shape(K, values, "blocked")
        assert (run, rotate) == ((256 if K <= 480 else 1024, False) if 256 < K <= 512 else (4 * columns, True))
        assert columns == (32 if K <= 256 else 16 if K <= 480 else 8)


# 5 to 8 workers' aligned rows of 5 to 20 M values take small tiles like fewer workers' (in 1024 x 1 up to 40 % longer).
@pytest.mark.gpu
@pytest.mark.parametrize("K", [4, 5, 6, 7, 8])
def test_aligned_rows_of_few_workers_take_small_tiles(K):
    need_gpu()
    for values in (5_500_000, 12_000_000, 19_500_000):
        threads, _, lds, _, _ = shape(K, values, "rows")
        assert threads == 256 and lds == 160 * 1024 // 4 - 2048
    assert (shape(K, 30_000_000, "rows")[0] == 256) == (K == 4)


# Rows that share cache lines: 1024 x 1 where K rows fill it (14 workers do not: 3 % longer), 33 to 39 workers wide tiles of their
# own (4 % longer in 1024 x 2).
@pytest.mark.gpu
@pytest.mark.parametrize("values", [100_000_000, 600_000_000])
def test_shapes_of_rows_that_share_lines(values):
    need_gpu()
    got = {K: shape(K, values, "rows", aligned=False) for K in (3, 5, 6, 7, 8, 9, 13, 14, 15, 16, 32, 33, 36, 39, 40, 64)}
    wide = {K for K in got if K <= 16 and got[K][0] == 1024}
    assert wide == {3, 7, 8, 15, 16} | ({6} if values > 500_000_000 else set())
    assert all(got[K][1] == 64 and got[K][2] > 64 * 1024 for K in (33, 36, 39)) and got[40][1] == got[64][1] == 32
    assert all(got[K][3] == 8192 for K in got)


# More than 7 neighbours are drawn through LDS, which only plans of up to 8192 tiles of about 32 columns do.
@pytest.mark.gpu
@pytest.mark.parametrize("K,p,q,most", [(8, -1, 7, None), (9, -1, 8, 8192 * 128), (16, -1, 8, 8192 * 128), (32, -1, 20, 8192 * 128),
                                        (64, 16, 8, 8192 * 256), (200, 5, 9, 8192 * 64)])
def test_only_small_plans_draw_through_lds(K, p, q, most):
    need_gpu()
    for P, expect in ((most, 1), (most + 1, 2)) if most else ((1 << 22, 1),):
        pl = B.Plan([0, P], K, q, p)
        assert pl.info.in_kernel_sampling == 2 - expect
        for place in ("blocked", "rows"):
            assert len(launches(lambda s: pl.sync_state(fake_state(pl, place), 0.9, 1.0, B.MODE_PAPER, 0, s))) == expect
        pl.destroy()


# Small states of many workers: a tile for every CU.
@pytest.mark.parametrize("K", [40, 64, 100, 130, 200, 256, 400, 512, 600, 1024])
def test_small_states_are_cut_into_enough_tiles(K):
    P = 4 * 1024 * 1024 // K
    info = B.Plan([0, P], K, 2, 0).info
    assert info.n_tiles >= 256 and P / (4 * info.tile_columns_blocked) >= 256 and P / (4 * info.tile_columns_blocked_ma) >= 128


# One rule per range of workers: inside a range nothing changes from one number of workers to the next.
@pytest.mark.parametrize("lo,hi", [(17, 32), (33, 64), (65, 128), (129, 512), (513, 1024)])
@pytest.mark.parametrize("values", [3_000_000, 200_000_000, 1_500_000_000])
def test_shapes_change_only_between_ranges_of_workers(lo, hi, values):
    infos = [B.Plan([0, values // K], K, 2, 0).info for K in range(lo, hi + 1, max(1, (hi - lo) // 16))]
    assert len({(i.threads, i.threads_blocked, i.workgroups_per_cu_blocked) for i in infos}) == 1


# A plan that names its shape but no bound: none on rows, a few workgroups per CU on blocked state.
@pytest.mark.gpu
@pytest.mark.parametrize("K,tile,blocked", [(4, (256, 1), 4), (8, (256, 1), 2), (16, (256, 4), 2), (32, (1024, 1), 2), (48, (512, 4), 1), (64, (1024, 1), 1)])
@pytest.mark.parametrize("P", [4096, 20_000_000])
def test_named_shapes_are_bound_by_layout_alone(K, tile, blocked, P):
    need_gpu()
    pl = B.Plan([0, P], K, 2, 0, tile=tile)
    needed = 16 * tile[0] * tile[1] + 16 * K                             # the tile and the neighbour rows, 4 ids each at most 8
    assert launches(lambda s: pl.sync_state(fake_state(pl, "rows"), 0.9, 1.0, B.MODE_PAPER, 0, s))[-1][2] <= needed
    lds = launches(lambda s: pl.sync_state(fake_state(pl), 0.9, 1.0, B.MODE_PAPER, 0, s))[-1][2]
    assert pl.info.workgroups_per_cu_blocked == blocked and lds >= 160 * 1024 // blocked - 4096
    pl.destroy()


# Plans that draw rows of more than 7 neighbours through LDS keep tiles of 32 columns: the draws are paid per tile.
@pytest.mark.parametrize("K,P", [(10, 100_000), (17, 700_000), (24, 500_000), (36, 330_000), (64, 60_000)])
def test_drawing_through_lds_takes_wide_tiles(K, P):
    info = B.Plan([0, P], K, 9, 5).info
    assert info.tile_columns >= 32 and info.tile_columns_blocked >= 32


# A final average asks for LDS that bounds the resident workgroups per CU, except where the more the faster: sums that
# the caches hold, and a single worker, which is a copy (1 x 590 M: 1303 us with 8 workgroups per CU, 746 without bound).
@pytest.mark.gpu
@pytest.mark.parametrize("place,aligned", [("blocked", True), ("rows", True), ("rows", False)])
@pytest.mark.parametrize("K,values,bounded", [(1, 600_000_000, False), (1, 9_000_000, False), (8, 40_000_000, False),
                                              (2, 150_000_000, True), (16, 150_000_000, True), (64, 59_000_000, False),
                                              (1024, 40_000_000, False), (1024, 600_000_000, True)])
def test_what_bounds_a_final_average(K, values, bounded, place, aligned):
    need_gpu()
    pl = B.Plan([0, values // K], K, 0, 0, seed=0)
    (blocks, threads, lds), = launches(lambda s: pl.final_average_state(fake_state(pl, place, aligned), 1 << 36, s))
    P = values // K
    assert threads == 64 and blocks == -(-(P // 4) // 64) + (P % 4 > 0)
    assert (lds > 0) == (bounded and not (K <= 3 and place == "blocked"))


# Sums whose theta stays in the caches from one of three states to the next are read by plain loads: streamed ones took
# up to 12 % longer at 21 M values, plain ones at 25 M.
@pytest.mark.gpu
@pytest.mark.parametrize("place,aligned", [("blocked", True), ("rows", True), ("rows", False)])
@pytest.mark.parametrize("K", [5, 8, 20, 64])
def test_a_final_average_from_the_caches_leaves_them_as_they_are(K, place, aligned):
    need_gpu()
    kernel = []
    for values in (10_000_000, 19_500_000 if place == "blocked" and K > 16 else 21_500_000, 25_000_000, 50_000_000):
        pl = B.Plan([0, values // K], K, 0, 0, seed=0)
        kernel += launches(lambda s: pl.final_average_state(fake_state(pl, place, aligned), 1 << 36, s), kernels=True)
        pl.destroy()
    assert kernel[0] == kernel[1] != kernel[2] == kernel[3]


# Sixteen rows in flight are for workers who nearly fill them: with 9 to 13 of them a final average of blocks took 8 to 25 % longer
# than with 4 rows and twice the waves.
@pytest.mark.gpu
@pytest.mark.parametrize("values", [70_000_000, 400_000_000, 1_200_000_000])
def test_rows_in_flight_of_a_final_average_are_filled(values):
    need_gpu()
    seen = {}
    for K in range(8, 17):
        pl = B.Plan([0, values // K], K, 0, 0, seed=0)
        call = lambda s: pl.final_average_state(fake_state(pl), 1 << 36, s)
        seen[K] = launches(call, kernels=True)[0], launches(call)[0][2]
        pl.destroy()
    assert len({seen[K] for K in range(8, 14)}) == len({seen[K] for K in range(14, 17)}) == 1
    assert seen[8][0] != seen[14][0] and seen[8][1] < seen[14][1]


# A final average takes its workgroups in rounds of as many as are resident: the last round is not nearly empty (128 x 0.59 M, 8.9
# workgroups per CU: 60 us in rounds of 8, 47 at once).
@pytest.mark.gpu
@pytest.mark.parametrize("place", ["blocked", "rows"])
@pytest.mark.parametrize("K,per_cu,waves", [(128, 8.9, 16), (300, 7.2, 8), (300, 10.6, 6), (96, 14.3, 8), (300, 15.3, 8),
                                            (65, 17.6, 6), (72, 19.1, 7), (60, 19.1, 7), (300, 17.9, 6), (200, 99, 6)])
def test_no_nearly_empty_last_round_of_a_final_average(K, per_cu, waves, place):
    need_gpu()
    import torch
    props = torch.cuda.get_device_properties(0)
    pl = B.Plan([0, int(per_cu * props.multi_processor_count) * 256], K, 0, 0, seed=0)
    (_, _, lds), = launches(lambda s: pl.final_average_state(fake_state(pl, place), 1 << 36, s))
    assert lds == 160 * 1024 // waves - 2048
    pl.destroy()


# A copy launches a workgroup for every 4 KB of a row, in runs of equal length, so that less than one for a run is
# left over, and no multiple of the work where a row is little longer than a run (512 blocks of 9 pieces in runs of 8: 26 us, 19 as
# launched; 1024 x 1000 in runs of 32: 58 us, 13).
@pytest.mark.gpu
@pytest.mark.parametrize("to", ["rows", "blocked"])
@pytest.mark.parametrize("frm", ["rows", "blocked"])
@pytest.mark.parametrize("K,P", [(1, 5), (16, 1000), (64, 1000), (1024, 1000), (256, 3000), (1024, 40_000), (8, 200_000), (512, 8200), (1024, 8200),
                                 (1024, 16_500), (1024, 40_500), (16, 270_000), (24, 1_100_000), (100, 700_000)])
@pytest.mark.parametrize("which", [1, 7])
def test_a_copy_launches_no_more_than_its_rows(which, K, P, frm, to):
    need_gpu()
    pl = B.Plan([0, P], K, 0, 0, seed=0)
    (blocks, threads, _), = launches(lambda s: pl.state_copy(fake_state(pl, to), fake_state(pl, frm), which, s))
    pieces, arrays = -(-(P + 31) // 1024), bin(which).count("1")
    assert threads == 256 and pieces * K * arrays <= blocks <= (pieces + pieces // 8) * K * arrays
    pl.destroy()


# (run, arrays that follow each other) of copies from rows into blocks: rows of 33 to 60 workers are copied whole only where the
# caches hold them (40 x 0.75 M 130 us, in runs of 64 KB 117); runs of 64 KB up to 200 workers (64 x 0.94 M 241 us, in runs of 32 KB 279).
@pytest.mark.gpu
@pytest.mark.parametrize("aligned", [True, False])
@pytest.mark.parametrize("K,values,walk", [(32, 17_000_000, (32, 3)), (33, 14_000_000, None), (33, 17_000_000, (16, 3)), (60, 30_000_000, (16, 3)),
                                           (61, 39_000_000, None), (64, 60_000_000, (16, 3)), (200, 400_000_000, (16, 3)), (256, 400_000_000, (8, 3))])
def test_walks_of_rows_into_blocks(K, values, walk, aligned):
    need_gpu()
    P = values // K
    pl = B.Plan([0, P], K, 0, 0, seed=0)
    got, = launches(lambda s: pl.state_copy(fake_state(pl), fake_state(pl, "rows", aligned), 7, s), args=_CopyArgs)
    pieces = -(-(P + 31) // 1024)
    run, fold = walk or (pieces, 1)
    assert (got.P, got.K, got.fold) == (P, K, fold) and got.run_len == -(-pieces // -(-pieces // run))
    pl.destroy()
