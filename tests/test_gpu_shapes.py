"""The fused kernel's shapes over the numbers of workers and the sizes of launch that choose them, against the CPU
oracle (needs an MI355X).  Both sides perform the same IEEE operations in the same order, so every float has to be
equal.  Element columns do not interact: of large states the oracle replays one element of
every stretch that is no wider than a tile, and both ends of every component."""
import numpy as np
import pytest

import oracle
from paper_1909_09010_amd import binding as B
from paper_1909_09010_amd import workloads as W
from test_launch_choice import fake_state, fused_args, tile_kinds

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def check(K, q, off, layout, mode, stride=None, every=None, rounds=(0, 1), narrow=False, stretches=False, **plan):
    """Syncs in ascending and descending order, steps if the plan has periods; `every`: one element of so many is compared, None: all;
    `narrow`: blocks as small as the plan takes; `stretches`: a sync of everything has tiles in stretches of every kind."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    off = np.asarray(off, dtype=np.int64)
    P, seed, ma = int(off[-1]), 5 + K, mode == B.MODE_GOSSIP_MA
    most = int(np.max(q))
    pl = B.Plan(off, K, q, (most + 1) // 2 if most > 2 else 0, seed=seed, **plan)
    st = W.DeviceState(K, P, DEV, layout, stride=stride, plan=pl)
    if narrow:
        size = pl.info.min_block_floats
        blocks = -(-P // size)
        st.arena = torch.empty(blocks * 3 * K * size, device=DEV)
        st.block_floats, st.worker_stride, st.block_stride, st.width = size, size, 3 * K * size, blocks * size
        st.arrays = [torch.as_strided(st.arena, (K, blocks, size), (size, 3 * K * size, 1), a * K * size) for a in range(3)]
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    for flat in [st.arena] if st.arena is not None else st.arrays:
        flat.normal_(0, 0.05, generator=g)
    cols, red = (np.arange(P, dtype=np.int64), off) if every is None else W.tile_columns(off, every, seed=K)
    idx = torch.from_numpy(cols).to(DEV)
    host = [np.ascontiguousarray(st.gather(a, idx).cpu().numpy()) for a in range(3)]
    pads = [st.padding(a).clone() for a in range(3)]
    if stretches:
        call = lambda s: pl.sync_state(st.desc(gossip_ma=ma), 0.9, 1.0, mode, 0, s)
        side_by_side, wide, narrow_kind = tile_kinds(call)
        assert side_by_side > 0 and wide > 0 and (narrow_kind > 0) == (fused_args(call).logT > 6)      # 64 tiles of 64 columns are 64 KB
    for r in rounds:
        if "periods" in plan:
            pl.sync_step_state(st.desc(gossip_ma=ma), 0.9, 1.0, mode, r, None)
        elif layout == "separate":
            pl.sync(st.arrays[0], *([None, None] if ma else st.arrays[1:]), st.worker_stride, 0.9, 1.0, mode, r, None)
        else:
            pl.sync_state(st.desc(gossip_ma=ma), 0.9, 1.0, mode, r, None)
        oracle.sync(red, K, pl.info.p, q, seed, r, host[0], *([None, None] if ma else host[1:]), np.float32(0.9),
                    np.float32(1.0), mode, active=(r % np.asarray(plan["periods"]) == 0).astype(np.uint8) if "periods" in plan else None)
    torch.cuda.synchronize()
    for a, name in enumerate(("theta", "omega", "delta")):
        assert np.array_equal(st.gather(a, idx).cpu().numpy(), host[a]), (name, pl.info.tile_columns, pl.info.threads)
        assert torch.equal(st.padding(a), pads[a]), "padding was touched"
    pl.destroy()


def stride_of(layout, P):
    return None if layout != "odd" else P | 1


# States that the caches hold.  Component edges inside tiles, on a block's edge (8192) and one float beside it; more than
# 9216 floats, so that a rotation of the XCDs would pass its first 8 groups.
@pytest.mark.parametrize("layout", ["blocked", "separate", "odd"])
@pytest.mark.parametrize("mode", [B.MODE_PAPER, B.MODE_NO_RESTART, B.MODE_GOSSIP_MA])
@pytest.mark.parametrize("K,q", [(3, 2), (5, 1), (6, 3), (9, 2), (10, 5), (13, 9), (17, 1), (19, 4), (21, 2), (22, 3), (24, 7), (25, 2), (29, 5),
                                 (30, 1), (32, 9), (33, 3), (36, 2), (44, 1), (45, 4), (56, 2), (57, 7), (60, 0), (63, 5)])
def test_small_launches(K, q, mode, layout):
    off = [0, 5, 4099, 4100, 8192, 8193, 13001, 18437]
    check(K, q, off, "separate" if layout == "odd" else layout, mode, stride_of(layout, off[-1]), rounds=(0, 1, 2))


# The sizes between: 2 to 5 M values, 5 to 20 M, and gossip-MA above that, in shapes of their own.
@pytest.mark.parametrize("layout", ["blocked", "rows", "odd"])
@pytest.mark.parametrize("values,mode", [(3_100_000, B.MODE_PAPER), (11_000_000, B.MODE_PAPER), (3_100_000, B.MODE_GOSSIP_MA),
                                         (11_000_000, B.MODE_GOSSIP_MA), (22_000_000, B.MODE_GOSSIP_MA)])
@pytest.mark.parametrize("K,q", [(1, 0), (2, 1), (4, 1), (7, 2), (8, 3), (12, 2), (16, 4), (24, 5), (32, 3), (47, 9), (64, 2), (96, 3), (128, 1), (200, 2),
                                 (300, 3), (600, 1)])
def test_launches_between(K, q, values, mode, layout):
    P = values // K
    off = [0, P // 3 | 1, P // 3 + 70 | 1, P // 3 * 2, P]
    check(K, q, off, "separate" if layout == "odd" else layout, mode, stride_of(layout, P), every=128 if K <= 128 else 16)


# Streamed accesses at sizes that take plain ones by themselves.
@pytest.mark.parametrize("layout", ["blocked", "separate", "odd"])
@pytest.mark.parametrize("K,q,mode", [(3, 2, B.MODE_PAPER), (16, 3, B.MODE_LITERAL), (24, 9, B.MODE_PAPER), (64, 5, B.MODE_GOSSIP_MA), (300, 2, B.MODE_PAPER)])
def test_cache_hints(K, q, mode, layout):
    off = [0, 5, 4099, 4100, 8192, 8193, 13001, 18437]
    check(K, q, off, layout if layout == "blocked" else "separate", mode, stride_of(layout, off[-1]), cache_hints=3)


# Just above 20 M values; 60 M of gossip-MA on rows that share lines.
@pytest.mark.parametrize("layout", ["blocked", "rows", "odd"])
@pytest.mark.parametrize("mode", [B.MODE_PAPER, B.MODE_GOSSIP_MA])
@pytest.mark.parametrize("K,q", [(1, 0), (3, 2), (5, 1), (12, 3), (16, 9), (17, 2), (25, 5), (32, 1), (33, 2), (45, 3), (63, 4), (64, 7), (65, 2),
                                 (128, 3), (129, 1), (300, 9), (512, 2), (513, 3), (1024, 2)])
def test_middle_launches(K, q, mode, layout):
    P = (64_000_000 if mode == B.MODE_GOSSIP_MA else 22_000_000) // K
    off = [0, P // 3 | 1, P // 3 + 70 | 1, P // 3 * 2, P]
    check(K, q, off, "separate" if layout == "odd" else layout, mode, stride_of(layout, P), every=128 if K <= 128 else 16)


# Beyond 500 M values other shapes, orders of the tiles and a sampler launch of their own.
@pytest.mark.parametrize("layout", ["blocked", "rows", "odd"])
@pytest.mark.parametrize("K,q,mode", [(3, 1, B.MODE_PAPER), (14, 2, B.MODE_NO_RESTART), (24, 3, B.MODE_PAPER), (40, 1, B.MODE_PAPER), (64, 5, B.MODE_PAPER),
                                      (100, 2, B.MODE_PAPER), (200, 9, B.MODE_PAPER), (300, 3, B.MODE_PAPER), (700, 2, B.MODE_PAPER),
                                      (12, 2, B.MODE_GOSSIP_MA), (48, 3, B.MODE_GOSSIP_MA), (200, 1, B.MODE_GOSSIP_MA), (700, 2, B.MODE_GOSSIP_MA)])
def test_large_launches(K, q, mode, layout):
    P = 510_000_000 // K
    off = [0, P // 5 | 1, P // 5 + 70 | 1, P // 3 * 2, P]
    check(K, q, off, "separate" if layout == "odd" else layout, mode, stride_of(layout, P), every=128 if K <= 128 else 32)


# The shapes that stream omega and Delta, in tiles that component edges cut: components of 1 to 3 floats, edges a float beside a
# block's (also of blocks narrower than a tile, whose columns are then read float by float), rows that end inside a column; one number of neighbours for
# all components or one each.
@pytest.mark.parametrize("place", ["blocked", "narrow", "rows", "odd"])
@pytest.mark.parametrize("K,values,q,mode", [
    (40, 5_600_000, [3, 0, 2, 6, 1, 4], B.MODE_PAPER), (64, 5_200_000, [2, 7, 5], B.MODE_PAPER), (48, 5_600_000, 9, B.MODE_LITERAL),
    (100, 2_200_000, [1, 4, 0, 6, 3], B.MODE_PAPER), (128, 2_300_000, 3, B.MODE_NO_RESTART), (300, 2_200_000, [1, 2], B.MODE_PAPER),
    (130, 20_400_000, [2, 0, 3], B.MODE_PAPER), (200, 20_500_000, [5, 1, 7, 4], B.MODE_PAPER), (300, 20_400_000, 3, B.MODE_PAPER),
    (300, 20_400_000, 2, B.MODE_GOSSIP_MA), (700, 21_000_000, [2, 1], B.MODE_GOSSIP_MA), (700, 64_000_000, [2, 1], B.MODE_GOSSIP_MA)])
def test_cut_tiles_of_streamed_shapes(K, values, q, mode, place):
    P = values // K // 8 * 8 + 3
    at = P // 128 * 64                                       # a multiple of the narrowest blocks
    off = [0, 1, 3, 4, 7, 61, 62, 126, 130, 8191, 8194, 8195, 12289, at + 62, at + 127, at + 193, at + 1021, P - 6, P - 5, P - 2, P]
    off = sorted(x for x in off if x <= P)
    q = q if np.ndim(q) == 0 else [q[i % len(q)] for i in range(len(off) - 1)]
    layout = {"narrow": "blocked", "odd": "separate"}.get(place, place)
    check(K, q, off, layout, mode, P | 1 if place == "odd" else None, narrow=place == "narrow")


# Aligned rows, whose whole tiles are dealt in stretches 32 KB apart: 64 tiles of T columns (256 * T floats) at a time, then 64 KB (16384 floats) at a
# time.  Components around both sizes, that begin on a tile, a float after and beside one, and a long one.
def stretched(K, q, values, mode, **plan):
    P, most = values // K, int(np.max(q))
    pl = B.Plan([0, P], K, most, (most + 1) // 2 if most > 2 else 0, **plan)
    T = 1 << fused_args(lambda s: pl.sync_state(fake_state(pl, "rows"), 0.9, 1.0, mode, 0, s)).logT
    pl.destroy()
    wide, narrow, tile = 256 * T, 16384, 4 * T
    off, at = [0, 5], 5
    for n in (narrow - 1, narrow + tile, wide, wide + narrow + tile + 3, -1, wide, narrow - tile, -1, 1, wide + tile, 2 * wide - 1):
        at = at + n if n > 0 else -(-at // tile) * tile       # -1: the next begins on a tile
        off.append(at)
    return sorted({x for x in off if x < P} | {P})


# Rows that begin on 4 KB and on a line; in both walks every float.  More than 7 neighbours have a sampler launch, or tiles would be too narrow.
@pytest.mark.parametrize("place", ["rows", "lines"])
@pytest.mark.parametrize("values,mode,K,q", [
    (values, mode, K, q) for values, mode, most in ((5_300_000, B.MODE_PAPER, 16), (20_500_000, B.MODE_PAPER, 128), (5_300_000, B.MODE_GOSSIP_MA, 8),
                                                    (20_500_000, B.MODE_GOSSIP_MA, 128))
    for K, q in ((1, 0), (2, 1), (3, 2), (4, 1), (5, 2), (8, 3), (12, 5), (16, 4), (24, 9), (32, 2), (33, 3), (48, 8), (64, 5), (100, 1), (128, 3),
                 (2, [1, 0]), (4, [2, 3]), (8, [3, 1]), (12, [6, 7, 1]), (16, [3, 2, 1, 0]), (32, [5, 2, 7]), (48, [4, 1, 6]), (100, [1, 3]))
    if K <= most and not (values < 6_000_000 and mode == B.MODE_PAPER and 5 <= K <= 8) and not (values > 6_000_000 and mode == B.MODE_GOSSIP_MA and (K == 3 or (np.max(q) > 4 and K in (24, 48, 64))))])
def test_tiles_in_stretches(values, mode, K, q, place):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    P = values // K
    plan = {"sampling": B.SAMPLING_SEPARATE} if int(np.max(q)) > 7 else {}
    off = stretched(K, q, values, mode, **plan)
    q = q if np.ndim(q) == 0 else [q[i % len(q)] for i in range(len(off) - 1)]
    check(K, q, off, "separate" if place == "lines" else place, mode, -(-P // 32) * 32 + 32 if place == "lines" else None, stretches=True, **plan)


# Under sync periods: what is due is not one run of components (odd steps), or the first or second half; every third step all.
@pytest.mark.parametrize("mode", [B.MODE_PAPER, B.MODE_GOSSIP_MA])
@pytest.mark.parametrize("due", ["others", "first", "second"])
@pytest.mark.parametrize("K,q", [(2, 1), (4, [1, 2]), (8, 2), (16, [3, 1]), (32, 4), (64, 2), (100, 3)])
def test_steps_of_tiles_in_stretches(K, q, due, mode):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    off = np.asarray(stretched(K, q, 21_000_000, mode))
    off = [*off, *(off[1:] + off[-1])]                       # the same twice: either half is enough for stretches
    m = len(off) - 1
    periods = [1 + 2 * {"others": i % 2, "first": int(i >= m // 2), "second": int(i < m // 2)}[due] for i in range(m)]
    check(K, q if np.ndim(q) == 0 else [q[i % len(q)] for i in range(m)], off, "rows", mode, rounds=(1, 2, 3), stretches=True, periods=periods)


# Every number of neighbours that a workgroup of a plan of several takes a path of its own for, in tiles that are whole, cut and thin.
@pytest.mark.parametrize("layout", ["blocked", "rows", "odd"])
@pytest.mark.parametrize("mode", [B.MODE_PAPER, B.MODE_GOSSIP_MA])
@pytest.mark.parametrize("K,values", [(8, 200_000), (9, 5_300_000), (16, 200_000), (24, 20_400_000), (40, 20_400_000), (100, 5_300_000)])
def test_every_number_of_neighbours(K, values, mode, layout):
    P = values // K
    off = sorted({0, 2, P // 8 | 1, P // 7 & ~3, P // 6 | 3, P // 5, P // 4 | 1, P // 3, P // 2 | 1, P - 1, P})
    q = [(3 * i + 5) % 8 for i in range(len(off) - 1)]
    check(K, q, off, "separate" if layout == "odd" else layout, mode, stride_of(layout, P), every=64)


# Gossip-MA of blocks that draws 5 to 7 neighbours in the kernel: before theta's loads where these fill all four slots of a thread (32, 49 and 64 workers), else behind them.
@pytest.mark.parametrize("sampling", [B.SAMPLING_AUTO, B.SAMPLING_SEPARATE])
@pytest.mark.parametrize("K,q", [(24, 6), (25, 5), (32, 6), (32, [5, 2, 7]), (48, 7), (49, 5), (64, 6), (64, [7, 1]), (100, 5)])
def test_drawing_before_and_behind_the_loads(K, q, sampling):
    P = 22_000_000 // K
    off = [0, P // 3 | 1, P // 3 + 70 | 1, P // 3 * 2, P]
    check(K, q if np.ndim(q) == 0 else [q[i % len(q)] for i in range(4)], off, "blocked", B.MODE_GOSSIP_MA, every=128, sampling=sampling)
