"""The fused kernel's work list at its edges, against the CPU oracle (needs an MI355X): numbers of
tiles around the groups in which consecutive tiles go to one XCD, forwards and backwards, on rows
that start anywhere.  Both sides perform the same IEEE operations in the same order, so every float
has to be equal, and floats outside the parameters keep their junk."""
import numpy as np
import pytest

import oracle
from paper_1909_09010_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def check_rows(K, q, off, stride, skew=(0, 0, 0), mode=B.MODE_PAPER, rounds=(0, 1), seed=3, **plan):
    """Syncs on three [K, stride] tensors whose bases are `skew` floats into their allocations."""
    off = np.asarray(off, dtype=np.int64)
    P = int(off[-1])
    pl = B.Plan(off, K, q, 0, seed=seed, **plan)
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    flat = [torch.randn(K * stride + s + 3, generator=g, device=DEV) * 0.05 for s in skew]
    dev = [f[s:s + K * stride].view(K, stride) for f, s in zip(flat, skew)]
    before = [f.clone() for f in flat]
    host = [d.cpu().numpy().copy() for d in dev]
    assert [d.data_ptr() % 16 for d in dev] == [4 * s % 16 for s in skew]
    for r in rounds:
        if mode == B.MODE_GOSSIP_MA:
            pl.sync(dev[0], None, None, stride, 0.9, 1.0, mode, r, None)
        else:
            pl.sync(*dev, stride, 0.9, 1.0, mode, r, None)
        oracle.sync(off, K, pl.info.p, q, seed, r, *host, np.float32(0.9), np.float32(1.0), mode)
    torch.cuda.synchronize()
    for f, d, h, s, b in zip(flat, dev, host, skew, before):
        assert np.array_equal(d.cpu().numpy(), h)                       # padding included: the oracle leaves it too
        assert torch.equal(f[:s], b[:s]) and torch.equal(f[s + K * stride:], b[s + K * stride:])
    info = pl.info
    pl.destroy()
    return info


# Consecutive tiles that one XCD takes: 2048 columns of a row where rows share cache lines, halved until the list has 4 groups of 8
# such runs, else one tile.  The lists here end before, at and after one and two groups of 2048 columns at the plan's own tile width.
@pytest.mark.parametrize("K", [4, 7, 16, 33])
@pytest.mark.parametrize("tiles", ["1", "9", "group-1", "group", "group+1", "2*group-1", "2*group+3"])
@pytest.mark.parametrize("odd", [0, 1])
def test_every_tile_is_taken_once_around_the_xcd_groups(K, tiles, odd):
    _need_gpu()
    mode = B.MODE_GOSSIP_MA if tiles == "2*group-1" else B.MODE_PAPER
    pl = B.Plan([0, 1 << 15], K, 1, 0, seed=0)               # small, as the plans below are: the same width
    columns = pl.info.tile_columns_blocked_ma if mode == B.MODE_GOSSIP_MA else pl.info.tile_columns
    pl.destroy()
    n = eval(tiles, {"group": 8 * max(1, 2048 // columns) if odd else 8})
    P = n * 4 * columns - (5 if odd else 0)
    assert K * P < 20_000_000
    stride = P + 3 if odd else -(-P // 1024) * 1024
    info = check_rows(K, 1, [0, P // 3, P], stride, (1, 0, 3) if odd else (0, 0, 0), mode=mode)
    assert mode == B.MODE_GOSSIP_MA or info.n_tiles in (n, n + 1)         # the component edge cuts one tile


# one piece is 256 columns of 4 floats; the destination's first column starts up to 31 floats before the row; above 4 M
# floats an array is copied in runs of 1, 8 or 32 pieces or whole rows, by kind, workers and size, into a blocked one all arrays together
@pytest.mark.parametrize("K,P", [(K, P) for K in (1, 3, 16, 33, 64) for P in (1, 3, 1023, 1024, 1057, 32 * 1024 - 1, 32 * 1024 + 5,
                                                                              3 * 32 * 1024 + 1021)] + [
    (1, 30_000_001), (3, 10_012_677), (16, 1_900_545), (17, 1_773_529), (32, 950_273), (33, 917_509), (64, 470_017),
    (128, 262_149), (1024, 33_797), (1, 4_000_001), (3, 1_400_001), (16, 250_007), (17, 240_001), (32, 125_003), (33, 125_001),
    (48, 91_001), (49, 90_003), (33, 1_230_001), (300, 136_003)])
@pytest.mark.parametrize("which", [7, 2, 5])
def test_state_copy_at_the_edges_of_its_pieces(K, P, which):
    _need_gpu()
    pl = B.Plan([0, P], K, 0, 0, seed=0)
    Bf = pl.info.min_block_floats * (1 if P < 40000 else 4)
    blocks = -(-P // Bf)
    ws, gap = Bf + (5 if K == 3 else 0), 7                   # K = 3: odd strides, so that columns cross no alignment
    bs = 3 * K * ws + gap
    g = torch.Generator(device=DEV)
    g.manual_seed(P)
    stride = P + 1
    rows = [torch.randn(K * stride + 9, generator=g, device=DEV) for _ in range(3)]
    skew = (0, 1, 6)
    arena = torch.full((blocks * bs + 64,), 7.0, device=DEV)
    want = arena.clone()
    blocked = B.make_state(*[arena.data_ptr() + 4 * (a * K * ws + 3) for a in range(3)], ws, Bf, bs)
    idx = torch.arange(P, device=DEV)
    at = (idx // Bf) * bs + idx % Bf
    for a in range(3):
        if which >> a & 1:
            for w in range(K):
                want[3 + a * K * ws + w * ws + at] = rows[a][skew[a] + w * stride:][:P]
    pl.state_copy(blocked, B.make_state(*[r.data_ptr() + 4 * s for r, s in zip(rows, skew)], stride), which, None)
    torch.cuda.synchronize()
    assert torch.equal(arena, want)
    back = [torch.full_like(r, 5.0) for r in rows]
    pl.state_copy(B.make_state(*[b.data_ptr() + 4 * s for b, s in zip(back, skew[::-1])], stride), blocked, which, None)
    torch.cuda.synchronize()
    for a in range(3):
        expect = torch.full_like(rows[a], 5.0)
        if which >> a & 1:
            for w in range(K):
                expect[skew[2 - a] + w * stride:][:P] = rows[a][skew[a] + w * stride:][:P]
        assert torch.equal(back[a], expect)
    pl.destroy()


# The kernel for many workers: 64 < K <= 128 with 4096 slots, above with 8192; component edges inside and at the
# ends of a tile, blocks as narrow as they may be (narrower than its tile), caller's tables, all modes.
@pytest.mark.parametrize("K,q", [(65, 2), (90, 5), (128, 7), (129, 4), (200, 1), (256, 3), (257, 0), (600, 9), (1024, 2)])
@pytest.mark.parametrize("mode", [0, 1, 2, 3])
def test_many_workers(K, q, mode):
    _need_gpu()
    off = [0, 1, 130, 130, 1029, 1030, 2048, 2300]
    P = off[-1]
    check_rows(K, q, off, P + 1, (1, 2, 0), mode=mode, seed=K)
    check_rows(K, q, off, 2304, mode=mode, seed=K)
    pl = B.Plan(off, K, q, 0, seed=K)
    assert mode != 1 or K <= 64 or pl.info.min_block_floats <= 4 * pl.info.tile_columns_blocked
    Bf = pl.info.min_block_floats
    blocks = -(-P // Bf)
    g = torch.Generator(device=DEV)
    g.manual_seed(K)
    arena = torch.randn(blocks * 3 * K * Bf, generator=g, device=DEV) * 0.05
    view = arena.view(blocks, 3, K, Bf)
    host = [view[:, a].permute(1, 0, 2).reshape(K, -1).cpu().numpy().copy() for a in range(3)]
    state = B.make_state(*[None if a and mode == 3 else arena.data_ptr() + 4 * a * K * Bf for a in range(3)], Bf, Bf, 3 * K * Bf)
    table = torch.zeros((len(off) - 1, K, max(q, 1)), dtype=torch.int32, device=DEV)
    for r in (0, 1):
        if r and q:
            pl.neighbours_device(r, table, None)
            pl.sync_table_state(table.flip(-1).contiguous(), state, 0.9, 1.0, mode, None)
        else:
            pl.sync_state(state, 0.9, 1.0, mode, r, None)
        oracle.sync(np.asarray(off, dtype=np.int64), K, pl.info.p, q, K, r, *host, np.float32(0.9), np.float32(1.0), mode)
    torch.cuda.synchronize()
    for a in range(3):
        assert np.array_equal(view[:, a].permute(1, 0, 2).reshape(K, -1).cpu().numpy(), host[a])
    pl.destroy()


def check_average(K, P):
    """Rows of an odd stride that start inside a line, and blocks; sums to an address that is and one that is not a multiple of 16."""
    _need_gpu()
    pl = B.Plan([0, P], K, 0, 0, seed=0)
    g = torch.Generator(device=DEV)
    g.manual_seed(P)
    stride = P + (1 if P % 2 == 0 else 2)
    flat = torch.randn(K * stride + 3, generator=g, device=DEV)
    rows = flat[3:].view(K, stride)
    want = oracle.final_average(rows.cpu().numpy(), P)
    out = torch.full((P + 8,), 7.0, device=DEV)
    pl.final_average(rows, stride, out[1:], None)
    Bf = 2 * pl.info.min_block_floats
    blocks = -(-P // Bf)
    arena = torch.full((blocks, K, Bf), float("nan"), device=DEV)
    arena.permute(1, 0, 2).copy_(torch.nn.functional.pad(rows[:, :P], (0, blocks * Bf - P)).view(K, blocks, Bf))
    out2 = torch.full((P + 8,), 7.0, device=DEV)
    pl.final_average_state(B.make_state(arena, None, None, Bf, Bf, K * Bf), out2[4:], None)
    torch.cuda.synchronize()
    assert np.array_equal(out[1:1 + P].cpu().numpy(), want) and np.array_equal(out2[4:4 + P].cpu().numpy(), want)
    assert bool((out[1 + P:] == 7).all()) and bool((out2[4 + P:] == 7).all()) and float(out[0]) == 7
    pl.destroy()


# one workgroup is 64 columns of 4 floats; groups of 8 or 32 workgroups are dealt to the XCDs, the last P % 4 floats go to
# one thread each; rows are read 4, 8 or 16 at a time, the last ones in halves of that
@pytest.mark.parametrize("K", [1, 2, 3, 4, 5, 6, 8, 9, 11, 14, 16, 17, 18, 21, 25, 32, 33, 35, 41, 64, 130])
@pytest.mark.parametrize("P", [1, 4, 255, 256, 2048 * 4 + 3, 4 * 64 * 33 - 1, 262146])
def test_final_average_at_its_edges(K, P):
    check_average(K, P)


# sums beyond the caches are streamed, from 60 M values on with the resident waves bounded; rows too short for that; blocked
# state of more than 500 M values of 33 to 64 workers moves on by an XCD from block to block
@pytest.mark.parametrize("K,P", [(1, 61_000_001), (2, 31_000_002), (3, 21_000_003), (5, 13_000_001), (8, 5_000_003), (11, 6_000_002), (16, 4_000_001),
                                 (20, 2_000_001), (33, 1_300_001), (48, 1_500_003), (70, 1_000_002), (130, 300_001), (130, 500_003), (300, 130_001),
                                 (300, 210_003), (300, 510_001), (1000, 70_002), (40, 13_000_003)])
def test_final_averages_beyond_the_caches(K, P):
    check_average(K, P)


# Rows drawn in registers (up to 7 neighbours, at the largest degree the ring wraps) and from a table, one number of
# neighbours for all components and one each: the same bits as the host's and the oracle's draws.
@pytest.mark.parametrize("K,p,q", [(2, 0, 1), (4, -1, 3), (5, 2, 4), (8, -1, 7), (9, -1, 8), (16, 0, [0, 1, 2, 3, 4, 5, 6]), (12, 5, [4, 2]),
                                   (40, 6, [7, 0, 7]), (300, -1, 7), (300, 4, [8, 1])])
@pytest.mark.parametrize("sampling", [B.SAMPLING_AUTO, B.SAMPLING_SEPARATE])
def test_draws_in_registers(K, p, q, sampling):
    _need_gpu()
    m = 7 if np.ndim(q) == 0 else len(q)
    off = np.concatenate([[0], np.cumsum([1000 + 37 * i for i in range(m)])]).astype(np.int64)
    P, seed = int(off[-1]), 2**63 + 11
    pl = B.Plan(off, K, q, p, seed=seed, sampling=sampling)
    g = torch.Generator(device=DEV)
    g.manual_seed(K)
    dev = [torch.randn((K, P), generator=g, device=DEV) * 0.05 for _ in range(3)]
    host = [d.cpu().numpy().copy() for d in dev]
    out = torch.zeros((m, K, pl.info.q), dtype=torch.int32, device=DEV)
    for rnd in (0, 1, 2**33 + 7):
        pl.sync(*dev, P, 0.9, 1.0, 1, rnd, None)
        oracle.sync(off, K, pl.info.p, q, seed, rnd, *host, np.float32(0.9), np.float32(1.0), 1)
        pl.neighbours_device(rnd, out, None)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), pl.neighbours_host(rnd))
    for d, h in zip(dev, host):
        assert np.array_equal(d.cpu().numpy(), h)
    pl.destroy()
