"""Calls that differ in what should cost nothing, timed against each other on one MI355X: within a call
family the time may not depend on odd sizes.  Passes are replayed from a HIP graph, so that the host's
launch time is not in them; the bounds are far from the noise (a few per cent) and from what a fault cost."""
import pytest

from paper_1909_09010_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def us(call, calls=20, replays=7):
    """Microseconds of one ``call(round)`` among others, the best of several replays."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    call(0, None)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for r in range(calls):
            call(r, torch.cuda.current_stream())
    best = float("inf")
    for _ in range(replays):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        graph.replay()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / calls)
    return best


def rows(K, stride):
    return [torch.randn(K * stride, device=DEV) * 0.05 for _ in range(3)]


def sync_us(off, K, q, stride, p=0, mode=B.MODE_PAPER, **plan):
    pl = B.Plan(off, K, q, p, seed=1, **plan)
    st = rows(K, stride)
    return us(lambda r, s: pl.sync(*(st if mode != B.MODE_GOSSIP_MA else [st[0], None, None]), stride, 0.9, 1.0, mode, r, s))


# The same tiles, with the component edges between 16-byte columns or inside one: a column that is cut issues all its
# loads at once like a whole one.  Measured 1.19 to 1.31; 1.5 to 1.7 where each waits for the one before.
@pytest.mark.parametrize("K", [16, 100, 200])
def test_columns_cut_by_a_component_edge_wait_for_nothing(K):
    T = 4 * 16
    edges = lambda shift: sync_us([0] + [T * i - shift for i in range(1, 48)] + [48 * T], K, 2, 48 * T, tile=(1024, 4))
    between, inside = edges(4), edges(2)
    assert inside < 1.45 * between, (inside, between)


# Averaging 9 neighbours instead of 7 may cost a little, preparing their rows may not: measured 0.98 to 1.21, and 1.36 to
# 1.99 where a thread sorts each row.
@pytest.mark.parametrize("K,mode", [(10, B.MODE_PAPER), (16, B.MODE_PAPER), (10, B.MODE_GOSSIP_MA), (24, B.MODE_GOSSIP_MA)])
def test_more_neighbours_than_fit_registers(K, mode):
    P = 60_000_000 // K // 1024 * 1024
    seven, nine = (sync_us([0, P], K, q, P, p=5, mode=mode, sampling=B.SAMPLING_SEPARATE) for q in (7, 9))
    assert nine < 1.32 * seven, (nine, seven)


# The last P % 4 elements of a final average are read by threads of their own, with as many rows in flight as a column of
# 4: measured 1.0 to 1.1, and 9 where one thread reads them one after the other.
@pytest.mark.parametrize("rest", [1, 3])
def test_the_last_elements_of_an_average_wait_for_nothing(rest):
    K, P = 1024, 4000
    st, out = torch.randn(K * (P + 4), device=DEV), torch.empty(P + 4, device=DEV)
    plans = {n: B.Plan([0, P + n], K, 0, 0, seed=0) for n in (0, rest)}
    whole, cut = (us(lambda r, s: plans[n].final_average(st, P + 4, out, s)) for n in (0, rest))
    assert cut < 1.6 * whole, (cut, whole)


# Rows are copied as fast from many workers' rows as from few: measured 0.93 to 1.01, and 1.13 to 1.25 in short runs of
# one worker after the other.
@pytest.mark.parametrize("K", [64, 200, 512])
def test_rows_of_many_workers_are_copied_like_those_of_one(K):
    n = 300_000_000 // K // 1024 * 1024
    a, b = torch.randn(K * n, device=DEV), torch.empty(K * n, device=DEV)
    plans = {k: B.Plan([0, K * n // k], k, 0, 0, seed=0) for k in (1, K)}
    state = lambda t, k: B.make_state(t, None, None, K * n // k)
    one, many = (us(lambda r, s: plans[k].state_copy(state(b, k), state(a, k), 1, s), calls=5) for k in (1, K))
    assert many < 1.1 * one, (many, one)


# A single worker's stride is no distance between rows: odd or padded, the same tiles go to the same XCDs.  Both run on the
# same buffers, in turn; where an odd stride counted as rows that share cache lines it took 8 % longer.
def test_the_stride_of_a_single_worker_does_not_matter():
    P = 150_000_000
    pl, st = B.Plan([0, P], 1, 0, 0, seed=1), rows(1, P + 1024)
    padded, odd = (min(us(lambda r, s: pl.sync(*st, stride, 0.9, 1.0, B.MODE_PAPER, r, s)) for _ in range(2))
                   for stride in (P + 1024 - P % 1024, P + 3))
    assert odd < 1.05 * padded, (odd, padded)
