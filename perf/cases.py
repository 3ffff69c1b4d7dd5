"""The framework's work as its users have it done, case by case: the synchronisation of K worker
replicas between two stretches of local training, and the calls around it (sync under per-component
periods, plain gossip averaging, the final model average, moving a state between placements).

Parameter sets are LSTM language models as in ``paper_1909_09010_amd.workloads`` (embedding, LSTM
layers, softmax) or the paper's own model; a case says how many workers there are, how many
neighbours a worker draws, how large the model is, how it is cut into components and where the
state lives:

  blocked   the one arena that the library recommends
  plain     three ordinary ``[K, P]`` tensors: rows follow each other without padding, so that for
            most parameter counts they are not 16-byte aligned
  padded    three ``[K, stride]`` tensors with the row length rounded up to 1024 floats

Keys of a case: entry (sync, step, final, move_in, move_out), place, kind ("lstm_lm" or "paper"),
K, q (0 = the paper-shaped mix of 3, 2 and 1 per component), p (0 = the paper's rule), vocab,
width (embedding and hidden size), layers, chunk (rows per component, 0 = whole tensors), mode
(the update rule: 0 classical, 1 as printed, 2 literal, 3 gossip averaging only).
"""
import dataclasses
import math

import numpy as np
import torch

from paper_1909_09010_amd import binding, workloads

DEVICE = "cuda:0"
MOST_WORKER_PARAMS = 2_500_000_000     # of a drawn case: below the largest listed one (4.5e9)
MOST_EXACT = 700_000_000               # worker-params that the 64-bit check takes in seconds


def _case(name, entry, place, K, q, vocab, width, layers=2, chunk=0, mode=1, kind="lstm_lm", p=0):
    c = {"entry": entry, "place": place, "kind": kind, "K": K, "q": q, "p": p, "vocab": vocab, "width": width,
         "layers": layers, "chunk": chunk, "mode": mode}
    return {"name": name, **c} if name else c


def listed():
    return [
        # A small model on four workers, synced every few mini-batches: nothing but latency.
        _case("sync_tiny", "sync", "blocked", 4, 1, 3001, 64),
        # A dozen workers (not a power of two) with a 2.7M-parameter model: between latency and bandwidth.
        _case("sync_small_k12", "sync", "blocked", 12, 2, 5003, 200),
        # The medium language model (10k words, width 650) on the paper's 8-worker setting.
        _case("sync_medium", "sync", "blocked", 8, 2, 10000, 650),
        # The large-vocabulary model cut into 256-row chunks on 16 workers: 53 GB of state, the largest.
        _case("sync_large_vocab", "sync", "blocked", 16, 3, 267735, 512, chunk=256),
        # 64 workers, width 1024, 1024-row chunks (the headline configuration with a 20k vocabulary).
        _case("sync_k64", "sync", "blocked", 64, 4, 20000, 1024, chunk=1024),
        # A whole fleet of small replicas.
        _case("sync_k256", "sync", "blocked", 256, 4, 10007, 256),
        # A trainer that keeps three ordinary [K, P] tensors and an odd parameter count.
        _case("sync_plain", "sync", "plain", 16, 3, 30003, 512),
        # The same trainer with padded rows and 32 workers.
        _case("sync_padded_k32", "sync", "padded", 32, 2, 30000, 650),
        # The paper's model and schedule: 16 groups, periods (16, 128), a q for each kind of group; the
        # pass is one of the seven syncs out of eight in which the embedding shards are not due.
        _case("step_paper", "step", "blocked", 16, 0, 267735, 512, layers=1, kind="paper", p=3),
        # Plain gossip averaging (no momentum slots are read or written).
        _case("gossip_ma", "sync", "blocked", 16, 2, 50000, 1024, chunk=1024, mode=3),
        # The model that is returned at the end of training.
        _case("final_average", "final", "blocked", 64, 4, 20000, 1024, chunk=1024),
        # A trainer's plain tensors moved into the recommended arena before a series of syncs.
        _case("move_in", "move_in", "plain", 16, 3, 30003, 512),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    entry = rng.choice(["sync"] * 8 + ["step"] * 2 + ["final"] * 2 + ["move_in", "move_out"])
    K = rng.choice([4, 8, 16, 32, 64, int(_log(rng, 2, 300)), int(_log(rng, 2, 100)), int(_log(rng, 2, 100))])
    most_q = min(2 * max(1, int(math.log2(K)) - 1), K - 1)
    q = rng.randint(1, max(1, min(most_q, 6)))
    place = rng.choice(["blocked", "blocked", "plain", "padded"])
    mode = 1 if entry != "sync" else rng.choice([1, 1, 1, 0, 2, 3])
    while True:
        vocab, width, layers = int(_log(rng, 600, 270000)), int(_log(rng, 40, 1100)), rng.randint(1, 4)
        if rng.random() < 0.4:
            width = max(32, width // 32 * 32)
        chunk = rng.choice([0, 0, 256, 1024])
        c = _case("", entry, place, K, q, vocab, width, layers, chunk, mode)
        if 700_000 <= K * _offsets(c)[-1] <= MOST_WORKER_PARAMS:
            return c


def _workload(c):
    base = workloads.WORKLOADS["paper_shaped" if c["kind"] == "paper" else "large_vocab"]
    if c["kind"] == "paper":
        return dataclasses.replace(base, K=c["K"], p=c["p"])
    return dataclasses.replace(base, name="case", K=c["K"], q=c["q"], p=c["p"], vocab=c["vocab"], embed=c["width"],
                               hidden=c["width"], layers=c["layers"], chunk_rows=c["chunk"] or None, eta=0.9,
                               w0_scale=0.02, drift_std=0.01, delta_std=1e-4)


def _offsets(c):
    return workloads.component_offsets(_workload(c))


def _q(c):
    """Neighbours per component: one number, or the paper-shaped mix (embedding shards 3, LSTM groups and head 2, tails 1)."""
    return c["q"] if c["q"] else [3] * 8 + [2] * 3 + [1] * 5


def _periods(c):
    """Embedding and softmax every 128 mini-batches, the rest every 16."""
    if c["entry"] != "step":
        return None
    w = _workload(c)
    if c["kind"] == "paper":
        return workloads.periods(w)
    off = workloads.component_offsets(w)
    ends = np.cumsum([rows * cols for _, rows, cols in workloads.tensors(w)])
    first, last = ends[0], ends[-3]                       # the embedding ends here, the softmax begins here
    return np.where((off[1:] <= first) | (off[:-1] >= last), 128, 16).astype(np.int32)


def _due(c):
    """Which components a pass of this case updates."""
    h = _periods(c)
    return np.ones(len(_offsets(c)) - 1, bool) if h is None else h == 16


def prepare(case, seed):
    w = _workload(case)
    off = workloads.component_offsets(w)
    P, K = int(off[-1]), case["K"]
    plan = binding.Plan(off, K, _q(case), w.p, seed=seed, periods=_periods(case))
    layout, stride = ("blocked", None) if case["place"] == "blocked" else ("separate", P if case["place"] == "plain" else None)
    st = workloads.init_state(w, DEVICE, layout=layout, stride=stride, seed=seed, plan=plan)
    s = {"entry": case["entry"], "place": case["place"], "mode": case["mode"], "plan": plan, "st": st, "eta": w.eta,
         "zeta": w.zeta, "round": 0, "desc": st.desc(case["mode"] == binding.MODE_GOSSIP_MA),
         "stream": torch.cuda.current_stream()}
    if case["entry"] == "final":
        s["out"] = torch.zeros(P, device=DEVICE)
        st.arrays[1:] = []                                # the slots are not needed any more
    elif case["entry"] in ("move_in", "move_out"):
        # the other side: the arena that the library recommends, or three plain tensors
        kind = ("separate", P) if layout == "blocked" else ("blocked", None)
        s["to"] = workloads.DeviceState(K, P, DEVICE, kind[0], stride=kind[1], plan=plan)
        s["to"].zero_()
        if case["entry"] == "move_out" and layout != "blocked":      # out of the arena into these tensors' placement
            s["to"], s["st"] = st, s["to"]
            for a in range(3):
                for k in range(K):
                    s["st"].set_row(a, k, st.get_row(a, k))
            st.zero_()
        s["src"], s["dst"] = s["st"].desc(), s["to"].desc()
    return s


def run(s):
    plan, st = s["plan"], s["st"]
    if s["entry"] == "sync":
        rnd = s["round"]
        s["round"] = rnd + 1
        if s["place"] == "blocked":
            plan.sync_state(s["desc"], s["eta"], s["zeta"], s["mode"], rnd, s["stream"])
        elif s["mode"] == binding.MODE_GOSSIP_MA:
            plan.sync(st.arrays[0], None, None, st.worker_stride, s["eta"], s["zeta"], s["mode"], rnd, s["stream"])
        else:
            plan.sync(*st.arrays, st.worker_stride, s["eta"], s["zeta"], s["mode"], rnd, s["stream"])
        return st.arrays[0] if s["mode"] == binding.MODE_GOSSIP_MA else tuple(st.arrays)
    if s["entry"] == "step":
        rnd = s["round"]
        s["round"] = rnd + 1
        step = 16 * (rnd // 7 * 8 + rnd % 7 + 1)          # the mini-batches at which only the frequent groups are due
        if s["place"] == "blocked":
            plan.sync_step_state(s["desc"], s["eta"], s["zeta"], s["mode"], step, s["stream"])
        else:
            plan.sync_step(*st.arrays, st.worker_stride, s["eta"], s["zeta"], s["mode"], step, s["stream"])
        return tuple(st.arrays)
    if s["entry"] == "final":
        if s["place"] == "blocked":
            plan.final_average_state(s["desc"], s["out"], s["stream"])
        else:
            plan.final_average(st.arrays[0], st.worker_stride, s["out"], s["stream"])
        return s["out"]
    plan.state_copy(s["dst"], s["src"], 7, s["stream"])
    return tuple(s["to"].arrays)


def work(case):
    off, K = _offsets(case), case["K"]
    P = int(off[-1])
    if case["entry"] == "final":
        return {"bytes": 4 * (K + 1) * P, "flops": K * P}
    if case["entry"] in ("move_in", "move_out"):
        return {"bytes": 24 * K * P, "flops": 0}
    sizes, due = np.diff(off), _due(case)
    q = np.broadcast_to(np.asarray(_q(case)), sizes.shape)
    synced = int(sizes[due].sum())
    per = 1 if case["mode"] == binding.MODE_GOSSIP_MA else 8
    flops = K * int((sizes * (q + per))[due].sum())
    return {"bytes": (8 if case["mode"] == binding.MODE_GOSSIP_MA else 24) * K * synced, "flops": flops}


def tolerance(case):
    if case["entry"] in ("move_in", "move_out"):
        return "exact"
    if case["entry"] == "final":
        return {"rel": 3e-7}
    # The momentum slot is a difference of averages that nearly cancel: it is up to 4e-7 from 64 bits
    # (replicas and global model: 1e-7).
    return {"rel": 1.6e-6}


# ---------------------------------------------------------------------------------------------
# The same passes in 64 bits.
# ---------------------------------------------------------------------------------------------
def _philox(ctr, key):
    """Philox-4x32-10 on arrays: four counter words, two key words."""
    c = [np.asarray(x, dtype=np.uint64) for x in ctr]
    k0, k1 = int(key[0]), int(key[1])
    low = np.uint64(0xFFFFFFFF)
    for _ in range(10):
        a, b = c[0] * np.uint64(0xD2511F53), c[2] * np.uint64(0xCD9E8D57)
        c = [(b >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), b & low, (a >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), a & low]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def _candidates(K, p):
    """Ring candidates of every worker: p to the left, p to the right, the worker and repeats dropped."""
    rows = []
    for w in range(K):
        row = []
        for v in [(w - d) % K for d in range(1, p + 1)] + [(w + d) % K for d in range(1, p + 1)]:
            if v != w and v not in row:
                row.append(v)
        rows.append(row)
    return np.asarray(rows, dtype=np.int64).reshape(K, -1)


def _table(m, K, p, q, seed, rnd):
    """Neighbours [m][K][q] that every (component, worker) draws in sync number `rnd`."""
    p = min(p if p else max(1, int(math.floor(math.log2(K))) - 1), K - 1)
    cand = _candidates(K, p)
    C = cand.shape[1]
    pool = np.broadcast_to(cand, (m, K, C)).copy()
    comp, worker = np.meshgrid(np.arange(m), np.arange(K), indexing="ij")
    full = np.zeros((m, K), np.uint64)
    for j in range(q):
        if j % 4 == 0:
            words = _philox((full + np.uint64(rnd & 0xFFFFFFFF), full + np.uint64(rnd >> 32), comp, worker + 65536 * (j // 4)),
                            (seed & 0xFFFFFFFF, seed >> 32))
        r = (j + ((words[j % 4] * np.uint64(C - j)) >> np.uint64(32)).astype(np.int64))[..., None]
        a, b = pool[..., j:j + 1].copy(), np.take_along_axis(pool, r, -1)
        np.put_along_axis(pool, r, a, -1)
        pool[..., j:j + 1] = b
    return pool[..., :q]


def _laid_out(rows, st, which):
    """[K, P] values in 64 bits, shaped like the state's array `which` (zeros where padding is)."""
    K, P = rows.shape
    full = torch.zeros((K, st.width), dtype=torch.float64, device=rows.device)
    full[:, :P] = rows
    return full.reshape(st.arrays[which].shape)


def exact(case, seed):
    off, K = _offsets(case), case["K"]
    P = int(off[-1])
    if K * P > MOST_EXACT:
        return None
    s = prepare(case, seed)
    st = s["st"]
    rows = [torch.stack([st.get_row(a, k) for k in range(K)]).double() for a in range(len(st.arrays))]
    if case["entry"] == "final":
        return rows[0].sum(0) / K
    if case["entry"] in ("move_in", "move_out"):
        return tuple(_laid_out(r, s["to"], a) for a, r in enumerate(rows))
    eta, zeta = float(np.float32(s["eta"])), float(np.float32(s["zeta"]))
    step = 16 if case["entry"] == "step" else 0
    qs, due = np.broadcast_to(np.asarray(_q(case)), len(off) - 1), _due(case)
    tables = {int(q): torch.from_numpy(_table(len(off) - 1, K, case["p"], int(q), seed, step)).to(DEVICE) for q in set(qs.tolist())}
    th, om, de = rows
    for i in range(len(off) - 1):
        a, b = int(off[i]), int(off[i + 1])
        if not due[i] or a == b:
            continue
        x, o, d = th[:, a:b], om[:, a:b], de[:, a:b]
        q = int(qs[i])
        avg = x.clone()
        for j in range(q):
            avg += x[tables[q][i, :, j]]
        avg /= q + 1
        if case["mode"] == binding.MODE_GOSSIP_MA:
            th[:, a:b] = avg
            continue
        start = o + eta * d if case["mode"] == binding.MODE_PAPER else o
        new = eta * d + zeta * (avg - start)
        om[:, a:b] = o + new
        th[:, a:b] = om[:, a:b] + (eta * new if case["mode"] != binding.MODE_NO_RESTART else 0)
        de[:, a:b] = new
    if case["mode"] == binding.MODE_GOSSIP_MA:
        return _laid_out(th, st, 0)
    return tuple(_laid_out(r, st, a) for a, r in enumerate(rows))
