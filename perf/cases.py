"""The work that is timed when the kernels of this package are tuned.

Five kinds of call, each through the package's public entry points:

  step      training steps (Trainer.step, or the two-stream loop of
            Trainer.prepare and Trainer.train_prepared): the batches in device
            memory, the tables of a model part-way through training;
  loss      Trainer.eval_loss over a held-out batch;
  walks     huge_sample_walks into the caller's buffers, as the producer of
            bench.py calls it: co-occurrence triples from a graph on the device;
  pairs     the evaluation's edge SNR: Evaluator.pairs, .distances, .summary;
  nearest   the evaluation's recall: Evaluator.knn and .recall.

The sizes are those of the workloads in synth/gen.py, of bench.py and of the
tests, with tables scaled to fit the card three times over (the 1e8-row tables
of the headline workload fill it once).  exact() is the same arithmetic in
64 bits in plain torch, from the definitions in include/huge.h.
"""
import ctypes
import math

import numpy as np
import torch

import paper_2307_14490_amd as P

DEV = "cuda"
M32 = 0xFFFFFFFF


# --------------------------------------------------------------------------- #
# Cases
# --------------------------------------------------------------------------- #
def listed():
    return [
        # smallest: the tiny SBM of the tests and the smoke run, latency-bound
        dict(name="step_tiny", kind="step", nodes=10_000, dim=32, negatives=5, batch=1024,
             table="f32", scatter="sorted", graph="sbm", draws="uniform",
             weights="count", steps=1),
        # the medium workload: an SBM with alias negatives over its degrees
        dict(name="step_medium", kind="step", nodes=1_000_000, dim=128, negatives=5,
             batch=65_536, table="f32", scatter="sorted", graph="sbm", draws="alias",
             weights="count", steps=1),
        # the headline loop: batches prepared beside the previous batch's update
        dict(name="loop_f32", kind="step", nodes=20_000_000, dim=128, negatives=5,
             batch=262_144, table="f32", scatter="sorted", graph="sbm", draws="uniform",
             weights="count", steps=6),
        # the same loop on bf16 tables
        dict(name="loop_bf16", kind="step", nodes=20_000_000, dim=128, negatives=5,
             batch=262_144, table="bf16", scatter="sorted", graph="sbm", draws="uniform",
             weights="count", steps=6),
        # the paper's 31 negatives, distance-weighted co-occurrences
        dict(name="step_k31", kind="step", nodes=10_000_000, dim=128, negatives=31,
             batch=131_072, table="f32", scatter="sorted", graph="sbm", draws="uniform",
             weights="float", steps=1),
        # hub-heavy graph: wide rows, power-law endpoints and negatives, ragged batch
        dict(name="step_hub", kind="step", nodes=2_000_000, dim=256, negatives=20,
             batch=100_003, table="f32", scatter="sorted", graph="powerlaw", draws="alias",
             weights="count", steps=1),
        # validation: the loss of a held-out batch, forward only
        dict(name="loss_heldout", kind="loss", nodes=10_000_000, dim=128, negatives=5,
             batch=262_144, table="f32", graph="sbm", draws="uniform", weights="count"),
        # the paper's sampler setting (Table 2): 128 walks of 3 steps from each seed
        dict(name="walks_seed", kind="walks", nodes=1_000_000, degree=22, graph="sbm",
             seeds=65_536, walks=128, steps=3, window=3, seed_only=True, hist=True),
        # DeepWalk windows: one walk of 20 steps from every node, an epoch's triples
        dict(name="walks_window", kind="walks", nodes=500_000, degree=22, graph="sbm",
             seeds=500_000, walks=1, steps=20, window=3, seed_only=False, hist=False),
        # the evaluation's edge SNR over a million edges and as many non-edges
        dict(name="pairs_medium", kind="pairs", nodes=1_000_000, degree=22, dim=128,
             edges=1_000_000, nons=1_000_000),
        # the evaluation's nearest rows of 100 sampled nodes over a large table
        dict(name="nearest_large", kind="nearest", nodes=10_000_000, dim=128, queries=100, k=10,
             degree=0),
        # the same with wide rows, and the recall against the graph
        dict(name="nearest_wide", kind="nearest", nodes=500_000, dim=256, queries=100, k=10,
             degree=22),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges: odd sizes, other widths and options."""
    kind = rng.choice(["step", "step", "step", "step", "loss", "walks", "walks", "pairs",
                       "nearest", "nearest"])
    if kind in ("step", "loss"):
        dim = 4 * _log(rng, 4, 96)
        nodes = _log(rng, 5_000, min(20_000_000, 2_560_000_000 // dim))
        negatives = rng.choice([3, 5, 5, 8, 10, 20, 31])
        table = rng.choice(["f32", "f32", "bf16"])
        scatter = "sorted"
        if table == "f32" and kind == "step" and rng.random() < 0.2:
            scatter = "atomic"
        # row bytes of a batch no more than the 31-negative step's
        top = 500_000_000 // (dim * (2 + negatives)) // (4 if scatter == "atomic" else 1)
        batch = _log(rng, 512, max(1024, min(262_144, top)))
        draws = rng.choice(["uniform", "alias"]) if nodes <= 2_000_000 else "uniform"
        graph = rng.choice(["sbm", "powerlaw"]) if draws == "alias" else "sbm"
        case = dict(kind=kind, nodes=nodes, dim=dim, negatives=negatives, batch=batch,
                    table=table, graph=graph, draws=draws,
                    weights=rng.choice(["count", "count", "float"]))
        if kind == "step":
            case.update(scatter=scatter, steps=rng.choice([1, 1, 4]))
            if case["steps"] > 1:
                case["batch"] = max(512, batch // 2)
        return case
    if kind == "walks":
        nodes = _log(rng, 5_000, 1_000_000)
        case = dict(kind=kind, nodes=nodes, degree=rng.randint(4, 40), graph=rng.choice(["sbm", "sbm", "powerlaw"]))
        if rng.random() < 0.5:
            walks, steps = _log(rng, 4, 256), rng.randint(2, 6)
            case.update(walks=walks, steps=steps, window=rng.randint(1, steps), seed_only=True,
                        hist=rng.random() < 0.7, seeds=min(nodes, 24_000_000 // (walks * steps)))
        else:
            walks, steps = rng.choice([1, 1, 2, 4, 8]), rng.randint(8, 40)
            window = rng.randint(1, 5)
            case.update(walks=walks, steps=steps, window=window, seed_only=False,
                        hist=rng.random() < 0.3,
                        seeds=min(nodes, 50_000_000 // (walks * steps * window * 2)))
        case["seeds"] = rng.randint(max(1, case["seeds"] // 8), case["seeds"])
        return case
    if kind == "pairs":
        nodes = _log(rng, 5_000, 1_000_000)
        return dict(kind=kind, nodes=nodes, degree=rng.randint(4, 30),
                    dim=4 * _log(rng, 4, 96), edges=_log(rng, 10_000, 1_000_000),
                    nons=_log(rng, 10_000, 1_000_000))
    dim = 4 * _log(rng, 8, 128)
    top = 1_280_000_000 // dim if dim <= 128 else 128_000_000 // dim
    return dict(kind=kind, nodes=_log(rng, 20_000, top), dim=dim, queries=rng.randint(1, 128),
                k=rng.choice([1, 5, 10, 10, 20, 32]), degree=0)


# --------------------------------------------------------------------------- #
# Inputs
# --------------------------------------------------------------------------- #
def _generator(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1_000_003 + salt)
    return g


def _rand(g, n):
    return torch.rand(n, generator=g, device=DEV, dtype=torch.float64)


def _hub_nodes(g, n, nodes):
    """Nodes drawn in proportion to about (i + 1)^(-1/1.1) (degree exponent 2.1),
    before relabelling."""
    top = (nodes + 1.0) ** (0.1 / 1.1) - 1.0
    return ((1.0 + _rand(g, n) * top) ** 11.0).long() - 1


def _relabel(nodes, x):
    """An affine bijection of the ids, so that degree or block order gives no
    memory locality."""
    a = int(nodes * 0.6180339887) | 1
    while math.gcd(a, nodes) != 1:
        a += 2
    return (x * a + nodes // 3) % nodes


def _batches(case, seed):
    """`steps` batches of triples: pairs of a 1000-block SBM (25 of 27 within a
    block), or power-law endpoints; counts with a heavy tail."""
    N, n = case["nodes"], case["batch"]
    g = _generator(seed, 1)
    out = []
    for _ in range(case.get("steps", 1)):
        if case["graph"] == "powerlaw":
            src, dst = _hub_nodes(g, n, N), _hub_nodes(g, n, N)
        else:
            blk = max(2, N // 1000)
            src = (_rand(g, n) * N).long()
            inside = (src // blk) * blk + (_rand(g, n) * blk).long()
            dst = torch.where(_rand(g, n) < 25.0 / 27.0, inside, (_rand(g, n) * N).long())
        src, dst = src.clamp_(max=N - 1), dst.clamp_(max=N - 1)
        count = (1.0 / (1e-3 + _rand(g, n)) ** 0.5).clamp_(max=30.0).floor()
        if case["weights"] == "float":
            weight = (count * (0.25 + _rand(g, n))).float()
        else:
            weight = count.int()
        out.append((_relabel(N, src).int(), _relabel(N, dst).int(), weight))
    return out


def _alias_weights(case, seed):
    """degree^0.75: Poisson degrees of an SBM, or the power law's expected ones."""
    N = case["nodes"]
    if case["graph"] == "sbm":
        mean = torch.full((N,), 22.0, dtype=torch.float64, device=DEV)
        return torch.poisson(mean, generator=_generator(seed, 6)).pow(0.75).cpu().numpy()
    i = torch.arange(N, device=DEV)
    w = torch.empty(N, dtype=torch.float64, device=DEV)
    w[_relabel(N, i)] = (i + 1.0).double() ** (-0.75 / 1.1)
    return w.cpu().numpy()


def _tables(case, seed):
    """Two tables as training leaves them: rows of norm about 1.5."""
    g = _generator(seed, 2)
    dt = torch.bfloat16 if case["table"] == "bf16" else torch.float32
    s = 1.5 / math.sqrt(case["dim"])
    out = []
    for _ in range(2):
        t = torch.empty((case["nodes"], case["dim"]), dtype=dt, device=DEV)
        out.append(t.normal_(0.0, s, generator=g))
    return out


def _lr(case):
    # hub rows take thousands of summed contributions per batch
    return 0.025 if case["graph"] == "sbm" else 1e-4


def _first(seed):
    return (int(seed) % 1000) * 10_000_000 + 12_345


def _community(nodes):
    """Nodes of one community of the graph and of the embedding."""
    return max(2, min(nodes // 20, 10_000))


def _graph(case, seed):
    """Symmetric CSR graph (ascending lists, no self loops): an SBM with ten of
    eleven edges inside a block, or power-law endpoints."""
    N, m = case["nodes"], case["nodes"] * case["degree"] // 2
    g = _generator(seed, 3)
    if case.get("graph") == "powerlaw":
        a, b = _hub_nodes(g, m, N), (_rand(g, m) * N).long()
    else:
        blk = _community(N)
        a = (_rand(g, m) * N).long()
        inside = (a // blk) * blk + (_rand(g, m) * blk).long()
        b = torch.where(_rand(g, m) < 10.0 / 11.0, inside, (_rand(g, m) * N).long())
    a, b = a.clamp_(max=N - 1), b.clamp_(max=N - 1)
    keep = a != b
    a, b = _relabel(N, a[keep]), _relabel(N, b[keep])
    key = torch.unique(torch.cat([a * N + b, b * N + a]))
    off = torch.zeros(N + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(torch.bincount(key // N, minlength=N), 0)
    return off, (key % N).int().contiguous()


def _embedding(case, seed):
    """A trained table: rows around the centre of their community of the graph."""
    g = _generator(seed, 4)
    N, D = case["nodes"], case["dim"]
    i = torch.arange(N, device=DEV)
    which = torch.empty_like(i)
    which[_relabel(N, i)] = i // _community(N)
    centre = torch.randn((N // _community(N) + 1, D), generator=g, device=DEV)
    t = torch.randn((N, D), generator=g, device=DEV)
    step = 1 << 20
    for r in range(0, N, step):
        t[r:r + step] += centre[which[r:r + step]]
    return t


def _queries(case, seed):
    g = _generator(seed, 5)
    return (_rand(g, case["queries"]) * case["nodes"]).int().clamp_(max=case["nodes"] - 1)


def _seed_pairs(case):
    """Co-occurrence pairs of one seed, at most."""
    w, L = case["window"], case["steps"] + 1
    return case["walks"] * (w if case["seed_only"] else 2 * w * L - w * (w + 1))


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("step", "loss"):
        S, T = _tables(case, seed)
        w = _alias_weights(case, seed) if case["draws"] == "alias" else None
        tr = P.Trainer(case["nodes"], case["dim"], case["negatives"], case["batch"], seed=seed,
                       alias_weights=w, scatter=case.get("scatter", "sorted"),
                       tables=(S, T), init=False, dtype=case["table"])
        n = case.get("steps", 1)
        return dict(case=case, tr=tr, batches=_batches(case, seed), pos=_first(seed),
                    losses=torch.zeros(n, dtype=torch.float64, device=DEV),
                    side=torch.cuda.Stream())
    if kind == "walks":
        off, nbr = _graph(case, seed)
        cfg = P.walk_config(case["nodes"], case["walks"], case["steps"], case["window"],
                            case["seed_only"], seed)
        cap = case["seeds"] * _seed_pairs(case)
        ws = P.load().huge_walk_workspace_bytes(ctypes.byref(cfg), case["seeds"])
        out = {c: torch.zeros(cap, dtype=torch.int32, device=DEV) for c in ("src", "dst", "cc")}
        if case["hist"]:
            out["hist"] = torch.zeros((cap, case["window"]), dtype=torch.int32, device=DEV)
        out["count"] = torch.zeros(1, dtype=torch.int64, device=DEV)
        out["status"] = torch.zeros(1, dtype=torch.int32, device=DEV)
        return dict(case=case, off=off, nbr=nbr, cfg=cfg, cap=cap, out=out, ws_bytes=ws,
                    ws=torch.empty(ws, dtype=torch.uint8, device=DEV))
    if kind == "pairs":
        off, nbr = _graph(case, seed)
        return dict(case=case, off=off, nbr=nbr, seed=int(seed), table=_embedding(case, seed),
                    ev=P.Evaluator(case["nodes"], case["dim"], case["edges"] + case["nons"]))
    st = dict(case=case, table=_embedding(case, seed), queries=_queries(case, seed),
              ev=P.Evaluator(case["nodes"], case["dim"], 8, k=case["k"]))
    if case["degree"]:
        st["off"], st["nbr"] = _graph(case, seed)
    return st


# --------------------------------------------------------------------------- #
# One pass
# --------------------------------------------------------------------------- #
QUANTILES = list(range(0, 101, 10))


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "step":
        return _run_steps(st, case)
    if kind == "loss":
        src, dst, w = st["batches"][0]
        out = st["tr"].eval_loss(src, dst, w, st["pos"], loss_out=st["losses"])
        st["pos"] += case["batch"]
        return {"loss": out}
    if kind == "walks":
        # the buffers hold the triples up to `count`, and zeros after them
        out = st["out"]
        rc = P.load().huge_sample_walks(
            ctypes.byref(st["cfg"]), st["off"].data_ptr(), st["nbr"].data_ptr(),
            st["nbr"].numel(), (case["nodes"] - case["seeds"]) // 2, case["seeds"],
            out["src"].data_ptr(), out["dst"].data_ptr(), out["cc"].data_ptr(),
            out["hist"].data_ptr() if case["hist"] else None, st["cap"],
            out["count"].data_ptr(), out["status"].data_ptr(), st["ws"].data_ptr(),
            st["ws_bytes"], torch.cuda.current_stream().cuda_stream)
        if rc != 0:
            raise P.HugeError(rc, "huge_sample_walks")
        return out
    if kind == "pairs":
        ev = st["ev"]
        u, v = ev.pairs(st["off"], st["nbr"], case["nodes"], st["seed"], case["edges"],
                        case["nons"])
        dist = ev.distances(st["table"], u, v)
        s = ev.summary(dist, case["edges"], case["nons"], QUANTILES)
        return {"u": u, "v": v, "dist": dist, "snr": s["snr"], "mean_edge": s["mean_edge"],
                "mean_non": s["mean_non"], "pct_edge": np.array(s["pct_edge"]),
                "pct_non": np.array(s["pct_non"])}
    ids, dist = st["ev"].knn(st["table"], st["queries"], case["k"])
    out = {"ids": ids, "dist": dist}
    if case["degree"]:
        out["recall"] = st["ev"].recall(st["off"], st["nbr"], case["nodes"], st["queries"], ids)
    return out


def _run_steps(st, case):
    tr, lr, n = st["tr"], _lr(case), case["batch"]
    B, losses = st["batches"], st["losses"]
    if len(B) == 1:
        tr.step(*B[0], st["pos"], lr, loss_out=losses)
        st["pos"] += n
    else:
        # batch k + 1 is prepared on a stream of its own while batch k is applied
        side = st["side"]
        tr.prepare(*B[0], st["pos"], stream=side)
        for k in range(len(B)):
            if k + 1 < len(B):
                tr.prepare(*B[k + 1], st["pos"] + (k + 1) * n, stream=side)
            tr.train_prepared(lr, loss_out=losses[k:k + 1])
        st["pos"] += n * len(B)
    return {"loss": losses, "S": tr.S, "T": tr.T}


# --------------------------------------------------------------------------- #
# What a pass cannot do without
# --------------------------------------------------------------------------- #
def _unique(draws, nodes):
    """Expected distinct values among `draws` uniform ones."""
    return nodes * -math.expm1(draws * math.log1p(-1.0 / nodes))


def _hub_unique(draws, nodes, power):
    """Expected distinct values among `draws` in proportion to (i + 1)^-power."""
    i = np.unique(np.geomspace(1, nodes + 1, 2000).astype(np.int64))
    lo, hi = i[:-1], i[1:]
    mid = 0.5 * (lo + hi - 1)
    w = mid ** -power
    return float(np.sum((hi - lo) * -np.expm1(-draws * w / np.sum((hi - lo) * w))))


def work(case):
    kind = case["kind"]
    if kind in ("step", "loss"):
        N, D, K, n = case["nodes"], case["dim"], case["negatives"], case["batch"]
        eb = 2 if case["table"] == "bf16" else 4
        if case["graph"] == "powerlaw":
            rows = _hub_unique(n, N, 1 / 1.1) + _hub_unique(n * (1 + K), N, 0.75 / 1.1)
        else:
            rows = _unique(n, N) + _unique(n * (1 + K), N)
        moves = 1 if kind == "loss" else 2  # read once; a step writes each row once too
        steps = case.get("steps", 1)
        flops = 2.0 * n * (1 + K) * D * (1 if kind == "loss" else 3)
        return {"bytes": steps * (12.0 * n + moves * eb * D * rows), "flops": steps * flops}
    if kind == "walks":
        hops = case["seeds"] * case["walks"] * case["steps"]
        if case["seed_only"]:
            per = _unique(case["walks"] * case["window"],
                          case["degree"] + case["degree"] ** 2 * max(1, case["window"] - 1))
        else:
            per = 0.9 * _seed_pairs(case)
        each = 12 + (4 * case["window"] if case["hist"] else 0)
        # per hop two offsets and a neighbour; the triples written once
        return {"bytes": 20.0 * hops + each * case["seeds"] * per, "flops": 0.0}
    if kind == "pairs":
        n = case["edges"] + case["nons"]
        return {"bytes": n * (8.0 * case["dim"] + 8 + 4 + 24), "flops": n * 10.0 * case["dim"]}
    N, D = case["nodes"], case["dim"]
    return {"bytes": 4.0 * N * D, "flops": 2.0 * N * D * case["queries"]}


def tolerance(case):
    kind = case["kind"]
    if kind == "walks":
        return "exact"
    if kind == "step":
        if case["table"] == "bf16":
            # an element at a rounding boundary may take the neighbouring bf16 value
            return {"rel": 2e-5, "max": 0.03}
        if case["scatter"] == "atomic":  # hub rows: sums in arbitrary order
            return {"rel": 3e-6, "max": 2e-4}
        return {"rel": 2e-7, "max": 5e-6}
    if kind == "loss":
        return {"rel": 2e-8}
    # distances from fp32 sums; ids of rows nearer each other than their rounding
    return {"rel": 5e-7, "max": 3e-6, "differ": 0.01}


# --------------------------------------------------------------------------- #
# The same in 64 bits
# --------------------------------------------------------------------------- #
def _mul32(a, b):
    """(high, low) 32-bit words of the products of 32-bit values held in int64."""
    p = a * b  # modulo 2^64
    return (p >> 32) & M32, p & M32


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 on int64 tensors of 32-bit counter words."""
    k0, k1 = int(seed) & M32, (int(seed) >> 32) & M32
    for _ in range(10):
        ha, la = _mul32(c0, 0xD2511F53)
        hb, lb = _mul32(c2, 0xCD9E8D57)
        c0, c1, c2, c3 = hb ^ c1 ^ k0, lb, ha ^ c3 ^ k1, la
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return c0, c1, c2, c3


def _scaled(lo, hi, n):
    """floor(x n / 2^64) of x = hi 2^32 + lo, for n < 2^31."""
    return (hi * n + ((lo * n) >> 32)) >> 32


def _alias_table(w):
    """Walker's table in exact integers (small buckets filled first in, first out)."""
    from collections import deque
    n = len(w)
    unit = 1 << 32
    scale = float(n) * 4294967296.0 / float(np.add.accumulate(w)[-1])
    mass = (w * scale).astype(np.uint64).tolist()
    largest = int(np.argmax(np.asarray(mass, dtype=np.uint64)))
    mass[largest] += n * unit - sum(mass)
    thr, alias = [M32] * n, list(range(n))
    small = deque(j for j in range(n) if mass[j] < unit)
    large = deque(j for j in range(n) if mass[j] >= unit)
    while small and large:
        s, l = small.popleft(), large[0]
        thr[s], alias[s] = mass[s], l
        mass[l] -= unit - mass[s]
        if mass[l] < unit:
            small.append(large.popleft())
    return (torch.tensor(thr, dtype=torch.int64, device=DEV),
            torch.tensor(alias, dtype=torch.int64, device=DEV))


def _negatives(case, seed, pos, n, table):
    K, N = case["negatives"], case["nodes"]
    p = (pos + torch.arange(n, device=DEV)).repeat_interleave(K)
    k = torch.arange(K, device=DEV).repeat(n)
    r0, r1, r2, _ = _philox(p & M32, p >> 32, k, torch.ones_like(p), seed)
    j = _scaled(r0, r1, N)
    if table is not None:
        j = torch.where(r2 < table[0][j], j, table[1][j])
    return j.view(n, K)


def _softplus(z):
    return z.clamp(min=0.0) + torch.log1p(torch.exp(-z.abs()))


def _exact_steps(case, seed):
    S, T = (t.double() for t in _tables(case, seed))
    table = _alias_table(_alias_weights(case, seed)) if case["draws"] == "alias" else None
    n, K, D, pos, lr = case["batch"], case["negatives"], case["dim"], _first(seed), _lr(case)
    if case["kind"] == "step":
        lr = float(np.float32(lr))
    losses = []
    chunk = max(1, (1 << 27) // ((2 + K) * D))
    for src, dst, w in _batches(case, seed):
        neg = _negatives(case, seed, pos, n, table)
        src, ctx = src.long(), torch.cat([dst.long().view(-1, 1), neg], 1)
        rs, is_ = torch.unique(src, return_inverse=True)
        rt, it = torch.unique(ctx, return_inverse=True)
        if case["kind"] == "step":
            gs = torch.zeros((rs.numel(), D), dtype=torch.float64, device=DEV)
            gt = torch.zeros((rt.numel(), D), dtype=torch.float64, device=DEV)
        total = torch.zeros((), dtype=torch.float64, device=DEV)
        for a in range(0, n, chunk):
            b = min(n, a + chunk)
            s, t, c = S[src[a:b]], T[ctx[a:b]], w[a:b].double().view(-1, 1)
            z = (s.unsqueeze(1) * t).sum(2)
            z[:, 0] *= -1.0
            total += (c * _softplus(z)).sum()
            if case["kind"] == "step":
                h = c * torch.sigmoid(z)
                h[:, 0] *= -1.0
                gs.index_add_(0, is_[a:b], (h.unsqueeze(2) * t).sum(1))
                gt.index_add_(0, it[a:b].reshape(-1),
                              (h.unsqueeze(2) * s.unsqueeze(1)).reshape(-1, D))
        losses.append(total)
        if case["kind"] == "step":
            S[rs] = _stored(case, S[rs] - lr * gs)
            T[rt] = _stored(case, T[rt] - lr * gt)
        pos += n
    out = {"loss": torch.stack(losses)}
    if case["kind"] == "step":
        out.update(S=S, T=T)
    return out


def _stored(case, x):
    """A bf16 table keeps bf16 values between steps; an fp32 one is followed in
    64 bits."""
    return x.bfloat16().double() if case["table"] == "bf16" else x


def _exact_pairs(case, seed):
    off, nbr = _graph(case, seed)
    N, E = case["nodes"], nbr.numel()
    j = torch.arange(case["edges"], device=DEV)
    r0, r1, _, _ = _philox(j & M32, j >> 32, torch.zeros_like(j),
                           torch.full_like(j, 0x80000001), seed)
    e = _scaled(r0, r1, E)
    u = torch.searchsorted(off, e, right=True) - 1
    v = nbr[e].long()
    keys = torch.repeat_interleave(torch.arange(N, device=DEV), off[1:] - off[:-1]) * N + nbr
    nu = torch.full((case["nons"],), -1, dtype=torch.int64, device=DEV)
    nv = nu.clone()
    left = torch.arange(case["nons"], device=DEV)
    for a in range(64):
        if left.numel() == 0:
            break
        r0, r1, r2, r3 = _philox(left & M32, left >> 32, torch.full_like(left, a),
                                 torch.full_like(left, 0x80000002), seed)
        x, y = _scaled(r0, r1, N), _scaled(r2, r3, N)
        at = torch.searchsorted(keys, x * N + y).clamp_(max=E - 1)
        good = (x != y) & (keys[at] != x * N + y)
        nu[left[good]], nv[left[good]] = x[good], y[good]
        left = left[~good]
    u, v = torch.cat([u, nu]), torch.cat([v, nv])
    table = _embedding(case, seed)
    dist = torch.empty(u.numel(), dtype=torch.float64, device=DEV)
    step = max(1, (1 << 27) // case["dim"])
    for a in range(0, u.numel(), step):
        x, y = table[u[a:a + step]].double(), table[v[a:a + step]].double()
        dist[a:a + step] = (x / x.norm(dim=1, keepdim=True) -
                            y / y.norm(dim=1, keepdim=True)).norm(dim=1)
    de, dn = dist[:case["edges"]].cpu().numpy(), dist[case["edges"]:].cpu().numpy()
    return {"u": u.int(), "v": v.int(), "dist": dist, "snr": float(dn.mean() / de.mean()),
            "mean_edge": float(de.mean()), "mean_non": float(dn.mean()),
            "pct_edge": np.percentile(de, QUANTILES), "pct_non": np.percentile(dn, QUANTILES)}


def _exact_nearest(case, seed):
    table, q = _embedding(case, seed), _queries(case, seed).long()
    x = table[q].double()
    x = x / x.norm(dim=1, keepdim=True)
    k, N = case["k"], case["nodes"]
    best = torch.full((q.numel(), 0), 0.0, dtype=torch.float64, device=DEV)
    ids = torch.zeros((q.numel(), 0), dtype=torch.int64, device=DEV)
    step = max(k + 1, min(1 << 20, (1 << 28) // case["dim"]))
    for a in range(0, N, step):
        y = table[a:a + step].double()
        y = y / y.norm(dim=1, keepdim=True)
        d2 = (2.0 - 2.0 * torch.mm(x, y.t())).clamp_(min=0.0)
        own = (q >= a) & (q < a + y.shape[0])
        d2[own.nonzero().view(-1), q[own] - a] = math.inf
        d2, at = torch.topk(d2, min(k, y.shape[0]), largest=False)
        best, ids = torch.cat([best, d2], 1), torch.cat([ids, at + a], 1)
        best, at = torch.topk(best, min(k, best.shape[1]), largest=False, sorted=True)
        ids = ids.gather(1, at)
    out = {"ids": ids.int(), "dist": best.sqrt()}
    if case["degree"]:
        off, nbr = _graph(case, seed)
        keys = torch.repeat_interleave(torch.arange(N, device=DEV), off[1:] - off[:-1]) * N + nbr
        want = q.view(-1, 1) * N + ids
        at = torch.searchsorted(keys, want).clamp_(max=keys.numel() - 1)
        out["recall"] = (keys[at] == want).double().mean(1)
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "walks":
        return None  # whole numbers only
    if kind in ("step", "loss"):
        return _exact_steps(case, seed)
    return _exact_pairs(case, seed) if kind == "pairs" else _exact_nearest(case, seed)
