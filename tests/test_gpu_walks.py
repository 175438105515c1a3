"""GPU random-walk sampler (Sec. 3.2, Alg. 1) against the CPU oracle, through
the C ABI: triples, co_counts and distance histograms bit-exact, in the same
order, on SBM, random and deterministic graphs, for the paper's seed pairs
and for window pairs; errors (a malformed graph, too small a capacity) are
reported and write nothing; the triples feed the training step."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import oracle as orc  # noqa: E402
import paper_2307_14490_amd as P  # noqa: E402
from gpu_common import assert_close, dev, say  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield
    torch.cuda.synchronize()


def _graph(kind, n, seed=0):
    rng = np.random.default_rng(seed)
    if kind == "sbm":
        from synth import csr_from_edges, sbm_edges
        edges = sbm_edges(n, 10, 8.0, 1.0, rng)
        off, nbr = csr_from_edges(n, edges)
    elif kind == "random_with_sinks":
        # directed edges; a tenth of the nodes have no out-edges
        m = 6 * n
        a = rng.integers(0, n, m)
        b = rng.integers(0, n, m)
        keep = (a % 10) != 3
        a, b = a[keep], b[keep]
        order = np.lexsort((b, a))
        a, b = a[order], b[order]
        off = np.zeros(n + 1, np.int64)
        np.add.at(off, a + 1, 1)
        off = np.cumsum(off)
        nbr = b.astype(np.int32)
    elif kind == "cycle":
        off = np.arange(n + 1, dtype=np.int64)
        nbr = ((np.arange(n) + 1) % n).astype(np.int32)
    else:
        raise ValueError(kind)
    return np.asarray(off, np.int64), np.asarray(nbr, np.int32)


CASES = [
    # graph, n, walks, steps, window, seed_only, note
    ("sbm", 3000, 128, 3, 3, True, "the paper's sampler: 128 walks of 3 steps per node"),
    ("sbm", 2000, 4, 10, 2, False, "tiny workload's walks: window pairs"),
    ("random_with_sinks", 5000, 8, 20, 3, False, "dead ends, window 3"),
    ("random_with_sinks", 5000, 16, 12, 12, True, "dead ends, seed pairs"),
    ("cycle", 257, 3, 64, 32, True, "deterministic walks, longest walk and window"),
    ("sbm", 1500, 1024, 3, 1, True, "most walks per seed"),
    ("sbm", 1000, 1, 40, 5, False, "one long walk per seed"),
]


@pytest.mark.parametrize("kind,n,walks,steps,window,seed_only,note", CASES)
def test_walk_triples_bit_exact(kind, n, walks, steps, window, seed_only, note):
    say(f"walks {kind} n={n} walks={walks} steps={steps} window={window} seed_only={seed_only}")
    off, nbr = _graph(kind, n, seed=n)
    first, count = 17, n - 40
    ref = orc.sample_walks(off, nbr, n, walks, steps, window, seed_only, seed=99,
                           first_seed=first, num_seeds=count)
    got = P.sample_walks(dev(off, torch), dev(nbr, torch), n, walks, steps, window, seed_only,
                         seed=99, first_seed=first, num_seeds=count)
    for name, g, r in zip(("src", "dst", "cc", "hist"), got, ref):
        g = g.cpu().numpy()
        assert g.shape == r.shape, (name, g.shape, r.shape)
        assert np.array_equal(g, r), name


def test_capacity_and_malformed_graph_are_reported():
    n = 500
    off, nbr = _graph("sbm", n, seed=1)
    doff, dnbr = dev(off, torch), dev(nbr, torch)
    src, dst, cc, hist = P.sample_walks(doff, dnbr, n, 8, 5, 2, True, seed=3)
    need = src.numel()
    with pytest.raises(P.HugeError) as e:
        P.sample_walks(doff, dnbr, n, 8, 5, 2, True, seed=3, capacity=need - 1)
    assert e.value.status == -4
    bad = nbr.copy()
    v = int(np.argmax(np.diff(off) > 0))     # a seed with neighbours: its first step is bad
    bad[off[v]:off[v + 1]] = n + 5
    with pytest.raises(P.HugeError) as e:
        P.sample_walks(doff, dev(bad, torch), n, 8, 5, 2, True, seed=3)
    assert e.value.status == -2
    # host-side argument checks
    with pytest.raises(P.HugeError):
        P.sample_walks(doff, dnbr, n, 2000, 5, 2, True)       # too many walks per seed
    with pytest.raises(P.HugeError):
        P.sample_walks(doff, dnbr, n, 8, 5, 6, True)          # window > steps
    with pytest.raises(P.HugeError):
        P.sample_walks(doff, dnbr, n, 8, 5, 2, True, first_seed=400, num_seeds=200)


def test_walk_triples_train_like_the_oracle():
    """Triples produced on the GPU train one step; the oracle produces its own
    triples from the same graph and takes the same step."""
    n, D, K = 4000, 32, 5
    off, nbr = _graph("sbm", n, seed=5)
    src, dst, cc, _ = P.sample_walks(dev(off, torch), dev(nbr, torch), n, 16, 4, 2, False,
                                     seed=8, with_hist=False)
    m = 3000
    tr = P.Trainer(n, D, K, m, seed=4)
    loss = tr.step(src[:m], dst[:m], cc[:m], 0, 0.05).item()
    assert tr.check() == 0
    rs, rd, rc, _ = orc.sample_walks(off, nbr, n, 16, 4, 2, False, seed=8)
    ids = np.arange(n)
    a = float(np.float32(0.5 / D))
    S = orc.init_rows(4, 0, ids, D, a)
    T = orc.init_rows(4, 1, ids, D, a)
    neg = orc.sample_negatives(4, 0, m, K, n)
    ref = orc.step_dense(S, T, rs[:m], rd[:m], rc[:m], neg, 0.05)
    assert loss == pytest.approx(ref, rel=1e-5)
    assert_close(tr.S.cpu().numpy(), S, "S")
    assert_close(tr.T.cpu().numpy(), T, "T")


# The group kernel's variants: pairs per seed at and around powers of two
# (1 .. 64 keys per lane), with the nodes of window pairs in the small sort
# and in the full one.
EDGES = [
    (1, 1, 1, True), (21, 3, 3, True), (16, 4, 4, True), (13, 5, 5, True), (43, 6, 3, True),
    (64, 8, 5, True), (101, 7, 7, True), (1024, 4, 4, True),
    (1, 1, 1, False), (1, 17, 2, False), (2, 9, 2, False), (1, 64, 32, False),
    (16, 20, 6, False), (2048 // 64, 64, 1, False), (5, 64, 3, False), (15, 20, 8, False),
    (1024, 2, 1, False),
]


@pytest.mark.parametrize("walks,steps,window,seed_only", EDGES)
def test_walk_group_variants_match_the_oracle(walks, steps, window, seed_only):
    say(f"walk group walks={walks} steps={steps} window={window} seed_only={seed_only}")
    n = 150
    off, nbr = _graph("random_with_sinks", n, seed=walks + steps)
    ref = orc.sample_walks(off, nbr, n, walks, steps, window, seed_only, seed=5, first_seed=3,
                           num_seeds=101)
    got = P.sample_walks(dev(off, torch), dev(nbr, torch), n, walks, steps, window, seed_only,
                         seed=5, first_seed=3, num_seeds=101)
    for name, g, r in zip(("src", "dst", "cc", "hist"), got, ref):
        assert np.array_equal(g.cpu().numpy(), r), name


@pytest.mark.parametrize("n", [2 ** 27 - 1, 2 ** 27 + 3])
def test_walks_on_ids_at_the_width_of_a_direct_key(n):
    """Ids up to 27 bits fit a pair key beside the distance; larger ones are
    taken by their places in the seed's sorted nodes.  Only the last 1000
    nodes have neighbours."""
    m, deg = 1000, 5
    off = np.zeros(n + 1, np.int64)
    off[n - m:] = np.arange(m + 1) * deg
    nbr = np.random.default_rng(1).integers(n - m, n, m * deg).astype(np.int32)
    first, count = n - 300, 300
    say(f"walks n={n}")
    ref = orc.sample_walks(off, nbr, n, 30, 6, 5, True, seed=2, first_seed=first,
                           num_seeds=count)
    got = P.sample_walks(dev(off, torch), dev(nbr, torch), n, 30, 6, 5, True, seed=2,
                         first_seed=first, num_seeds=count)
    for name, g, r in zip(("src", "dst", "cc", "hist"), got, ref):
        assert np.array_equal(g.cpu().numpy(), r), name


def test_triple_counts_are_scanned_over_many_ranges():
    """5,000 seeds of a cycle: every seed has the same number of triples, so
    the places of all of them are known."""
    n, steps = 5000, 4
    off, nbr = _graph("cycle", n)
    src, dst, cc, hist = P.sample_walks(dev(off, torch), dev(nbr, torch), n, 2, steps, steps,
                                        True, seed=1)
    assert src.numel() == n * steps
    want = np.repeat(np.arange(n), steps)
    assert np.array_equal(src.cpu().numpy(), want)
    ring = (np.arange(n)[:, None] + np.arange(1, steps + 1)) % n
    assert np.array_equal(dst.cpu().numpy(), np.sort(ring, axis=1).reshape(-1))
    assert (cc == 2).all() and (hist.sum(1) == 2).all()


@pytest.mark.parametrize("seed_only", [True, False])
def test_more_seeds_than_waves_of_one_launch(seed_only):
    """2^26 + 5 seeds of one walk of one step: their nodes fit the workspace,
    but a wave for each in one launch would be more than 2^32 - 1 threads."""
    n = 2 ** 26 + 5
    say(f"walks n={n} of one step, seed_only={seed_only}")
    off = torch.arange(n + 1, dtype=torch.int64, device="cuda")
    nbr = (off[:-1] + 1).remainder(n).int()
    src, dst, cc, _ = P.sample_walks(off, nbr, n, 1, 1, 1, seed_only, seed=1, with_hist=False)
    ids = off[:-1].int()
    if seed_only:
        assert torch.equal(src, ids) and torch.equal(dst, nbr)
    else:  # (s, s + 1) and (s + 1, s), ascending by source
        a, b = torch.minimum(ids, nbr), torch.maximum(ids, nbr)
        assert torch.equal(src.view(-1, 2), torch.stack([a, b], 1))
        assert torch.equal(dst.view(-1, 2), torch.stack([b, a], 1))
    assert bool((cc == 1).all())


@pytest.mark.parametrize("walks,steps,window,seed_only", [(1024, 4, 4, True), (16, 40, 1, False)])
def test_a_small_workspace_takes_the_seeds_in_chunks(walks, steps, window, seed_only):
    """2048 bytes of nodes per seed, an eighth (0.8) of what the walks need: the
    same triples as with room for all."""
    import ctypes
    n, seeds = 400, 101
    off, nbr = _graph("sbm", n)
    doff, dnbr = dev(off, torch), dev(nbr, torch)
    say(f"walks in chunks walks={walks} steps={steps}")
    want = P.sample_walks(doff, dnbr, n, walks, steps, window, seed_only, seed=4, first_seed=7,
                          num_seeds=seeds)
    cfg = P.walk_config(n, walks, steps, window, seed_only, 4)
    few = P.walk_config(n, 1, 1, 1, True, 4)  # 2048 bytes per seed are the least reported
    need = P.load().huge_walk_workspace_bytes(ctypes.byref(few), seeds)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    assert ws.data_ptr() % 256 == 0
    total = want[0].numel()
    out = [torch.empty_like(x) for x in want]
    count = torch.zeros(1, dtype=torch.int64, device="cuda")
    status = torch.zeros(1, dtype=torch.int32, device="cuda")

    def run(nbytes):
        return P.load().huge_sample_walks(
            ctypes.byref(cfg), doff.data_ptr(), dnbr.data_ptr(), dnbr.numel(), 7, seeds,
            *(x.data_ptr() for x in out), total, count.data_ptr(), status.data_ptr(),
            ws.data_ptr(), nbytes, torch.cuda.current_stream().cuda_stream)

    assert run(need - 1) == -4
    assert run(need) == 0
    assert int(status.item()) == 0 and int(count.item()) == total
    for x, y in zip(out, want):
        assert torch.equal(x, y)
