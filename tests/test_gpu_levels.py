"""GPU parity of the level kernel at the sizes where its work split, its
strings of launches and its hand-over to the host change, against the oracle:
levels around a tile's states, rules of one to five participants, states
without successors, strings of more levels than a control block holds, limits
on the buffers that send some levels to the host, tables too large for
buffers of their own size."""
import numpy as np
import pytest

import oracle
import paper_1801_05857_amd as gx
import workloads as W

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gx.lib()


def _same(got, want, table=None):
    assert got.n_states == want.n_states
    assert got.levels.tolist() == want.levels.tolist()
    assert got.n_transitions == want.n_transitions
    assert np.array_equal(got.deadlocks, want.deadlocks)
    if table is not None:
        assert np.array_equal(table.dump(), want.visited)


def _star(width, tail):
    """A root with `width` successors, each the start of a chain of `tail`
    states: levels 1, width, width, ... (width, tail as the test likes), the
    chains' ends deadlocks."""
    n = 1 + width * tail
    trans = [(0, 0, 1 + i) for i in range(width)]
    trans += [(1 + i + width * k, 0, 1 + i + width * (k + 1)) for k in range(tail - 1)
              for i in range(width)]
    return W._net([n], [0], [trans], 1, np.zeros((0, 1)), f"star_{width}x{tail}")


# level sizes at the edges of a tile, a workgroup and the string of launches
@pytest.mark.parametrize("width", [1, 2, 31, 32, 33, 63, 64, 65, 511, 513])
@pytest.mark.parametrize("dedup", [False, True])
def test_level_sizes(width, dedup):
    tail = 70 if width < 64 else 18
    net = _star(width, tail)
    want = oracle.explore(net, want_visited=True)
    with gx.Table(want.words, 16, 2 * want.n_states, subgroup=4, max_hashes=64) as t:
        for _ in range(2):
            t.clear()
            _same(gx.explore(net, t, local_dedup=dedup), want, t)


def _mixed_rules(seed, P, n):
    """Free transitions and rules of one to five participants over P processes
    of n states, several transitions a label and state; some rules are never
    enabled."""
    rng = W.SplitMix64(seed)
    labels = 8
    trans = [[(s, rng.below(labels), rng.below(n)) for s in range(n) for _ in range(3)]
             for _ in range(P)]
    rules = np.full((6, P), -1, dtype=np.int32)
    for r, k in enumerate((1, 2, 3, 4, 5, 3)):
        for i in range(min(k, P)):
            rules[r, (r + i) % P] = r if r < 5 else labels  # rule 5: a label nobody has
    return W._net([n] * P, [0] * P, trans, labels + 1, rules, f"mixed_{seed}")


@pytest.mark.parametrize("seed,P,n", [(1, 2, 9), (2, 3, 7), (3, 5, 5), (4, 6, 4), (5, 7, 3),
                                      (6, 12, 2)])
@pytest.mark.parametrize("B", [4, 8, 16, 32, 64])
def test_rules_of_every_size(seed, P, n, B):
    net = _mixed_rules(seed, P, n)
    want = oracle.explore(net, want_visited=True)
    if B // (4 if want.words == 3 else want.words) < 1:
        pytest.skip("bucket smaller than a slot")
    with gx.Table(want.words, B, 2 * want.n_states, max_hashes=64) as t:
        _same(gx.explore(net, t), want, t)


# a limit on the frontier keeps the plain bound of a level's successors: small
# levels are strung together, wide ones go to the host, in turn
@pytest.mark.parametrize("frontier,slices", [(0, 0), (1 << 15, 0), (1 << 17, 0), (0, 2000),
                                             (1 << 17, 5000)])
def test_host_and_device_levels_in_turn(frontier, slices):
    net = W.large_random_network(live=4)
    want = oracle.explore(net, want_visited=True)
    with gx.Table(want.words, 16, 2 * want.n_states, max_hashes=64) as t:
        for _ in range(2):
            t.clear()
            try:
                got = gx.explore(net, t, frontier_capacity=frontier, slice_states=slices)
            except gx.GxError as e:  # the widest level may exceed the limit
                assert e.code == gx.GX_ENOMEM and frontier == 1 << 15
                continue
            _same(got, want, t)


def test_table_larger_than_its_buffers():
    """A table of more than 256 MiB: its buffers grow with the levels."""
    net = W.large_random_network(live=4)
    want = oracle.explore(net, want_visited=True)
    with gx.Table(want.words, 16, (300 << 20) // 16, subgroup=4, max_hashes=16) as t:
        for _ in range(2):
            t.clear()
            _same(gx.explore(net, t), want)


def test_full_table_inside_a_string():
    """The table fills up in the middle of a string of levels: an error, and
    what is stored is reachable."""
    net = W.large_random_network(live=4)
    want = oracle.explore(net, want_visited=True)
    with gx.Table(want.words, 16, want.n_states // 3, subgroup=4, max_hashes=4) as t:
        with pytest.raises(gx.GxError) as e:
            gx.explore(net, t)
        assert e.value.code == gx.GX_ETABLEFULL
        have = {r.tobytes() for r in want.visited}
        dump = t.dump()
        assert all(r.tobytes() in have for r in dump)
        assert len({r.tobytes() for r in dump}) == len(dump)


@pytest.mark.parametrize("n", [1, 5, 40])
def test_batches_of_uneven_levels(n):
    """A batch whose instances' levels differ a hundredfold shares lanes by
    the step's states; the persistent schedule by the level's."""
    nets = [W.random_lts(300 + i, 3 + i % 6, 16, 2 + i % 5, 3, 16, 0.25, 0.1) for i in range(n)]
    want = [oracle.explore(net, want_visited=True) for net in nets]
    caps = [max(64, 4 * w.n_states) for w in want]
    for persistent in (False, True):
        with gx.Batch(nets, caps, bucket_words=16, subgroup=4, max_hashes=32, keep_states=True,
                      persistent=persistent) as b:
            b.run()
            for (st, got), w in zip(b.results(), want):
                assert st == gx.GX_OK
                _same(got, w)
                assert np.array_equal(got.states, w.visited)


def _shared_targets(P, n, copies, rules):
    """Cycles of n states whose steps are offered `copies` times, beside
    self-loops; with rules, neighbours meet on labels offered several times,
    to the same target, to the source and to another one."""
    trans, rows = [], []
    for p in range(P):
        t = [(s, 0, (s + 1) % n) for s in range(n) for _ in range(copies)]
        t += [(s, 0, s) for s in range(0, n, 2) for _ in range(copies + 1)]
        if rules:
            t += [(s, 1, d) for s in range(n) for d in (s, s, (s + 2) % n)]
        trans.append(t)
    if rules:
        rows = [[1 if x in (p, (p + 1) % P) else -1 for x in range(P)] for p in range(P - 1)]
        rows.append([1] * P)
    return W._net([n] * P, [0] * P, trans, 2, np.asarray(rows or np.zeros((0, P)), np.int32),
                  "shared_targets")


@pytest.mark.parametrize("P,n,copies,rules", [(1, 2, 1, False), (1, 7, 40, False), (3, 9, 1, True),
                                              (3, 9, 3, True), (4, 8, 2, True), (5, 6, 2, False),
                                              (4, 17, 2, False)])
@pytest.mark.parametrize("dedup", [False, True])
def test_transitions_that_share_a_successor(P, n, copies, rules, dedup):
    """Every transition counts, each successor is formed once; a state whose
    steps all lead to itself is no deadlock."""
    net = _shared_targets(P, n, copies, rules)
    want = oracle.explore(net, want_visited=True)
    with gx.Table(want.words, 16, max(64, 2 * want.n_states), max_hashes=64) as t:
        got = gx.explore(net, t, local_dedup=dedup)
        _same(got, want, t)
        if dedup:
            assert t.stats().lookups + got.local_duplicates == want.n_transitions + 1
    with gx.Batch([net], [2 * want.n_states], bucket_words=16, subgroup=4, max_hashes=64) as b:
        b.run()
        (st, got), = b.results()
        assert st == gx.GX_OK
        _same(got, want)


@pytest.mark.parametrize("width,tail", [(3, 200), (40, 9), (700, 6)])
def test_one_table_on_streams_in_turn(width, tail):
    """The host goes on from what a string's last launch has reported: the next
    exploration of the table, on another stream, must not meet what is left of
    the one before (strings of more launches than reports are kept, too)."""
    net = _star(width, tail)
    want = oracle.explore(net, want_visited=True)
    streams = [torch.cuda.Stream() for _ in range(3)]
    with gx.Table(want.words, 16, 2 * want.n_states, max_hashes=64) as t:
        for k in range(24):
            s = streams[k % 3]
            t.clear(stream=s)
            _same(gx.explore(net, t, stream=s), want, t if k % 6 == 5 else None)
