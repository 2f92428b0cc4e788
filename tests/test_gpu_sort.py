"""GPU parity of the sorted lists: table dumps at the sizes where the device's
gather and radix sort change shape (chunks, rounds, words and digits in which
keys do not differ), violation and deadlock lists longer than the host sorts,
reachable sets of batches and servers, against numpy's order of the same
rows."""
import numpy as np
import pytest

import oracle
import paper_1801_05857_amd as gx
import workloads as W

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    gx.lib()
    return torch.device("cuda:0")


def _rows(keys):
    return keys[np.lexsort(keys.T[::-1])]


def _fill(t, keys, dev):
    k = torch.from_numpy(np.ascontiguousarray(keys).view(np.int32)).to(dev)
    st = torch.empty(keys.shape[0], dtype=torch.uint8, device=dev)
    t.find_or_put(k, st)
    assert (st.cpu().numpy() == gx.GX_NEW).all()


@pytest.mark.parametrize("w", [1, 2, 3, 4])
@pytest.mark.parametrize("n", [0, 1, 255, 2047, 2048, 2049, 5 * 2048 + 3, 300_001])
def test_dump_sizes(dev, w, n):
    keys = W.distinct_keys(n, w, seed=11 + w)
    with gx.Table(w, 16, max(40_000, 2 * n), max_hashes=64) as t:
        if n:
            _fill(t, keys, dev)
        for _ in range(2):
            assert np.array_equal(t.dump(), _rows(keys))


@pytest.mark.parametrize("w", [1, 2, 3, 4])
@pytest.mark.parametrize("bits", ["high", "word0", "last", "all"])
def test_dump_digits(dev, w, bits):
    """Keys that differ in a few bits only, the highest among them."""
    n = 4000
    i = np.arange(n, dtype=np.uint32)
    keys = np.full((n, w), 0x12345678, dtype=np.uint32)
    if bits == "high":
        keys[:, 0] = (i << np.uint32(20)) | np.uint32(5)
    elif bits == "word0":
        keys[:, 0] = i * np.uint32(3)
    elif bits == "last":
        keys[:, w - 1] = i << np.uint32(7)
    else:
        x = W.distinct_keys(n, w, seed=3)
        keys = x ^ np.uint32(0x80000000)
    with gx.Table(w, 32, 60_000, max_hashes=64) as t:
        _fill(t, keys, dev)
        assert np.array_equal(t.dump(), _rows(keys))


def test_dump_after_exploration_and_again(dev):
    """The dump uses the exploration's buffers: the next exploration into the
    table is unchanged."""
    net = W.large_random_network(live=3)
    want = oracle.explore(net, want_visited=True)
    with gx.Table(want.words, 16, 2 * want.n_states, max_hashes=64) as t:
        for _ in range(3):
            t.clear()
            got = gx.explore(net, t)
            assert got.levels.tolist() == want.levels.tolist()
            assert np.array_equal(t.dump(), want.visited)
            assert np.array_equal(t.dump(), want.visited)


def test_many_violations_with_the_initial_state_bad(dev):
    """Bad from the first state on: its record goes to its place among the
    others."""
    net = W.large_random_network(live=3)
    aut = (2, 0, [(0, 0, 1), (1, 0, 0)])
    want = oracle.explore_automaton(net, aut, [0])
    comp, mp, flags = gx.add_monitor(net, aut, [0])
    assert len(want.violations) > 4096
    with gx.Table(want.words, 16, 2 * want.n_states, max_hashes=64) as t:
        got = gx.explore(comp, t, monitor=(mp, flags))
        assert got.violation_level == 0
        assert np.array_equal(got.violations, want.violations)


def test_many_deadlocks(dev):
    net = W.wide_rule(6, 5)
    want = oracle.explore(net)
    with gx.Table(want.words, 16, 4 * want.n_states, max_hashes=64) as t:
        got = gx.explore(net, t)
        assert len(got.deadlocks) == 5 ** 6
        assert np.array_equal(got.deadlocks, want.deadlocks)


def test_kept_states_of_batches_and_servers(dev):
    nets = [W.large_random_network(live=3), W.token_ring(8), W.tiny_cycles()]
    want = [oracle.explore(n, want_visited=True) for n in nets]
    caps = [2 * w.n_states for w in want]
    with gx.Batch(nets, caps, bucket_words=16, subgroup=4, max_hashes=64, keep_states=True) as b:
        for _ in range(2):
            b.run()
            for (st, got), w in zip(b.results(), want):
                assert st == gx.GX_OK and np.array_equal(got.states, w.visited)
    with gx.Server(1 << 30, max_hashes=64, bucket_words=16, subgroup=4, keep_states=True) as s:
        ids = [s.submit(n, w.n_states) for n, w in zip(nets, want)]
        for i, w in zip(ids, want):
            st, got, _ = s.poll(i)
            assert st == gx.GX_OK and np.array_equal(got.states, w.visited)


@pytest.mark.parametrize("w", [1, 2, 3])
@pytest.mark.parametrize("n", [512 * 2048, 512 * 2048 + 1])
def test_dump_at_the_change_of_prefix_sums(dev, w, n):
    keys = W.distinct_keys(n, w, seed=5 + w)
    with gx.Table(w, 16, 2 * n, max_hashes=64) as t:
        _fill(t, keys, dev)
        assert np.array_equal(t.dump(), _rows(keys))
