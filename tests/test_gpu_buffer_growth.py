"""The device buffers of explorations and dumps: small models in large tables
take little memory beside the table, and levels, deadlocks and violations
beyond the first buffers make them grow in the middle of an exploration."""
import numpy as np
import pytest
import torch

import oracle
import paper_1801_05857_amd as gx
import workloads as W

from test_gpu_levels import _star

pytestmark = pytest.mark.gpu


def _used():
    torch.cuda.synchronize()
    free, total = torch.cuda.mem_get_info()
    return total - free


@pytest.mark.parametrize("monitor", [False, True])
def test_small_model_in_a_large_table(monitor):
    """4096 states, a table of 256 MiB: 2^26 slots."""
    net = W.tiny_cycles()
    mon = (0, np.arange(8) % 2) if monitor else None
    with gx.Table(1, 32, 1 << 20) as t:  # (kernels are loaded before anything is measured)
        gx.explore(net, t, monitor=mon)
    with gx.Table(1, 32, 1 << 26) as t:
        before = _used()
        assert gx.explore(net, t, monitor=mon).n_states == 4096
        assert _used() - before <= 16 << 20


def test_dump_keeps_no_lists():
    n = 1 << 22
    keys = torch.from_numpy(W.distinct_keys(n, 4, 3).view(np.int32)).cuda()
    status = torch.zeros(n, dtype=torch.uint8, device="cuda")
    with gx.Table(4, 16, 2 * n, max_hashes=64) as t:
        t.find_or_put(keys, status)
        before = _used()
        first = t.dump()
        assert len(first) == n and np.array_equal(t.dump(), first)
        # (two lists of 64 MiB; the sort's own workspace is 2 MiB)
        assert _used() - before <= 16 << 20


@pytest.mark.parametrize("opts", [{}, {"local_dedup": True}, {"slice_states": 5000}])
@pytest.mark.parametrize("slots", [0, 1 << 25])  # (2^25 slots are 512 MiB: buffers grow by need)
def test_levels_and_violations_outgrow_the_buffers(opts, slots):
    """Hundreds of thousands of states, levels of tens of thousands with tens
    of successors a state, half of them violating; explored twice."""
    net = W.large_random_network(4)
    want = oracle.explore(net, want_visited=True)
    bad = np.zeros(64, np.uint8)
    locals0 = want.visited[:, 0] & 63  # process 0: the first six bits
    hit = np.unique(locals0)[:2]
    bad[hit] = 1
    expect = want.visited[np.isin(locals0, hit)]
    assert len(expect) > 1 << 16 and want.levels.max() > 1 << 14
    with gx.Table(want.words, 16, slots or 2 * want.n_states, max_hashes=64) as t:
        before = _used()
        for _ in range(2):
            t.clear()
            got = gx.explore(net, t, monitor=(0, bad), **opts)
            # (no buffer of a large table's size)
            assert slots == 0 or _used() - before < 384 << 20
            assert got.levels.tolist() == want.levels.tolist()
            assert got.n_transitions == want.n_transitions
            assert np.array_equal(got.deadlocks, want.deadlocks)
            assert np.array_equal(got.violations, expect)
        assert np.array_equal(t.dump(), want.visited)


@pytest.mark.parametrize("width,tail", [(70_000, 3), (30_000, 7)])
@pytest.mark.parametrize("monitor", [False, True])
def test_more_deadlocks_and_violations_than_a_buffer(width, tail, monitor):
    """A star of chains: `width` deadlocks in the last level, every state of
    the monitored ones violating."""
    net = _star(width, tail)
    n = 1 + width * tail
    mon = (0, np.ones(n, np.uint8)) if monitor else None
    with gx.Table(1, 16, 4 * n, max_hashes=64) as t:
        for _ in range(2):
            t.clear()
            got = gx.explore(net, t, monitor=mon)
            assert got.levels.tolist() == [1] + [width] * tail
            assert len(got.deadlocks) == width
            if monitor:
                assert got.violation_level == 0
                assert got.violations[:, 0].tolist() == list(range(n))
