"""First levels whose limit is a state or a few: networks of very wide steps
and small frontiers leave the LDS launch the smallest rings it can have."""
import numpy as np
import pytest

import oracle
import paper_1801_05857_amd as gx
import workloads as W

pytestmark = pytest.mark.gpu


def _same(got, want, t):
    assert got.n_states == want.n_states
    assert got.n_transitions == want.n_transitions
    assert got.levels.tolist() == want.levels.tolist()
    assert np.array_equal(got.deadlocks, want.deadlocks)
    assert np.array_equal(t.dump(), want.visited)


@pytest.mark.parametrize("wide", [(33, 32), (40, 50), (64, 64)])  # 3, 2 and 1 states
def test_steps_of_many_successors(wide):
    """One rendezvous with wide[0] x wide[1] successors, and a way back."""
    trans = [np.array([[0, 0, d] for d in range(k)] + [[s, 1, 0] for s in range(1, k)], np.uint32)
             for k in wide]
    net = W._net(list(wide), [0, 0], trans, 2, np.array([[0, 0]], np.int32), "wide")
    want = oracle.explore(net, want_visited=True)
    with gx.Table(want.words, 16, 2 * want.n_states, max_hashes=64) as t:
        _same(gx.explore(net, t), want, t)


@pytest.mark.parametrize("capacity", [1, 2, 3, 4, 7])
@pytest.mark.parametrize("length", [3, 150])
def test_small_frontiers(capacity, length):
    """A cycle: levels of one state, limits of `capacity` states."""
    trans = [np.array([[s, 0, (s + 1) % length] for s in range(length)], np.uint32)]
    net = W._net([length], [0], trans, 1, np.zeros((0, 1), np.int32), "cycle")
    want = oracle.explore(net, want_visited=True)
    with gx.Table(want.words, 16, 4 * length, max_hashes=64) as t:
        _same(gx.explore(net, t, frontier_capacity=capacity), want, t)
