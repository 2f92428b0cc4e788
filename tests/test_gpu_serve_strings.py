"""The exploration server's strings of steps: levels that outgrow a string of
eight and one of four steps in its middle, levels with a step a string, and
more requests admitted in one round than there are staging regions, with
results known from the networks' form."""
import math

import numpy as np
import pytest

import paper_1801_05857_amd as gx
import workloads as W

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _grid(P, n):
    """P processes of n states, every state a step to every other: level d
    holds the states that differ from the initial one in d processes."""
    trans = np.array([[s, 0, d] for s in range(n) for d in range(n) if s != d], np.uint32)
    net = W._net([n] * P, [0] * P, [trans] * P, 1, np.zeros((0, P)), f"grid_{P}x{n}")
    levels = [math.comb(P, d) * (n - 1) ** d for d in range(P + 1)]
    return net, levels, n ** P * P * (n - 1)


def _check(srv, request, levels, transitions):
    status, got, _ = srv.poll(request)
    assert status == gx.GX_OK
    assert got.levels.tolist() == levels
    assert got.n_states == sum(levels) and got.n_transitions == transitions
    assert len(got.deadlocks) == 0


# 2^26 states: levels of 1.25 M, 3.75 M (more than 2^21, in a string of eight
# steps), 8.4 M, 14 M, 16.9 M (more than 2^24, in one of four), 13.8 M and less
BIG = (13, 4)


def _widened(P, n, idle):
    """_grid(P, n) beside `idle` processes of 16 states that never move."""
    net, levels, trans = _grid(P, n)
    net = W._net([n] * P + [16] * idle, [0] * (P + idle), list(net.trans) + [[]] * idle, 1,
                 np.zeros((0, P + idle)), "widened")
    return net, levels, trans


@pytest.mark.parametrize("mixed", [False, True])
def test_levels_outgrow_their_string(mixed):
    """Alone, and with small requests of the same and of other slot widths
    that end before, in and after the large levels."""
    want = [_grid(*BIG)]
    if mixed:
        want += [_grid(1, 5), _grid(9, 3), _grid(6, 6), _grid(20, 2), _widened(3, 2, 9),
                 _widened(9, 3, 11), _widened(3, 4, 20)]
        assert {gx.network_words(net) for net, _, _ in want} == {1, 2, 3}
    with gx.Server(16 << 30, max_hashes=32, bucket_words=16, subgroup=4) as srv:
        for _ in range(2):
            ids = [srv.submit(net, sum(levels)) for net, levels, _ in want]
            for request, (_, levels, trans) in zip(ids, want):
                _check(srv, request, levels, trans)
        assert srv.stats()["failed"] == 0


def test_more_admissions_than_staging_regions():
    """Two requests hold the whole budget; 200 more wait and are admitted
    together, each with its own network."""
    big, big_levels, big_trans = _grid(*BIG)
    small = [_grid(P, n) for P, n in ((1, 2), (2, 3), (3, 4), (4, 5), (5, 3), (6, 2), (2, 31))]
    pick = np.random.default_rng(1).integers(0, len(small), 200)
    views = [gx.network_view(net) for net, _, _ in small]
    # a request of 2^26 states reserves 4 GiB at load 0.5
    with gx.Server(8 << 30, max_hashes=32, bucket_words=16, subgroup=4) as srv:
        first = [srv.submit(big, 1 << 26) for _ in range(2)]
        ids = [srv.submit(views[k], sum(small[k][1])) for k in pick]
        for request in first:
            _check(srv, request, big_levels, big_trans)
        for request, k in zip(ids, pick):
            _check(srv, request, *small[k][1:])
        s = srv.stats()
        assert s["failed"] == 0 and s["active_peak"] > 64
