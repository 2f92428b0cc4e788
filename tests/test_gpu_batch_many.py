"""Stepped batches of many small instances: a group's job is found by rounds of
as many probes as a workgroup has threads, so instance counts at the edges of
one and two rounds, with instances that end at different steps."""
import numpy as np
import pytest

import paper_1801_05857_amd as gx
import workloads as W

pytestmark = pytest.mark.gpu


def _cycle(n, copies):
    """`copies` independent cycles of n states: n ** copies states, level k
    holds those whose steps add up to k."""
    trans = np.array([[s, 0, (s + 1) % n] for s in range(n)], np.uint32)
    net = W._net([n] * copies, [0] * copies, [trans] * copies, 1, np.zeros((0, copies)), "cycles")
    levels = np.ones(1, np.int64)
    for _ in range(copies):
        levels = np.convolve(levels, np.ones(n, np.int64))
    return net, levels


SHAPES = [(2, 1), (3, 2), (5, 3), (17, 2), (40, 1), (9, 4), (4, 5)]


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 511, 513, 4097, 65537])
def test_instance_counts(n):
    shapes = SHAPES[:3] if n > 1000 else SHAPES
    built = [_cycle(*s) for s in shapes]
    views = [gx.network_view(net) for net, _ in built]
    pick = np.random.default_rng(n).integers(0, len(built), n)
    if n == 65537:
        pick[:] = 0
        pick[[0, 1, 32768, 65535, 65536]] = 2  # (the rest end after one step)
    caps = [2 * int(lv.sum()) + 64 for _, lv in built]
    with gx.Batch([views[k] for k in pick], [caps[k] for k in pick], bucket_words=8, subgroup=8,
                  max_hashes=32, max_levels=64) as b:
        for _ in range(2):
            b.run()
            for k, (status, r) in zip(pick, b.results()):
                (cycle, copies), levels = shapes[k], built[k][1]
                assert status == gx.GX_OK
                assert np.array_equal(r.levels, levels)
                assert r.n_transitions == copies * cycle ** copies and len(r.deadlocks) == 0
