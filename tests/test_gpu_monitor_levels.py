"""A safety monitor over many levels: violations at the ends and in the middle
of a string of level launches, on levels of one state and of several
workgroups, with levels that go to the host in between, against the levels
known from the network's form."""
import numpy as np
import pytest

import paper_1801_05857_amd as gx
import workloads as W

from test_gpu_levels import _gpu, _star  # noqa: F401

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

TAIL = 50


def _wide_star(width, idle):
    """_star(width, TAIL) beside `idle` processes of 256 states that never
    move: the state of level k, chain i is local state 1 + i + width (k - 1)."""
    star = _star(width, TAIL)
    return W._net([star.n_states[0]] + [256] * idle, [0] * (1 + idle),
                  [star.trans[0]] + [[]] * idle, 1, np.zeros((0, 1 + idle)), "wide_star")


@pytest.mark.parametrize("width,idle", [(1, 0), (7, 3), (700, 3), (64, 9)])
@pytest.mark.parametrize("bad", [[], [0], [1], [15], [16], [17], [33, 34], [50], [0, 3, 40]])
@pytest.mark.parametrize("opts", [{}, {"slice_states": 65}, {"frontier_capacity": 1 << 17}])
def test_violations_by_level(width, idle, bad, opts):
    net = _wide_star(width, idle)
    flags = np.zeros(net.n_states[0], dtype=np.uint8)
    for k in bad:  # every other chain's state of that level
        flags[0 if k == 0 else slice(1 + width * (k - 1), 1 + width * k, 2)] = 1
    per = {k: 1 if k == 0 else (width + 1) // 2 for k in bad}
    words = gx.network_words(net)
    with gx.Table(words, 16, 4 * (1 + width * TAIL), max_hashes=64) as t:
        for stop in (False, True, False):
            t.clear()
            got = gx.explore(net, t, monitor=(0, flags), stop_on_violation=stop, **opts)
            last = min(bad) if stop and bad else TAIL
            assert got.levels.tolist() == [1] + [width] * last
            assert got.violation_level == (min(bad) if bad else None)
            hit = [min(bad)] if stop and bad else bad
            assert len(got.violations) == sum(per[k] for k in hit)
            local = np.flatnonzero(flags[:1 + width * last])
            packed = gx.network_pack(net, np.stack([local] + [0 * local] * idle, axis=1))
            assert got.violations.tolist() == sorted(packed.tolist())
