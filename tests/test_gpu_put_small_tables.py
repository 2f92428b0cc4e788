"""Find-or-put of many more keys than the table has slots or buckets: keys
meet in a bucket by the hundred, claims are made in turns, and what is already
stored is found as fast as in a table with room."""
import numpy as np
import pytest
import torch

import paper_1801_05857_amd as gx
import workloads as W

pytestmark = pytest.mark.gpu


def _keys(n, distinct, w, seed):
    base = W.distinct_keys(distinct, w, seed)
    pick = np.random.default_rng(seed).integers(0, distinct, n)
    return base[pick], pick


@pytest.mark.parametrize("w", [1, 2, 3, 4])
@pytest.mark.parametrize("B,G", [(4, 4), (16, 4), (32, 8), (32, 4)])
@pytest.mark.parametrize("buckets,n,distinct", [(1, 4096, 3), (1, 70001, 40), (7, 1 << 17, 20),
                                                (64, 1 << 18, 200), (64, 1 << 18, 5000),
                                                (2048, 1 << 19, 3000)])
def test_many_keys_few_buckets(w, B, G, buckets, n, distinct):
    """A key is stored by one of its occurrences and found by the others, or
    refused by all of them."""
    keys, pick = _keys(n, distinct, w, 7 * w + B)
    slots = buckets * (B // (4 if w == 3 else w))
    with gx.Table(w, B, slots, subgroup=G, max_hashes=4) as t:
        dev = torch.from_numpy(keys.view(np.int32)).cuda()
        status = torch.full((n,), 99, dtype=torch.uint8, device="cuda")
        n_new = torch.zeros(1, dtype=torch.int64, device="cuda")
        t.find_or_put(dev, status, n_new)
        st = status.cpu().numpy()
        new, seen, full = (np.bincount(pick[st == k], minlength=distinct) for k in (1, 0, 2))
        assert set(np.unique(st)) <= {0, 1, 2}
        here = np.bincount(pick, minlength=distinct) > 0
        assert (new <= 1).all() and ((new == 1) == (here & (full == 0))).all()
        assert (seen[full > 0] == 0).all()
        stored = W.distinct_keys(distinct, w, 7 * w + B)[new == 1]
        want = stored[np.lexsort(stored.T[::-1])]
        assert np.array_equal(t.dump(), want)
        s = t.stats()
        assert (s.stored, s.lookups, s.full) == (new.sum(), n, full.sum()) == (
            int(n_new.item()), n, (st == 2).sum())
        # again: nothing is new, what was refused still is
        t.find_or_put(dev, status, n_new)
        again = status.cpu().numpy()
        assert ((again == 2) == (st == 2)).all() and not (again == 1).any()


def test_found_keys_do_not_wait_for_buckets():
    """2^19 lookups in 128 buckets against the same in 2^15: the device is as
    busy with either (times of a launch, the best of several)."""
    best = []
    for buckets in (128, 1 << 15):
        keys, _ = _keys(1 << 19, 1024, 2, 5)
        with gx.Table(2, 32, buckets * 16, subgroup=8) as t:
            dev = torch.from_numpy(keys.view(np.int32)).cuda()
            status = torch.zeros(len(keys), dtype=torch.uint8, device="cuda")
            n_new = torch.zeros(1, dtype=torch.int64, device="cuda")
            for _ in range(3):
                t.find_or_put(dev, status, n_new)
            times = []
            for _ in range(9):
                a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                a.record()
                for _ in range(4):
                    t.find_or_put(dev, status, n_new)
                b.record()
                torch.cuda.synchronize()
                times.append(a.elapsed_time(b) / 4)
            best.append(min(times))
    # (0.009 and 0.010 ms; few workgroups for few buckets took 1.5 ms)
    assert best[0] < 10 * best[1], best
