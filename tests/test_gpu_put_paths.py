"""GPU parity of find-or-put on both sides of the line between its two kernels
(4-lane subgroups with every key in flight; wider subgroups), and where
4-lane subgroups meet: pieces of wide buckets, full buckets, many keys of one
bucket at once.  The result of a call is a set and one NEW per absent key, so
every comparison is exact."""
import numpy as np
import pytest

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


def _put(table, keys, dev):
    k = torch.from_numpy(np.ascontiguousarray(keys).view(np.int32)).to(dev)
    st = torch.full((keys.shape[0],), 255, dtype=torch.uint8, device=dev)
    n_new = torch.zeros(1, dtype=torch.int64, device=dev)
    table.find_or_put(k, st, n_new)
    return st.cpu().numpy(), int(n_new.item())


def _rows(keys):
    return keys[np.lexsort(keys.T[::-1])]


# launches of more keys than one per lane, for every subgroup width that has a
# kernel of its own, and the last one below the line
@pytest.mark.parametrize("w,B,G", [(1, 32, 8), (2, 16, 8), (2, 32, 16), (3, 16, 16), (4, 32, 8),
                                   (1, 64, 64), (2, 32, 32), (4, 64, 16), (2, 16, 4), (3, 32, 4)])
@pytest.mark.parametrize("extra", [0, 1])
def test_line_between_kernels(dev, w, B, G, extra):
    cus = torch.cuda.get_device_properties(dev).multi_processor_count
    n = 2048 * cus + extra
    keys = W.distinct_keys(n, w, seed=31 + w)
    with gx.Table(w, B, 2 * n, subgroup=G, max_hashes=64) as t:
        st, n_new = _put(t, keys, dev)
        assert n_new == n and (st == gx.GX_NEW).all()
        order = W.permutation(n, 5).astype(np.int64)
        st, n_new = _put(t, keys[order], dev)
        assert n_new == 0 and (st == gx.GX_SEEN).all()
        assert np.array_equal(t.dump(), _rows(keys))
        s = t.stats()
        assert (s.stored, s.lookups, s.full, s.invalid) == (n, 2 * n, 0, 0)


# one bucket (and two), filled to its last slot by keys that all arrive at
# once, each several times; one key more than fits is FULL
@pytest.mark.parametrize("w", [1, 2, 3, 4])
@pytest.mark.parametrize("B", [4, 8, 16, 32, 64])
def test_one_bucket(dev, w, B):
    S = 4 if w == 3 else w
    slots = B // S
    keys = W.distinct_keys(slots, w, seed=7)
    with gx.Table(w, B, 1, subgroup=8, max_hashes=1) as t:
        st, n_new = _put(t, np.tile(keys, (257, 1)), dev)
        assert n_new == slots == int((st == gx.GX_NEW).sum())
        assert set(np.unique(st).tolist()) <= {gx.GX_NEW, gx.GX_SEEN}
        assert np.array_equal(t.dump(), _rows(keys))
        more = W.distinct_keys(slots + 1, w, seed=7)
        st, n_new = _put(t, more, dev)
        assert n_new == 0 and (st[:slots] == gx.GX_SEEN).all() and st[slots] == gx.GX_FULL


# fills that pass from the first piece of a 32-word bucket to its second and
# on to the next bucket, word 0xFFFFFFFF refused, in calls of every size
@pytest.mark.parametrize("w,B", [(1, 32), (2, 32), (4, 32), (3, 16)])
@pytest.mark.parametrize("n", [1, 3, 63, 64, 65, 257, 5000])
def test_rest_of_a_fill(dev, w, B, n):
    S = 4 if w == 3 else w
    keys = W.distinct_keys(n, w, seed=n)
    bad = np.full((2, w), 5, np.uint32)
    bad[:, w - 1] = 0xFFFFFFFF
    with gx.Table(w, B, max(B // S, int(n / 0.9)), subgroup=4, max_hashes=256) as t:
        st, n_new = _put(t, np.concatenate([keys, bad]), dev)
        assert n_new == n and (st[:n] == gx.GX_NEW).all() and (st[n:] == gx.GX_INVALID).all()
        st, n_new = _put(t, keys[::-1].copy(), dev)
        assert n_new == 0 and (st == gx.GX_SEEN).all()
        assert np.array_equal(t.dump(), _rows(keys))
        assert t.stats().invalid == 2
