"""CSR construction of long lists by 32-bit keys, at the edges of its rule and of its tiles: ids of the widest
ranges, one item or user range, segments of the leading digit that are empty, one tile or one key, repeats
across tiles, and the list that is just too wide for it.  Checked against numpy: the lists are too long for
the oracle's comparisons of every option."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

LARGE = 4 << 20


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2511_20564_amd.device as d
    d.B.load_library()
    return d


def expected(n_users, n_items, u, i):
    """Row pointers and columns of the symmetrised structure without self-loops."""
    key = np.unique(u.astype(np.int64) * n_items + i)
    users, items = key // n_items, key % n_items
    turned = np.argsort(items, kind="stable")
    col = np.concatenate([items + n_users, users[turned]])
    row_ptr = np.zeros(n_users + n_items + 1, dtype=np.int64)
    np.cumsum(np.bincount(np.concatenate([users, items + n_users]), minlength=n_users + n_items), out=row_ptr[1:])
    return row_ptr, col


@pytest.mark.parametrize("n_users,n_items,n_edges,hot_users,hot_items", [
    (1 << 20, 1 << 20, LARGE, None, None),            # 40 bits together: the widest
    ((1 << 20) + 1, 1 << 20, LARGE, None, None),      # 41: the 64-bit way
    (1 << 23, 1 << 17, LARGE + 8191, None, None),     # user ids without pairs, a tile one key short
    (300, 1 << 22, LARGE + 1, None, None),            # two ids to a leading digit of the user
    (200, 300_000, LARGE, None, None),                # a leading digit that is the whole id
    (250_000, 1, LARGE, None, None),                  # one item: one segment of items
    (250_000, 2, LARGE + 5, None, None),
    (500_000, 513, LARGE, None, None),
    (1 << 20, 1 << 18, LARGE + 70_000, 4097, None),   # all pairs in the first segments of users: most are empty
    (700_001, 300_007, LARGE + 12345, None, 40),      # items of many tiles, most segments empty
    (2000, 500, 6_000_000, None, None),               # nearly all pairs repeated, runs of equal keys across tiles
])
def test_long_lists(dev, n_users, n_items, n_edges, hot_users, hot_items):
    rng = np.random.default_rng(n_edges + n_users + n_items)
    u = rng.integers(0, hot_users or n_users, n_edges, dtype=np.int32)
    i = rng.integers(0, hot_items or n_items, n_edges, dtype=np.int32)
    row_ptr, col = expected(n_users, n_items, u, i)
    print(n_users, n_items, n_edges, flush=True)
    g = dev.build_graph(n_users, n_items, torch.from_numpy(u).cuda(), torch.from_numpy(i).cuda(), add_self_loops=False)
    assert np.array_equal(g.row_ptr.cpu().numpy(), row_ptr)
    assert np.array_equal(g.col_idx.cpu().numpy(), col)
    g = dev.build_graph(n_users, n_items, torch.from_numpy(u).cuda(), torch.from_numpy(i).cuda())
    n = n_users + n_items
    rp, ci = g.row_ptr.cpu().numpy(), g.col_idx.cpu().numpy()
    assert np.array_equal(rp, row_ptr + np.arange(n + 1))
    rows = np.repeat(np.arange(n), np.diff(rp))
    assert np.array_equal(ci[ci != rows], col)


@pytest.mark.parametrize("where,user,item", [(0, -1, 5), (LARGE - 1, 5, 100_000), (8192, 600_000, 3)])
def test_bad_id_in_a_long_list(dev, where, user, item):
    rng = np.random.default_rng(7)
    u = rng.integers(0, 600_000, LARGE, dtype=np.int32)
    i = rng.integers(0, 100_000, LARGE, dtype=np.int32)
    u[where], i[where] = user, item
    with pytest.raises(dev.B.E2egError) as e:
        dev.build_graph(600_000, 100_000, torch.from_numpy(u).cuda(), torch.from_numpy(i).cuda())
    assert e.value.status == dev.B.E2EG_ERR_BAD_INDEX
