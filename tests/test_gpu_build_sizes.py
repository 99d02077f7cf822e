"""CSR construction at the sizes where its ways part: the bucketed one for small lists (ranges of 256 ids or
fewer, ranges of one id, ranges too full for it), the general one, and the two shapes of its sort."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2511_20564_amd.device as d
    d.B.load_library()
    return d


def pairs(n_users, n_items, n_edges, seed, hot_users=None, hot_items=None):
    rng = np.random.default_rng(seed)
    u = rng.integers(0, hot_users or n_users, n_edges, dtype=np.int32)
    i = rng.integers(0, hot_items or n_items, n_edges, dtype=np.int32)
    return u, i


@pytest.mark.parametrize("n_users,n_items,n_edges,hot_users,hot_items", [
    (1, 1, 3, None, None),                        # one-bit ids
    (255, 257, 4096, None, None),                 # exactly one tile; ranges of one id, of two
    (256, 256, 4097, None, None),
    (3000, 5, 9000, None, None),                  # fewer items than ranges
    (70_001, 20_011, 300_000, None, None),
    (100_000, 50_000, 20_000, 100, None),         # a range of users with more pairs than fit: the general way
    (100_000, 50_000, 8_192, 100, None),          # exactly as many as fit
    (60_000, 70_000, 60_000, None, 3),            # ranges of items of many tiles
    (1 << 20, 1 << 12, 1 << 20, None, None),      # the largest bucketed list, the widest ranges
    ((1 << 20) + 1, 4000, 50_000, None, None),    # ids too wide for buckets
    (90_000, 40_000, (1 << 20) + 1, None, None),  # one pair too many for buckets
    (200_000, 90_000, 4 << 20, None, None),       # the large sort
])
def test_csr_matches_the_oracle(dev, oracle, n_users, n_items, n_edges, hot_users, hot_items):
    u, i = pairs(n_users, n_items, n_edges, n_edges + n_users, hot_users, hot_items)
    row_ptr, col = oracle.build_csr(n_users, n_items, u, i)
    ud, id_ = torch.from_numpy(u).cuda(), torch.from_numpy(i).cuda()
    for loops in (True, False):
        print(n_users, n_items, n_edges, loops, flush=True)
        g = dev.build_graph(n_users, n_items, ud, id_, add_self_loops=loops)
        rp, ci = g.row_ptr.cpu().numpy(), g.col_idx.cpu().numpy()
        if loops:
            assert np.array_equal(rp, row_ptr) and np.array_equal(ci, col)
        else:
            rows = np.repeat(np.arange(n_users + n_items), np.diff(row_ptr))
            off = col != rows
            assert np.array_equal(ci, col[off]) and np.array_equal(np.diff(rp), np.diff(row_ptr) - 1)


def test_bad_id_in_a_bucketed_list(dev):
    u, i = pairs(5000, 3000, 10_000, 3)
    for bad in ((7777, 5000), (9999, -1)):
        b = u.copy()
        b[bad[0]] = bad[1]
        with pytest.raises(dev.B.E2egError) as e:
            dev.build_graph(5000, 3000, torch.from_numpy(b).cuda(), torch.from_numpy(i).cuda())
        assert e.value.status == dev.B.E2EG_ERR_BAD_INDEX
