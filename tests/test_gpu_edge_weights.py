"""Edge weights and the sampling table by tiles of entries: fewer entries than a search's last read, tiles of more
rows than fit in LDS (isolated nodes), either side the larger, rows of one tile and more, repeats."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_users,n_items,n_edges,hot", [
    (1, 1, 1, 1),
    (2, 1, 3, 1),                   # 5 or 6 entries
    (3000, 2000, 20, 10),           # nearly all nodes isolated: tiles of more than 1024 rows
    (5000, 700, 40_000, 700),       # more users: weights enter in the users' rows
    (700, 5000, 40_000, 5000),      # more items
    (40, 9000, 60_000, 9000),       # long rows on the smaller side
    (9000, 40, 60_000, 3),          # rows of several tiles
])
def test_weights_and_table(n_users, n_items, n_edges, hot):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2511_20564_amd.device as dev
    rng = np.random.default_rng(n_users + n_edges)
    u = rng.integers(0, n_users, n_edges, dtype=np.int32)
    i = rng.integers(0, hot, n_edges, dtype=np.int32)
    w = rng.uniform(0.1, 3.0, n_edges).astype(np.float32)
    w[rng.random(n_edges) < 0.1] = 0.0   # ignored
    print(n_users, n_items, n_edges, flush=True)
    g = dev.build_weighted_graph(n_users, n_items, *(torch.from_numpy(a).cuda() for a in (u, i, w)))
    rp, col, val = (t.cpu().numpy() for t in (g.row_ptr, g.col_idx, g.val))
    rows = np.repeat(np.arange(n_users + n_items), np.diff(rp))
    best = np.zeros((n_users, n_items), dtype=np.float32)
    np.maximum.at(best, (u, i), w)
    a, b = np.minimum(rows, col), np.maximum(rows, col) - n_users
    expect = np.where(rows == col, np.float32(1), best[np.minimum(a, n_users - 1), np.clip(b, 0, n_items - 1)])
    assert np.array_equal(val, expect)
    table = dev.sampler_table(g)[:8 * (g.nnz + 1)].view(torch.int64).cpu().numpy()
    p = np.where(rows == col, np.float32(0), val)
    top = np.zeros(n_users + n_items, dtype=np.float32)
    np.maximum.at(top, rows, p)
    with np.errstate(invalid="ignore", divide="ignore"):
        q = np.floor(p / top[rows] * np.float32(16777216.0))
    q = np.where(p > 0, np.maximum(q, 1), 0).astype(np.int64)
    assert np.array_equal(table, np.concatenate([[0], np.cumsum(q)]))
