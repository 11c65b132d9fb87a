"""A vertex that very many edges reach in one round: rows of any width, arrivals on either side of the inbox (32 slots for
rows of fewer than 32 entries, 64 for wider ones) and of a full set of late lists; and a hub on narrow rows must not cost
more than the same hub on wide ones."""
import numpy as np
import pytest

from gpu_util import assert_snapshot_equal, snapshot_to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rn():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2310_20419_amd as m
    m.load_library()
    return m


def _star(oracle, n, d, S, R, planted):
    """RandomGraph lists with vertex 0, the centre of the data, planted in the lists of vertices 1 .. planted."""
    g = np.random.default_rng(8)
    X = np.clip(128 + g.normal(0, 40, size=(n, d)), 0, 255).astype(np.uint8)
    X[0] = 128
    snap = oracle.random_graph(X, S, 5, R)
    for u in range(1, planted + 1):
        m = snap.deg[u]
        if 0 not in snap.ids[u, :m]:
            snap.ids[u, m - 1] = 0
            snap.dist[u, m - 1] = float(((X[u].astype(np.int64) - 128) ** 2).sum())
        order = np.lexsort((snap.ids[u, :m], snap.dist[u, :m]))
        snap.ids[u, :m], snap.dist[u, :m] = snap.ids[u, :m][order], snap.dist[u, :m][order]
    return X, snap


@pytest.mark.parametrize("R", [1, 3, 8, 24, 31, 32, 128])
@pytest.mark.parametrize("planted", [4, 10, 20, 35, 60, 400])
def test_arrivals_around_the_inbox(rn, oracle_mod, R, planted):
    import torch
    S = min(R, 8)
    X, snap = _star(oracle_mod, 900, 32, S, R, planted)
    Xd = torch.from_numpy(X).cuda()
    for t in range(3):
        keys, deg = snapshot_to_device(snap, False, R)
        snap, evals, props = oracle_mod.update_neighbors_sync(X, snap, R)
        st = rn.rnnd_update_neighbors(Xd, keys, deg, R, 1)
        assert st.algo_evals[0] == evals and st.proposals[0] == props
        assert_snapshot_equal(snap, False, keys, deg, "R %d planted %d round %d" % (R, planted, t))


def test_hub_on_narrow_rows_costs_no_more_than_on_wide_ones(rn):
    """20,000 lists name the centre, which then receives about 140,000 edges in one round; only the row width differs.
    The round takes about 4 ms; with fewer late lists for narrow rows it took four times as long."""
    import torch
    n, planted = 100_000, 20_000
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    X = (128 + 40 * torch.randn(n, 32, device="cuda", generator=g)).round().clamp(0, 255).to(torch.uint8)
    X[0] = 128
    ms = {}
    for R in (8, 32):
        keys, deg = rn.rnnd_random_graph(X, 8, R, 5)
        dist = ((X[1:planted + 1].int() - 128) ** 2).sum(1).long()
        keys[1:planted + 1, 7] = (dist << 32) | 1           # vertex 0, new
        keys[1:planted + 1, :8] = torch.sort(keys[1:planted + 1, :8], dim=1).values
        took = []
        for _ in range(5):
            k, e = keys.clone(), deg.clone()
            took.append(rn.rnnd_update_neighbors(X, k, e, R, 1).round_ms[0])
        ms[R] = min(took)
    assert ms[8] < 2 * ms[32], ms
