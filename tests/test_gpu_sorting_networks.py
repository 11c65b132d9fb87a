"""The sorts of the merges and of the search at every width they come in (16, 32, 64, 128 and 256 keys), on keys of which many have equal
distances, so that the low halves decide: graphs and search results must be those of the oracle in every entry."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rn():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2310_20419_amd as m
    m.load_library()
    return m


def rows(n, values, seed):
    """Bytes of few values: distances are small whole numbers, most of them shared by many pairs."""
    return np.random.default_rng(seed).integers(0, values, (n, 32), dtype=np.uint8)


# lists of up to 8 .. 128 entries; two values and 600 rows make hubs whose received edges overflow their inboxes
@pytest.mark.parametrize("n,values", [(600, 2), (600, 7), (3000, 2)])
@pytest.mark.parametrize("S,R", [(5, 8), (12, 16), (20, 33), (31, 64), (40, 65), (60, 96), (100, 128)])
def test_merges_of_tied_keys(rn, n, values, S, R):
    import oracle
    import torch
    X = rows(n, values, S)
    g, d, _, _ = rn.rnnd_build_ex(torch.from_numpy(X).cuda(), S, R, 2, 4, 11)
    want = oracle.build_sync(X, S, R, 2, 4, 11)
    assert (d.cpu().numpy() == want.snap.deg).all() and (g.cpu().numpy() == want.snap.ids).all()


@pytest.mark.parametrize("L,K", [(3, 8), (16, 16), (40, 17), (64, 33), (65, 64), (128, 96)])
@pytest.mark.parametrize("dtype", ["uint8", "float32"])
def test_searches_of_tied_keys(rn, dtype, L, K):
    import oracle
    import torch
    X, Q = rows(2000, 3, 1).astype(dtype), rows(37, 3, 2).astype(dtype)
    Xd = torch.from_numpy(X).cuda()
    g, d = rn.rnnd_build(Xd, 20, 96, 2, 4, 5)
    ids, _, evals = rn.rnnd_search(Xd, g, d, torch.from_numpy(Q).cuda(), L, K, min(L, 10), 7)
    want, want_evals = oracle.search(X, g.cpu().numpy(), d.cpu().numpy(), Q, L, K, min(L, 10), 7)
    assert (ids.cpu().numpy() == want).all() and evals == want_evals
