"""The ways a search is launched: a team of wavefronts per query where there are few queries, one wavefront where there
are many; a table of evaluated vertices that overflows into the bitmap, or the bitmap alone; every row length's way of
evaluating.  Results, distances and evaluation counts must be the oracle's."""
import numpy as np
import pytest

import workloads as wl
from test_gpu_search import built, check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rn():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2310_20419_amd as m
    m.load_library()
    return m


# rows of at most 128, at most 512 and more bytes; rows that cannot be read in 16-byte pieces; queries too long for LDS
@pytest.mark.parametrize("kind,d", [("gauss_u8", 32), ("heavy_u8", 128), ("heavy_u8", 144), ("heavy_u8", 784), ("gauss_u8", 33),
                                    ("unit_f32", 32), ("unit_f32", 100), ("unit_f32", 132), ("unit_f32", 101), ("beta_f32", 960),
                                    ("unit_f32", 8000), ("unit_f32", 8001)])
@pytest.mark.parametrize("nq", [9, 1500])      # a team per query; one wavefront per query, several queries each
def test_row_lengths_and_team_sizes(rn, oracle_mod, kind, d, nq):
    X = wl.custom(kind, 900 if d > 1000 else 2500, d, 5)
    Q = wl.custom(kind, nq if d < 500 else 9 if nq < 100 else 1030, d, 6)
    graph, degree = built(rn, X, 10, 48, 2, 4)
    for L, K in ((20, 12), (64, 32)) if d < 500 else ((33, 16),):
        check(rn, oracle_mod, X, graph, degree, Q, L, K, 10, 77, "%s d %d nq %d L %d K %d" % (kind, d, nq, L, K))


@pytest.mark.parametrize("kind,d,L,K", [("unit_f32", 64, 30, 40), ("heavy_u8", 160, 24, 40), ("unit_f32", 64, 128, 90)])
@pytest.mark.parametrize("nq", [3, 1100])
def test_queries_that_outgrow_the_table(rn, oracle_mod, kind, d, L, K, nq):
    """Long random lists instead of a built graph: nearly every neighbour is new, so far more vertices are evaluated per
    place of the candidate list than on a finished index, and the table overflows into the bitmap."""
    import torch
    n, W = 30_000, 96
    X = wl.custom(kind, n, d, 8)
    Q = wl.custom(kind, nq, d, 9)
    g = np.random.default_rng(3).integers(0, n, size=(n, W)).astype(np.int32)      # duplicates within a row now and then
    graph, degree = torch.from_numpy(g).cuda(), torch.full((n,), W, dtype=torch.int32, device="cuda")
    check(rn, oracle_mod, X, graph, degree, Q, L, K, 10, 5, "%s d %d L %d K %d nq %d" % (kind, d, L, K, nq))


def test_short_rows_of_a_large_index_use_the_table(rn, oracle_mod):
    """Rows of at most 128 bytes and more than 262,144 vertices: the table, evaluated at once with the lookup."""
    import torch
    n = 270_000
    X = wl.custom("gauss_u8", n, 48, 4)
    Q = wl.custom("gauss_u8", 1300, 48, 5)
    g = np.random.default_rng(4).integers(0, n, size=(n, 40)).astype(np.int32)
    graph, degree = torch.from_numpy(g).cuda(), torch.full((n,), 40, dtype=torch.int32, device="cuda")
    for L, K in ((16, 10), (48, 40)):
        check(rn, oracle_mod, X, graph, degree, Q, L, K, 10, 5, "L %d K %d" % (L, K))
