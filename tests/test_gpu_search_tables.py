"""The size of a search's table of evaluated vertices follows from L, K, the row length, the number of vertices and the
number of queries: one case on either side of each line, on built graphs (tables that hold a query) and on random ones
(tables that overflow).  Results, distances and evaluation counts must be the oracle's."""
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


# up to 1,024 queries a team or a table of 8,192; 1,025 .. about 2,000 all resident with 4,096 slots; 4,000 with 2,048; more: the
# smallest table that holds what is expected.  L on either side of 1,024 / 2,048 slots and of the bitmap alone
@pytest.mark.parametrize("nq", [1024, 1025, 4100, 9000])
@pytest.mark.parametrize("kind,d", [("gauss_u8", 32), ("unit_f32", 40), ("unit_f32", 33)])
def test_tables_on_a_built_graph(rn, oracle_mod, kind, d, nq):
    X = wl.custom(kind, 4000, d, 5)
    Q = wl.custom(kind, nq, d, 6)
    graph, degree = built(rn, X, 12, 64, 2, 5)
    for L, K in ((16, 32), (20, 32), (21, 32), (48, 48), (71, 32), (72, 32), (105, 32), (106, 32), (119, 24), (120, 32), (128, 64)):
        if nq > 1025 and L not in (20, 21, 71, 72, 119, 120):
            continue
        check(rn, oracle_mod, X, graph, degree, Q, L, K, 10, 77, "%s d %d nq %d L %d K %d" % (kind, d, nq, L, K))


@pytest.mark.parametrize("n", [262_144, 262_145])
@pytest.mark.parametrize("nq", [1025, 6000])
def test_tables_that_overflow(rn, oracle_mod, n, nq):
    import torch
    X = wl.custom("gauss_u8", n, 32, 4)
    Q = wl.custom("gauss_u8", nq, 32, 5)
    g = np.random.default_rng(4).integers(0, n, size=(n, 40)).astype(np.int32)
    graph, degree = torch.from_numpy(g).cuda(), torch.full((n,), 40, dtype=torch.int32, device="cuda")
    for L, K in ((18, 36), (32, 40)):
        check(rn, oracle_mod, X, graph, degree, Q, L, K, 10, 5, "n %d nq %d L %d K %d" % (n, nq, L, K))
