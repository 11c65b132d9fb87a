"""Float rows on which the 32-row tiles decide too little are scanned in groups of 16 rows instead.  Which form a round takes is
decided on the device and changes no graph, so it is read from the statistics here: rows that need it must get it, others not."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rn():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2310_20419_amd as m
    m.load_library()
    return m


def rows(kind, N, d, seed=1):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)

    def normal(*shape):
        return torch.randn(*shape, device="cuda", generator=g)
    if kind == "tight":      # clusters far smaller than the distances between them
        return normal(512, d)[torch.randint(0, 512, (N,), device="cuda", generator=g)] + 0.003 * normal(N, d)
    X = normal(64, d)[torch.randint(0, 64, (N,), device="cuda", generator=g)] + 0.5 * normal(N, d)
    if kind == "unit":
        X = X / X.norm(dim=1, keepdim=True)
    return X.contiguous()


@pytest.mark.parametrize("n,d", [(20_000, 96), (70_000, 100), (140_000, 64)])
def test_rows_that_need_groups_get_them(rn, n, d):
    st = rn.rnnd_build_ex(rows("tight", n, d), 20, 96, 2, 4, 3)[3]
    assert 1 <= st.group_scans <= 7
    assert rn.rnnd_build_ex(rows("plain", n, d), 20, 96, 2, 4, 3)[3].group_scans == 0


@pytest.mark.parametrize("n,d,R", [(1_200, 96, 96), (2_000, 96, 96), (5_000, 33, 48), (20_000, 96, 96)])
def test_rounds_with_little_to_do_decide_nothing(rn, n, d, R):
    """The last rounds before an AddReverseEdges call have a handful of active vertices: their few pairs say nothing about the
    form that suits the thousands of the next round."""
    for seed in range(4):
        st = rn.rnnd_build_ex(rows("unit", n, d, seed), 20, R, 4, 15, seed)[3]
        assert min(st.active[:60]) < 64 and st.group_scans == 0, (seed, list(st.active[:60]))
