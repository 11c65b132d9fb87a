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
    elif kind == "far":      # far from the origin, next to the distances
        X = X + 200
    elif kind == "places":   # two of them, far apart
        X[::2] += 1e4
    elif kind == "outliers":
        X[::23] *= 1e3
    elif kind == "sizes":    # norms over twelve binades
        X = X * torch.exp2(torch.randint(-6, 7, (N, 1), device="cuda", generator=g).float())
    return X.contiguous()


def DTYPES():
    import torch
    return {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


def builds(rn, X, R):
    """The statistics of a synchronous build and of one in four runs per pass, both checked against the pair-at-a-time kernel."""
    import torch
    S, out = min(20, R // 2), []
    for f in (lambda: rn.rnnd_build_ex(X, S, R, 2, 4, 3), lambda: rn.rnnd_build_blocks(X, S, R, 2, 4, 3, 4)):
        got = f()
        try:
            rn.rnnd_set_kernel_variant(1)
            want = f()
        finally:
            rn.rnnd_set_kernel_variant(0)
        used = torch.arange(R, device="cuda")[None, :] < want[1][:, None]
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]) and torch.equal(got[2][used], want[2][used])
        assert list(got[3].algo_evals[:8]) == list(want[3].algo_evals[:8]) and want[3].group_scans == 0
        out.append(got[3])
    return out


@pytest.mark.parametrize("R", [32, 96, 128])
@pytest.mark.parametrize("kind,dtype", [("tight", "f32"), ("sizes", "f32"), ("far", "f16"), ("sizes", "f16"), ("far", "bf16"), ("sizes", "bf16")])
@pytest.mark.parametrize("n,d", [(20_000, 96), (70_000, 160), (140_000, 64)])
def test_rows_that_need_groups_get_them(rn, n, d, kind, dtype, R):
    """Launches of every width: lists of up to 32, 96 and 128 entries, all classes in one launch (R = 96, 65,536 vertices) and in
    two, vertices with too many undecided pairs finished by the scan (131,072 vertices) and in a launch of their own."""
    X = rows(kind, n, d).to(DTYPES()[dtype])
    whole, blocks = builds(rn, X, R)
    assert 1 <= whole.group_scans <= 8 and 1 <= blocks.group_scans <= 32


@pytest.mark.parametrize("R", [32, 96, 128])
@pytest.mark.parametrize("kind,dtype", [("places", "f32"), ("sizes", "f32"), ("outliers", "f32"), ("far", "f16"), ("sizes", "bf16"), ("outliers", "bf16")])
@pytest.mark.parametrize("n,d", [(8_192, 96), (140_000, 64)])
def test_the_first_round_knows(rn, n, d, kind, dtype, R):
    """A sample of the random graph's lists tells it: every round of the build takes groups, and every run."""
    X = rows(kind, n, d).to(DTYPES()[dtype])
    whole, blocks = builds(rn, X, R)
    assert whole.group_scans == 8 and blocks.group_scans >= (32 if n >= 40_000 else 1)


def test_the_first_round_of_a_step_call_knows(rn):
    X = rows("far", 20_000, 96).to(DTYPES()["f16"])
    keys, deg = rn.rnnd_random_graph(X, 20, 64, 4)
    assert [rn.rnnd_update_neighbors(X, keys, deg, 64, 1).group_scans for _ in range(2)] == [1, 1]
    X = rows("unit", 20_000, 96).to(DTYPES()["f16"])
    keys, deg = rn.rnnd_random_graph(X, 20, 64, 4)
    assert [rn.rnnd_update_neighbors(X, keys, deg, 64, 1).group_scans for _ in range(2)] == [0, 0]


@pytest.mark.parametrize("R", [32, 96, 128])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", [20_000, 140_000])
def test_rows_that_repeat(rn, n, dtype, R):
    """Ties in bulk: whatever form a scan takes it leaves vertices to the next one, in the scan or (140,000) in a launch of its own, lists of more
    than 96 entries to the pair-at-a-time kernel."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    X = rows("plain", n // 50, 64).repeat_interleave(50, 0)[torch.randperm(n // 50 * 50, device="cuda", generator=g)]
    builds(rn, X.contiguous().to(DTYPES()[dtype]), R)


@pytest.mark.parametrize("R", [32, 96, 128])
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
def test_ordinary_rows_stay_with_the_tiles(rn, dtype, R):
    for kind in ("plain", "unit"):
        assert [s.group_scans for s in builds(rn, rows(kind, 20_000, 96).to(DTYPES()[dtype]), R)] == [0, 0]


@pytest.mark.parametrize("n,d,R", [(1_200, 96, 96), (2_000, 96, 96), (5_000, 33, 48), (20_000, 96, 96)])
def test_rounds_with_little_to_do_decide_nothing(rn, n, d, R):
    """The last rounds before an AddReverseEdges call have a handful of active vertices: their few pairs say nothing about the
    form that suits the thousands of the next round."""
    for seed in range(4):
        st = rn.rnnd_build_ex(rows("unit", n, d, seed), 20, R, 4, 15, seed)[3]
        assert min(st.active[:60]) < 64 and st.group_scans == 0, (seed, list(st.active[:60]))
