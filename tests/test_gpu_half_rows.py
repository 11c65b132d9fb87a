"""Float32 builds whose Gram blocks come from a half-precision copy of the rows.  The copy only decides what lies beyond its
error bound, so graphs, stored distances and counts must be the pair-at-a-time kernel's, whatever the rows: far from the
origin, tiny, huge, of very different sizes, repeated, not finite."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N = 33_000      # one scan launch for lists of 33 .. 96 slots, two otherwise
KINDS = ["plain", "centre 1e3", "centre 1e6", "scale 1e-30", "scale 1e-20", "scale 1e15", "sizes", "tight", "two places", "outlier", "copies", "zeros", "nan", "inf"]


@pytest.fixture(scope="module")
def rn():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2310_20419_amd as m
    m.load_library()
    return m


def _rows(kind, d, N=N):
    import torch
    g = np.random.default_rng(11)
    X = (g.normal(size=(64, d))[g.integers(0, 64, size=N)] + 0.5 * g.normal(size=(N, d))).astype(np.float32)
    if kind.startswith("centre"):
        X = X + np.float32(kind.split()[1])
    elif kind.startswith("scale"):
        X = X * np.float32(kind.split()[1])
    elif kind == "sizes":                          # norms over twelve binades
        X = X * np.exp2(g.integers(-6, 7, size=(N, 1))).astype(np.float32)
    elif kind == "tight":                          # clusters far smaller than the distances between them: rounds that read whole rows
        X = (g.normal(size=(512, d))[g.integers(0, 512, size=N)] + 0.003 * g.normal(size=(N, d))).astype(np.float32)
    elif kind == "two places":
        X[::2] += 1e4
    elif kind == "outlier":                        # rows the half-precision range does not hold
        X[::997] *= np.float32(1e12)
    elif kind == "copies":
        X = X[g.permutation(np.repeat(np.arange(330), N // 330))]
    elif kind == "zeros":
        X[::2] = 0
    elif kind in ("nan", "inf"):
        X[::1009, d // 2] = float(kind)
        X[1::1013, 0] = -float(kind)
    return torch.from_numpy(np.ascontiguousarray(X, dtype=np.float32)).cuda()


@pytest.mark.parametrize("d", [16, 33, 96, 100, 960])
@pytest.mark.parametrize("kind", KINDS)
def test_same_as_the_pair_at_a_time_kernel(rn, kind, d):
    import torch
    X = _rows(kind, d)
    _compare(rn, X, ((20, 96, 2, 2), (8, 16, 1, 2), (40, 128, 1, 2)))


@pytest.mark.parametrize("n,dtype", [(256, "f32"), (257, "f32"), (70_000, "f32"), (70_000, "f16"), (70_000, "bf16")])
def test_sizes_where_the_launches_change(rn, n, dtype):
    import torch
    for d, kind in ((32, "plain"), (100, "plain"), (320, "plain"), (48, "tight")):
        X = _rows(kind, d, n).to({"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[dtype])
        _compare(rn, X, ((20, 96, 2, 2), (40, 64, 1, 2)))


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("R", [16, 96])
def test_a_vertex_that_receives_thousands_of_edges(rn, dtype, R):
    """Row 0 is nearer to every other row than any two of those are to each other, so whatever is pruned is redirected to it:
    most of its edges arrive past its inbox, and past what its merge closes by itself."""
    import torch
    g = np.random.default_rng(3)
    X = g.normal(size=(6000, 96))
    X /= np.linalg.norm(X, axis=1, keepdims=True)
    X[0] = 0
    X = torch.from_numpy(X.astype(np.float32)).cuda().to({"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[dtype])
    try:
        rn.rnnd_set_kernel_variant(1)
        keys, deg = rn.rnnd_random_graph(X, 8, R, 4)
        ids = (keys[:, :8] >> 1) & 0x7FFFFFFF
        assert int((ids == 0).sum()) < 600
        # every list starts with row 0
        d0 = (X.double() ** 2).sum(1).float()
        own = (d0.view(torch.int32).long() << 32) | 1
        has = (ids == 0).any(1)
        keys[1:, 7][~has[1:]] = own[1:][~has[1:]]
        keys[1:, :8] = keys[1:, :8].sort(dim=1).values
    finally:
        rn.rnnd_set_kernel_variant(0)
    out = []
    for v in (1, 0):
        k, dg = keys.clone(), deg.clone()
        try:
            rn.rnnd_set_kernel_variant(v)
            st = rn.rnnd_update_neighbors(X, k, dg, R, 2)
            # one run per pass is the same round, through the launches of large inputs: classify, merge, compact
            k1, dg1 = keys.clone(), deg.clone()
            rn.rnnd_update_neighbors_blocks(X, k1, dg1, R, 1, 2)
            # a build in which row 0 is in one list of seven from the start
            small = X[:700].contiguous()
            out.append((k, dg, rn.rnnd_build_ex(small, R, R, 2, 2, 4), st.proposals[0], k1, dg1, rn.rnnd_build_blocks(small, R, R, 2, 2, 4, 1)))
        finally:
            rn.rnnd_set_kernel_variant(0)
    used = torch.arange(R, device="cuda")[None, :] < out[0][1][:, None]
    assert torch.equal(out[0][1], out[1][1]) and torch.equal(out[0][0][used], out[1][0][used])
    assert torch.equal(out[0][2][0], out[1][2][0]) and out[0][3] == out[1][3] > 30_000
    assert torch.equal(out[0][1], out[1][5]) and torch.equal(out[0][0][used], out[1][4][used])
    assert torch.equal(out[0][2][0], out[1][6][0]) and torch.equal(out[0][2][1], out[1][6][1])


def _compare(rn, X, settings):
    import torch
    N = len(X)
    for S, R, T1, T2 in settings:
        try:
            rn.rnnd_set_kernel_variant(1)
            want = rn.rnnd_build_ex(X, S, R, T1, T2, 5)
        finally:
            rn.rnnd_set_kernel_variant(0)
        got = rn.rnnd_build_ex(X, S, R, T1, T2, 5)
        used = torch.arange(R, device="cuda")[None, :] < want[1][:, None]
        bad = int((got[0] != want[0]).any(1).sum())
        assert bad == 0, "%d of %d rows differ, R = %d" % (bad, N, R)
        assert torch.equal(got[1], want[1]) and torch.equal(got[2][used], want[2][used])
        n = T1 * T2
        assert list(got[3].algo_evals[:n]) == list(want[3].algo_evals[:n])
        assert list(got[3].proposals[:n]) == list(want[3].proposals[:n])


@pytest.mark.parametrize("kind", ["plain", "centre 1e3", "tight"])
@pytest.mark.parametrize("n,d", [(1500, 4096), (600, 20_000)])
def test_long_rows(rn, n, d, kind):
    """The error of the norms that the tiles form grows with the length of a row, and the bound with it."""
    _compare(rn, _rows(kind, d, n), ((20, 96, 2, 3), (8, 16, 1, 2)))
