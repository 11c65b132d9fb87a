"""The scans by tiles send the edges they redirect to their targets themselves, beyond a size (rows of more than 1,024 bytes, with the inboxes more
than 1.75 GB) a kernel after the scan does.  The pair-at-a-time kernel always leaves them to that kernel, and every form decides alike: the
graphs, the degrees and the number of redirected edges must be the same."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rn():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2310_20419_amd as m
    m.load_library()
    return m


def rows(n, d, dtype, seed):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    c = torch.rand(5, d, device="cuda", generator=g) * 160 + 40
    x = torch.empty(n, d, device="cuda", dtype=getattr(torch, dtype))
    for lo in range(0, n, 65536):
        hi = min(n, lo + 65536)
        y = c[torch.randint(0, 5, (hi - lo,), device="cuda", generator=g)] + 12 * torch.randn(hi - lo, d, device="cuda", generator=g)
        x[lo:hi] = (y.round().clamp(0, 255) if dtype == "uint8" else y / 64).to(x.dtype)
    return x


def launches_of(f):
    """f's result, and the names of the kernels it launched."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        out = f()
        torch.cuda.synchronize()
    return out, [e.name for e in p.events()]


def compare(rn, X, S, R, T1, T2, own=None):
    """own: whether the edges must have been scattered by the scans."""
    import torch
    out = []
    try:
        for variant in (0, 1):
            rn.rnnd_set_kernel_variant(variant)
            def build():
                return rn.rnnd_build_ex(X, S, R, T1, T2, 5, want_keys=False)
            if own is None:
                g, dg, _, st = build()
            else:
                (g, dg, _, st), names = launches_of(build)
                assert any("k_random_graph" in k for k in names), names
                assert any("k_scatter" in k for k in names) == (variant == 1 or not own), names
            out.append((g, dg, list(st.proposals[:T1 * T2])))
    finally:
        rn.rnnd_set_kernel_variant(0)
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1]) and out[0][2] == out[1][2]


# full random lists in five clusters: a list of S entries has almost all of them redirected at once, more than a wavefront has lanes where S is
# 90 or 120, to a handful of targets
@pytest.mark.parametrize("S,R", [(7, 8), (30, 32), (60, 64), (90, 96), (120, 128)])
@pytest.mark.parametrize("dtype,d", [("uint8", 32), ("uint8", 200), ("float32", 96), ("float16", 64), ("bfloat16", 33)])
def test_edges_arrive_whatever_the_width_of_the_lists(rn, dtype, d, S, R):
    compare(rn, rows(1500, d, dtype, S), S, R, 2, 3)


# lists of up to 32 entries of few rows: half the blocks for rows of up to 256 bytes, and from 4 rows for each byte on
@pytest.mark.parametrize("n,d", [(700, 128), (700, 129), (1_535, 192), (1_536, 192), (9, 4000)])
@pytest.mark.parametrize("R", [32, 128])
def test_short_lists_of_few_rows(rn, n, d, R):
    compare(rn, rows(n, d, "float32", 5), min(30, n - 1), R, 2, 3)


# rows whose norms lie over twelve binades take groups of 16 rows, from the first or the second round on, whose edges are walked after the scan: a wavefront has one or two
# vertices of 8,192, whatever the class, more of 60,000
@pytest.mark.parametrize("n", [8_192, 60_000])
@pytest.mark.parametrize("S,R", [(30, 32), (60, 64), (90, 96), (120, 128)])
@pytest.mark.parametrize("dtype", ["float32", "bfloat16"])
def test_edges_of_groups_arrive(rn, dtype, n, S, R):
    import torch
    X = rows(n, 64, dtype, S)
    X = (X.float() * torch.exp2((torch.arange(n, device="cuda") % 13 - 6).float())[:, None]).to(X.dtype)
    compare(rn, X, S, R, 1, 3)
    assert rn.rnnd_build_ex(X, S, R, 1, 3, 5, want_keys=False)[3].group_scans >= 2


# rows of up to 1,024 bytes: always; longer ones up to 1.75e9 / (1088 + 512) = 1,093,750 rows of 1,088 bytes, / (16384 + 512) = 103,574 of 16,384
@pytest.mark.parametrize("dtype,n,d,own", [("uint8", 1_302_084, 784, True), ("uint8", 1_200_000, 1024, True),
                                           ("uint8", 1_093_750, 1025, True), ("uint8", 1_093_751, 1025, False),
                                           ("float32", 1_150_000, 512, True), ("bfloat16", 1_093_751, 544, False),
                                           ("float16", 103_574, 8192, True), ("float16", 103_575, 8192, False), ("float32", 103_575, 8192, False)])
def test_either_side_of_the_line(rn, dtype, n, d, own):
    compare(rn, rows(n, d, dtype, 3), 6, 32, 1, 2, own)


# streamed uint8 rows, lists of up to 128 entries: up to 49,152 rows; and each launch that leaves its edges, of all classes (up to 524,288 rows), of the short
# and the longer lists (up to 2,097,152), of every class
@pytest.mark.parametrize("n,d,S,R,own", [(49_152, 129, 120, 128, True), (49_153, 129, 120, 128, False), (524_289, 129, 100, 128, False),
                                         (2_097_153, 129, 20, 128, False), (1_093_751, 1025, 40, 64, False), (1_093_751, 1025, 70, 96, False)])
def test_streamed_bytes_in_long_lists(rn, n, d, S, R, own):
    compare(rn, rows(n, d, "uint8", 4), S, R, 1, 2, own)


# beyond the line: what the scans leave in props, for every width of the lists
@pytest.mark.parametrize("S,R", [(7, 8), (30, 32), (60, 64), (90, 96), (120, 128)])
@pytest.mark.parametrize("dtype,n,d", [("uint8", 106_000, 16000), ("float32", 103_600, 8192), ("bfloat16", 103_600, 8192)])
def test_edges_left_to_the_kernel_after_the_scan(rn, dtype, n, d, S, R):
    compare(rn, rows(n, d, dtype, S), S, R, 1, 2, False)
