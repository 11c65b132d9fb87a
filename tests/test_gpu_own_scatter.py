"""The scans by tiles send the edges they redirect to their targets themselves, beyond a size (rows and inboxes of more than 1.75 GB,
rows streamed) a kernel after the scan does.  The pair-at-a-time kernel always leaves them to that kernel, and every form decides alike: the
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


def compare(rn, X, S, R, T1, T2):
    import torch
    out = []
    try:
        for variant in (0, 1):
            rn.rnnd_set_kernel_variant(variant)
            g, dg, _, st = rn.rnnd_build_ex(X, S, R, T1, T2, 5, want_keys=False)
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


# 1.75e9 / (832 + 512) = 1,302,083 rows of 784 bytes
@pytest.mark.parametrize("n", [1_302_083, 1_302_084])
def test_either_side_of_the_line(rn, n):
    compare(rn, rows(n, 784, "uint8", 3), 6, 32, 1, 2)
