"""Up to 131,072 vertices a round's classify, merge and compact are one launch.  Block-sequential builds always take the three
separate ones, and one run per pass is the synchronous round, so the two must give the same graph."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rn():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2310_20419_amd as m
    m.load_library()
    return m


@pytest.mark.parametrize("dtype", ["u8", "f32"])
@pytest.mark.parametrize("n", [17, 127, 4096, 8191, 65_537, 131_072, 131_073])
def test_one_launch_and_three_give_the_same_graph(rn, n, dtype):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    c = torch.rand(64, 32, device="cuda", generator=g) * 192
    X = c[torch.randint(0, 64, (n,), device="cuda", generator=g)] + 20 * torch.randn(n, 32, device="cuda", generator=g)
    X = X.round().clamp(0, 255).to(torch.uint8) if dtype == "u8" else X
    for S, R in ((8, 12), (16, 96), (16, 128)):
        S = min(S, n - 1)
        want = rn.rnnd_build_blocks(X, S, R, 2, 3, 9, 1)
        got = rn.rnnd_build_ex(X, S, R, 2, 3, 9)
        used = torch.arange(R, device="cuda")[None, :] < want[1][:, None]
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]) and torch.equal(got[2][used], want[2][used])
        for name in ("active", "proposals", "algo_evals"):
            assert list(getattr(got[3], name)[:6]) == list(getattr(want[3], name)[:6])
