"""Float32 builds whose Gram blocks come from a half-precision copy of the rows.  The copy only decides what lies beyond its
error bound, so graphs, stored distances and counts must be the pair-at-a-time kernel's, whatever the rows: far from the
origin, tiny, huge, of very different sizes, repeated, not finite."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N = 33_000      # past the size from which builds make the copy
KINDS = ["plain", "centre 1e3", "centre 1e6", "scale 1e-30", "scale 1e-20", "scale 1e15", "sizes", "outlier", "copies", "zeros", "nan", "inf"]


@pytest.fixture(scope="module")
def rn():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2310_20419_amd as m
    m.load_library()
    return m


def _rows(kind, d):
    import torch
    g = np.random.default_rng(11)
    X = (g.normal(size=(64, d))[g.integers(0, 64, size=N)] + 0.5 * g.normal(size=(N, d))).astype(np.float32)
    if kind.startswith("centre"):
        X = X + np.float32(kind.split()[1])
    elif kind.startswith("scale"):
        X = X * np.float32(kind.split()[1])
    elif kind == "sizes":                          # norms over twelve binades
        X = X * np.exp2(g.integers(-6, 7, size=(N, 1))).astype(np.float32)
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
    for S, R, T1, T2 in ((20, 96, 2, 2), (8, 16, 1, 2), (40, 128, 1, 2)):
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
