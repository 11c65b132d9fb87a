"""Rows on which the prune test of the float scan is delicate: far from the origin every Gram-form distance loses its
leading digits, copies of a row differ by nothing at all, very small coordinates have squares that single precision cannot
hold.  The matrix-core scans (automatic, and in double precision throughout) must take the decisions the pair-at-a-time kernel takes: the same graphs, the same stored distances, the same counts."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N = 2400      # past the 2,048 vertices from which the step-wise call pads too


@pytest.fixture(scope="module")
def rn():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2310_20419_amd as m
    m.load_library()
    return m


def _rows(kind, d, seed):
    g = np.random.default_rng(seed)
    X = (g.normal(size=(8, d))[g.integers(0, 8, size=N)] + 0.5 * g.normal(size=(N, d))).astype(np.float32)
    if kind.startswith("centre"):
        X = X + np.float32(kind.split()[1])
    elif kind.startswith("scale"):
        X = X * np.float32(kind.split()[1])
    elif kind == "copies":                        # 24 rows, 100 times each
        X = X[g.permutation(np.repeat(np.arange(24), N // 24))]
    elif kind == "zeros":                         # half the rows are the origin
        X[::2] = 0
    return np.ascontiguousarray(X, dtype=np.float32)


FAR = [("f32", k, d) for k in ("centre 1e3", "centre 1e5", "centre 1e6", "centre 1e7", "copies", "zeros") for d in (96, 100, 33)] + \
      [(t, k, d) for t in ("f16", "bf16") for k in ("centre 200", "copies") for d in (64, 100)]
SMALL = [("f32", k, d) for k in ("scale 1e-19", "scale 1e-20", "scale 1e-21", "scale 1e-22", "scale 1e-23", "scale 1e-38") for d in (96, 100)] + \
        [("bf16", k, d) for k in ("scale 1e-20", "scale 1e-22", "scale 1e-23") for d in (64, 100)] + [("f16", "scale 1e-4", 64)]


def _compare(rn, X, S, R, T1, T2, seed, label):
    import torch
    try:
        rn.rnnd_set_kernel_variant(1)
        want = rn.rnnd_build_ex(X, S, R, T1, T2, seed)
        got = {}
        for v in (0, 2):
            rn.rnnd_set_kernel_variant(v)
            got[v] = rn.rnnd_build_ex(X, S, R, T1, T2, seed)
    finally:
        rn.rnnd_set_kernel_variant(0)
    used = torch.arange(R, device="cuda")[None, :] < want[1][:, None]
    for v, g in got.items():
        assert g[3].kernel_variant == 3
        bad = int((g[0] != want[0]).any(1).sum())
        assert bad == 0, "%s, variant %d: %d of %d rows differ" % (label, v, bad, len(X))
        assert torch.equal(g[1], want[1]) and torch.equal(g[2][used], want[2][used])
        assert list(g[3].algo_evals[:T1 * T2]) == list(want[3].algo_evals[:T1 * T2])
        assert list(g[3].proposals[:T1 * T2]) == list(want[3].proposals[:T1 * T2])


def _device(X, dtype):
    import torch
    return torch.from_numpy(X).cuda().to({"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[dtype])


@pytest.mark.parametrize("dtype,kind,d", FAR)
def test_rows_far_from_the_origin_and_copies(rn, dtype, kind, d):
    X = _device(_rows(kind, d, 7), dtype)
    for S, R in ((20, 96), (40, 128), (10, 24)):
        _compare(rn, X, S, R, 2, 3, 5, "%s %s d %d R %d" % (dtype, kind, d, R))


@pytest.mark.parametrize("dtype,kind,d", SMALL)
def test_squares_too_small_for_single_precision(rn, dtype, kind, d):
    X = _device(_rows(kind, d, 7), dtype)
    for S, R in ((20, 96), (10, 24)):
        _compare(rn, X, S, R, 2, 3, 5, "%s %s d %d R %d" % (dtype, kind, d, R))
