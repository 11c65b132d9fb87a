"""Coordinates that are NaN or infinite, in float rows of every kind that is padded (both orders of the copy, each storage
type) and in rows the matrix-core scan takes as they are: builds, single rounds and block-sequential passes must give what
the pair-at-a-time kernel gives, and a large finite value must not be taken for an infinite one."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N = 2304      # past the 2,048 vertices from which the step-wise call pads too
ROWS = [("f32", 33), ("f32", 100), ("f32", 96), ("f16", 40), ("f16", 100), ("f16", 64), ("bf16", 24), ("bf16", 65), ("bf16", 96)]


@pytest.fixture(scope="module")
def rn():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2310_20419_amd as m
    m.load_library()
    return m


def _rows(dtype, d, bad):
    import torch
    g = np.random.default_rng(5)
    X = (g.normal(size=(8, d))[g.integers(0, 8, size=N)] + 0.5 * g.normal(size=(N, d))).astype(np.float32)
    t = torch.from_numpy(X).cuda().to({"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[dtype])
    value = torch.finfo(t.dtype).max if bad == "largest" else float(bad)
    for r, c in ((0, 0), (3, 0), (700, 1), (701, d - 1), (702, d - 1), (2000, d // 2)):
        t[r, c] = value if r != 702 else -value
    return t


def _variant(rn, v, f):
    try:
        rn.rnnd_set_kernel_variant(v)
        return f()
    finally:
        rn.rnnd_set_kernel_variant(0)


@pytest.mark.parametrize("bad", ["nan", "inf", "largest"])
@pytest.mark.parametrize("dtype,d", ROWS)
def test_same_as_the_pair_at_a_time_kernel(rn, dtype, d, bad):
    import torch
    X = _rows(dtype, d, bad)
    R, padded = 64, d * X.element_size() % 64 != 0

    def build():
        return rn.rnnd_build_ex(X, 20, R, 2, 3, 4)
    want = _variant(rn, 1, build)
    used = torch.arange(R, device="cuda")[None, :] < want[1][:, None]
    for v in (0, 2):
        got = _variant(rn, v, build)
        if padded:
            assert got[3].kernel_variant == (3 if bad == "largest" else 1)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]) and torch.equal(got[2][used], want[2][used])
        assert list(got[3].algo_evals[:6]) == list(want[3].algo_evals[:6])

    def steps():
        keys, deg = rn.rnnd_random_graph(X, 20, R, 4)
        evals = [rn.rnnd_update_neighbors(X, keys, deg, R, 2).algo_evals[k] for k in range(2)]
        rn.rnnd_add_reverse_edges(keys, deg, R)
        evals += [rn.rnnd_update_neighbors_blocks(X, keys, deg, R, 3, 1).algo_evals[0]]
        return keys, deg, evals
    want = _variant(rn, 1, steps)
    used = torch.arange(R, device="cuda")[None, :] < want[1][:, None]
    for v in (0, 2):
        got = _variant(rn, v, steps)
        assert torch.equal(got[1], want[1]) and torch.equal(got[0][used], want[0][used]) and got[2] == want[2], (v, got[2], want[2])


@pytest.mark.parametrize("dtype,d", [("f32", 33), ("f32", 100), ("bf16", 65)])
def test_a_single_round_does_not_wait_for_the_rows(rn, dtype, d):
    """The padded copy of a step-wise call is made and used without a look at it by the host: a call with nothing to do
    takes the matrix-core scan whatever X holds."""
    X = _rows(dtype, d, "nan")
    keys, deg = rn.rnnd_random_graph(X, 20, 64, 4)
    assert rn.rnnd_update_neighbors(X, keys, deg, 64, 1).kernel_variant == 3


@pytest.mark.parametrize("S,R", [(8, 16), (20, 64)])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 320), ("f16", 64), ("f16", 512), ("bf16", 320)])
def test_rows_of_nan_of_either_sign(rn, dtype, d, S, R):
    """A distance that is not a number is stored, and compared, with the sign its sum happens to end with, which depends on the
    order of the sum: only the routine that all stored distances come from may decide such a pair."""
    import torch
    g = np.random.default_rng(6)
    X = (g.normal(size=(8, d))[g.integers(0, 8, size=N)] + 0.5 * g.normal(size=(N, d))).astype(np.float32)
    t = torch.from_numpy(X).cuda().to({"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[dtype])
    bits = t.view(torch.int32 if dtype == "f32" else torch.int16)
    quiet = {"f32": 0x7FC00000, "f16": 0x7E00, "bf16": 0x7FC0}[dtype]
    for k in range(6):      # a quarter of the rows holds one, of either sign
        rows = torch.from_numpy(g.permutation(N)[:N // 16]).cuda()
        bits[rows, int(g.integers(0, d))] = quiet if k % 2 else quiet - (1 << (31 if dtype == "f32" else 15))
    assert int((bits[torch.isnan(t)] < 0).sum()) > 300 and int((bits[torch.isnan(t)] > 0).sum()) > 300

    def build():
        return rn.rnnd_build_ex(t, S, R, 2, 3, 4)
    want = _variant(rn, 1, build)
    used = torch.arange(R, device="cuda")[None, :] < want[1][:, None]
    got = _variant(rn, 0, build)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]) and torch.equal(got[2][used], want[2][used])
