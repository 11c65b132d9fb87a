"""A redirected edge that its target's list holds already: the merge drops the second of two equal keys, and a key is the distance's bits with the id.
Where the two distances of one pair differ in their bits -- numbers that are none, with the sign that the order of their operands gave them; a snapshot whose
distances were summed in another order -- both entries stay, whichever launches a round consists of."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N = 2304
DTYPES = {"f32": "float32", "f16": "float16", "bf16": "bfloat16"}


@pytest.fixture(scope="module")
def rn():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2310_20419_amd as m
    m.load_library()
    return m


def _rows(n, d, dtype, seed):
    import torch
    g = np.random.default_rng(seed)
    X = (g.normal(size=(8, d))[g.integers(0, 8, size=n)] + 0.5 * g.normal(size=(n, d))).astype(np.float32)
    return torch.from_numpy(X).cuda().to(getattr(torch, DTYPES[dtype]))


def _variant(rn, v, f):
    try:
        rn.rnnd_set_kernel_variant(v)
        return f()
    finally:
        rn.rnnd_set_kernel_variant(0)


def _same(R, got, want):
    import torch
    used = torch.arange(R, device="cuda")[None, :] < want[1][:, None]
    assert torch.equal(got[1], want[1]) and torch.equal(got[0][used], want[0][used])


@pytest.mark.parametrize("S,R", [(8, 16), (20, 64), (60, 128)])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 320), ("f16", 64), ("bf16", 320)])
def test_nan_of_either_sign_in_every_launch_of_the_merge(rn, dtype, d, S, R):
    import torch
    X = _rows(N, d, dtype, 6)
    g = np.random.default_rng(7)
    bits = X.view(torch.int32 if dtype == "f32" else torch.int16)
    quiet = {"f32": 0x7FC00000, "f16": 0x7E00, "bf16": 0x7FC0}[dtype]
    for k in range(6):      # a quarter of the rows holds one, of either sign
        rows = torch.from_numpy(g.permutation(N)[:N // 16]).cuda()
        bits[rows, int(g.integers(0, d))] = quiet if k % 2 else quiet - (1 << (31 if dtype == "f32" else 15))

    def sync():
        _, deg, keys, _ = rn.rnnd_build_ex(X, S, R, 2, 3, 4)
        return keys, deg

    def blocks():
        _, deg, keys, _ = rn.rnnd_build_blocks(X, S, R, 2, 3, 4, 1)
        return keys, deg
    want = _variant(rn, 1, sync)
    _same(R, sync(), want)             # classify, merge and compact in one launch
    _same(R, blocks(), want)           # a launch each
    try:
        rn.rnnd_set_event_timing(True)
        _same(R, sync(), want)         # a launch each
    finally:
        rn.rnnd_set_event_timing(False)


@pytest.mark.parametrize("n,d,dtype", [(N, 64, "f16"), (N, 96, "bf16"), (N, 100, "bf16"), (140_000, 32, "f16")])
def test_a_snapshot_whose_distances_were_rounded_elsewhere(rn, n, d, dtype):
    """Every third distance of the snapshot is the next float: Alg. 4's lists hold what they are given.  More than 131,072 vertices: the merge is a launch
    of its own, as in block-sequential passes."""
    import torch
    R, X = 64, _rows(n, d, dtype, 8)
    keys, deg = rn.rnnd_random_graph(X, 20, R, 4)
    rn.rnnd_update_neighbors(X, keys, deg, R, 2)
    rn.rnnd_add_reverse_edges(keys, deg, R)
    used = torch.arange(R, device="cuda")[None, :] < deg[:, None]
    other = used & ((keys >> 1) % 3 == 0)
    keys = torch.where(used, keys + (other.to(torch.int64) << 32), torch.iinfo(torch.int64).max).sort(dim=1).values.contiguous()

    def rounds(call):
        k, m = keys.clone(), deg.clone()
        call(k, m)
        return k, m
    calls = [lambda k, m: rn.rnnd_update_neighbors(X, k, m, R, 3), lambda k, m: rn.rnnd_update_neighbors_blocks(X, k, m, R, 1, 3)]
    want = _variant(rn, 1, lambda: rounds(calls[0]))
    twice = want[0] >> 1 & 0x7FFFFFFF
    twice = twice.masked_fill(torch.arange(R, device="cuda")[None, :] >= want[1][:, None], -1).sort(dim=1).values
    assert int(((twice[:, 1:] == twice[:, :-1]) & (twice[:, 1:] >= 0)).sum()) > 0, "no vertex is held twice: the test shows nothing"
    for call in calls:
        _same(R, rounds(call), want)
