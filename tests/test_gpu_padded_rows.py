"""Rows the matrix tiles do not fit (odd lengths, long uint8 rows, an X that is not 16-byte aligned) are scanned on a
padded copy: the graph, the stored distances and the counters must be the oracle's, and the same bits as the generic
kernel's on X itself."""
import numpy as np
import pytest

import workloads as wl
from gpu_util import assert_snapshot_equal

pytestmark = pytest.mark.gpu

N = 2304      # past the 2,048 vertices from which the step-wise call pads too


@pytest.fixture(scope="module")
def rn():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2310_20419_amd as m
    m.load_library()
    return m


def _u8(n, d, seed, k=6, spread=12):
    g = np.random.default_rng(seed)
    c = g.integers(20, 236, size=(k, d))
    return np.clip(c[g.integers(0, k, size=n)] + g.integers(-spread, spread + 1, size=(n, d)), 0, 255).astype(np.uint8)


def _float(n, d, seed):
    g = np.random.default_rng(seed)
    return (g.normal(size=(8, d))[g.integers(0, 8, size=n)] + 0.5 * g.normal(size=(n, d))).astype(np.float32)


def _device(X, dtype, offset):
    """X on the device, `offset` elements past a 16-byte boundary."""
    import torch
    t = torch.from_numpy(X).cuda().to(dtype)
    if not offset:
        return t
    flat = torch.empty(t.numel() + 16, dtype=dtype, device="cuda")
    v = flat[offset:offset + t.numel()].view(t.shape)
    v.copy_(t)
    assert v.data_ptr() % 16 != 0
    return v


U8 = [(1, 0), (16, 0), (32, 1), (33, 0), (65, 0), (100, 3), (128, 5), (129, 0), (191, 0), (192, 0), (193, 0), (256, 0), (784, 0)]
FLOAT = [("f32", 1, 0), ("f32", 3, 0), ("f32", 4, 0), ("f32", 20, 0), ("f32", 31, 0), ("f32", 33, 0), ("f32", 36, 0),
         ("f32", 48, 1), ("f32", 100, 0), ("f32", 130, 0), ("f16", 7, 0), ("f16", 40, 0), ("f16", 64, 1), ("f16", 100, 0),
         ("bf16", 24, 0), ("bf16", 65, 0), ("bf16", 136, 0)]
CASES = [("u8",) + c for c in U8] + FLOAT


def _params(i):
    # degree caps on either side of the kernels' list lengths; S large enough for long lists now and then
    return [(10, 24, 2, 3), (40, 128, 2, 2), (20, 96, 2, 4), (33, 64, 2, 2)][i % 4]


@pytest.mark.parametrize("i,dtype,d,offset", [(i,) + c for i, c in enumerate(CASES)])
def test_build_equals_oracle_and_generic_kernel(rn, oracle_mod, i, dtype, d, offset):
    import torch
    S, R, T1, T2 = _params(i)
    X = _u8(N, d, i) if dtype == "u8" else _float(N, d, i)
    if dtype in ("f16", "bf16"):
        X = torch.from_numpy(X).to(getattr(torch, {"f16": "float16", "bf16": "bfloat16"}[dtype])).float().numpy()
    Xd = _device(X, {"u8": torch.uint8, "f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[dtype], offset)
    want = oracle_mod.build_sync(X, S, R, T1, T2, 3 + i)
    graph, degree, keys, st = rn.rnnd_build_ex(Xd, S, R, T1, T2, 3 + i)
    assert st.kernel_variant == (2 if dtype == "u8" else 3)
    assert_snapshot_equal(want.snap, dtype != "u8", keys, degree, "%s d %d" % (dtype, d))
    assert list(st.algo_evals[:T1 * T2]) == want.round_evals.tolist()
    assert list(st.proposals[:T1 * T2]) == want.round_props.tolist()
    # the generic kernel on X itself: the same bits
    try:
        rn.rnnd_set_kernel_variant(1)
        g1, d1, k1, s1 = rn.rnnd_build_ex(Xd, S, R, T1, T2, 3 + i)
    finally:
        rn.rnnd_set_kernel_variant(0)
    assert s1.kernel_variant == 1 and torch.equal(graph, g1) and torch.equal(degree, d1)
    used = torch.arange(R, device="cuda")[None, :] < degree[:, None]
    assert torch.equal(keys[used], k1[used])
    # step by step on X, the way of a caller that keeps the snapshot: RandomGraph on X, rounds on the copy
    sk, sd = rn.rnnd_random_graph(Xd, S, R, 3 + i)
    rn.rnnd_update_neighbors(Xd, sk, sd, R, T2)
    step = oracle_mod.random_graph(X, S, 3 + i, R)
    for _ in range(T2):
        step, _, _ = oracle_mod.update_neighbors_sync(X, step, R)
    assert_snapshot_equal(step, dtype != "u8", sk, sd, "%s d %d, steps" % (dtype, d))


@pytest.mark.parametrize("mode", [1, 2, 3])
def test_every_launch_form_of_the_long_uint8_rows(rn, oracle_mod, mode):
    """One launch for all classes, the short-list launch plus one, a launch per class."""
    import torch
    X = _u8(N, 200, 77, k=3, spread=9)            # tight clusters: lists of every length up to 128
    want = oracle_mod.build_sync(X, 60, 128, 2, 3, 11)
    try:
        rn.rnnd_set_scan_launches(mode)
        graph, degree, keys, st = rn.rnnd_build_ex(torch.from_numpy(X).cuda(), 60, 128, 2, 3, 11)
    finally:
        rn.rnnd_set_scan_launches(0)
    assert_snapshot_equal(want.snap, False, keys, degree, "mode %d" % mode)
    assert list(st.algo_evals[:6]) == want.round_evals.tolist()


@pytest.mark.parametrize("dtype,d", [("u8", 100), ("f32", 33), ("bf16", 65)])
@pytest.mark.parametrize("n,R", [(300, 128), (300, 32), (40_000, 96), (70_000, 64), (140_000, 48)])
def test_launch_forms_by_size(rn, dtype, d, n, R):
    """Sizes on either side of the rules that choose how many launches a scan takes: the generic kernel's graph."""
    import torch
    X = torch.from_numpy(_u8(n, d, 2, k=40, spread=30) if dtype == "u8" else _float(n, d, 2)).cuda()
    X = X.to(torch.bfloat16) if dtype == "bf16" else X
    got = rn.rnnd_build_ex(X, 20, R, 2, 3, 4)
    assert got[3].kernel_variant == (2 if dtype == "u8" else 3)
    try:
        rn.rnnd_set_kernel_variant(1)
        want = rn.rnnd_build_ex(X, 20, R, 2, 3, 4)
    finally:
        rn.rnnd_set_kernel_variant(0)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    assert list(got[3].algo_evals[:6]) == list(want[3].algo_evals[:6])


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("d", [33, 100])
def test_nan_and_infinity_go_to_the_generic_kernel(rn, bad, d):
    """A coordinate that is not finite: the same graph as the generic kernel gives on X."""
    import torch
    X = _float(N, d, 5)
    X[[3, 700, 701, 2000], [0, 1, d - 1, d // 2]] = bad
    Xd = torch.from_numpy(X).cuda()
    got = rn.rnnd_build_ex(Xd, 20, 64, 2, 3, 4)
    assert got[3].kernel_variant == 1
    try:
        rn.rnnd_set_kernel_variant(1)
        want = rn.rnnd_build_ex(Xd, 20, 64, 2, 3, 4)
    finally:
        rn.rnnd_set_kernel_variant(0)
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


def test_static_build_without_room_for_the_copy(rn):
    """rnnd_build_static takes what it took before: where its array has no room for the padded copy it works on X."""
    import torch
    d, R, T1, T2 = 784, 96, 2, 2
    n = 17_000
    while rn.rnnd_workspace_bytes(n, d, rn.RNND_U8, R, T1 * T2) > rn.RNND_STATIC_SCRATCH_BYTES:
        n -= 100
    for rows in (n, 3000):          # no room; room
        X = torch.from_numpy(_u8(rows, d, 9)).cuda()
        graph = torch.empty((rows, R), dtype=torch.int32, device="cuda")
        degree = torch.empty((rows,), dtype=torch.int32, device="cuda")
        rn.rnnd_build_static(X, 20, R, T1, T2, 5, graph, degree)
        g0, d0 = rn.rnnd_build(X, 20, R, T1, T2, 5)
        assert torch.equal(graph, g0) and torch.equal(degree, d0)
