"""The padded copy of X is an extra: a call that finds no room for it does without, and gives up nothing it had."""
import gc

import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rn():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2310_20419_amd as m
    m.load_library()
    return m


def _free():
    import torch
    gc.collect()
    torch.cuda.empty_cache()
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_no_room_for_the_copy_leaves_the_kept_block_alone(rn):
    """X takes a little more than half of the card, so its padded copy cannot be had.  The build works on X itself, in the
    block that an earlier call left, which is larger than it needs and stays as it is."""
    import torch
    rn.rnnd_release_workspace()
    _free()
    n0 = 5_000_000
    keys = torch.full((n0, 96), -1, dtype=torch.int64, device="cuda")
    deg = torch.zeros((n0,), dtype=torch.int32, device="cuda")
    rn.rnnd_add_reverse_edges(keys, deg, 96)             # leaves a block of more than 10 GB
    del keys, deg
    before = _free()
    d, R = 33_025, 2
    n = int(0.52 * torch.cuda.mem_get_info()[1]) // d
    assert rn.rnnd_workspace_bytes(n, d, rn.RNND_U8, R, 1) < 6 << 30
    X = torch.zeros((n, d), dtype=torch.uint8, device="cuda")
    graph, degree, _, st = rn.rnnd_build_ex(X, 1, R, 1, 1, 3, want_keys=False)
    assert st.kernel_variant == 1 and int(degree.min()) == int(degree.max()) == 1 and int(graph[:, 0].min()) >= 0
    del X, graph, degree
    after = _free()
    rn.rnnd_release_workspace()
    assert abs(after - before) < 1 << 30, "the kept block changed by %.1f GB" % ((after - before) / 2**30)
