"""A single round on a large snapshot copies only the rows its active lists name when few vertices are active: rounds from
a fresh snapshot to a converged one, each from the same snapshot as the pair-at-a-time kernel's, on a workspace filled with
garbage, so that a row that was not copied shows."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,S,R", [("f32", 100, 20, 48), ("f32", 33, 40, 128), ("bf16", 65, 10, 24), ("f16", 40, 20, 96)])
def test_rounds_down_to_convergence(dtype, d, S, R):
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2310_20419_amd as rn
    n = 33_000
    g = np.random.default_rng(2)
    X = (g.normal(size=(60, d))[g.integers(0, 60, size=n)] + 0.5 * g.normal(size=(n, d))).astype(np.float32)
    X = torch.from_numpy(X).cuda().to({"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[dtype])
    rn.rnnd_release_workspace()
    rn.rnnd_set_workspace_poison(True)
    try:
        keys, deg = rn.rnnd_random_graph(X, S, R, 3)
        active, used = [], None
        for t in range(40):
            k1, d1 = keys.clone(), deg.clone()
            rn.rnnd_set_kernel_variant(1)
            want = rn.rnnd_update_neighbors(X, k1, d1, R, 1)
            rn.rnnd_set_kernel_variant(0)
            got = rn.rnnd_update_neighbors(X, keys, deg, R, 1)
            active.append(got.active[0])
            assert got.kernel_variant == 3 and got.active[0] == want.active[0] and got.algo_evals[0] == want.algo_evals[0]
            used = torch.arange(R, device="cuda")[None, :] < d1[:, None]
            assert torch.equal(deg, d1) and torch.equal(keys[used], k1[used]), "round %d, %d active" % (t, active[-1])
            if active[-1] == 0:
                break
        # the line is at one vertex in 64: rounds on both sides of it, with work to do
        assert active[0] == n and any(0 < a < n // 64 for a in active), active
    finally:
        rn.rnnd_set_kernel_variant(0)
        rn.rnnd_set_workspace_poison(False)
        rn.rnnd_release_workspace()
