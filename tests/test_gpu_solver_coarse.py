"""The reconstruction loop with its coarse wavelet levels in one launch, against the loop with a launch per level (the
two-stream form): one to three coarse levels, all but the finest of a small image, and none.

Both do the same operations in the same order but for the ball norm's sum in FP64, whose order may change a few last bits
of single precision: 1e-5 of the image's norm after 25 iterations.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1307_3424_amd as wp  # noqa: E402

L = synth.fov_L()


@pytest.mark.parametrize("N,levels", [(256, 4), (256, 3), (256, 2), (128, 4), (64, 4), (64, 2), (32, 3), (512, 1)])
@pytest.mark.parametrize("graph", [0, 1])
def test_coarse_levels_match_a_launch_per_level(N, levels, graph):
    rng = np.random.default_rng([N, levels])
    M, iters = 2000, 25
    u, v, w = synth.uvw(N, M, L, "gaussian", 0.25, 10 / (4 * L * L), rng)
    plan = wp.Plan(N, L)
    G = wp.build_G(plan, *(torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (u, v, w)), 0.99)
    G.order = wp.WP_ORDER_SORTED
    x = np.zeros((N, N), np.complex64)
    x[N // 4:N // 2, N // 3:N // 2] = 1.0
    y = wp.apply_Phi(plan, G, torch.from_numpy(x.reshape(-1)).cuda())
    y = y + 0.01 * torch.from_numpy(synth.random_complex(M, rng).astype(np.complex64)).cuda()
    nu = wp.power_norm2(plan, G, torch.ones(N * N, dtype=torch.float32, device="cuda"), 20)
    eps = 0.01 * float(np.sqrt(2 * M))
    plan.set_tuning("solve_graph", graph)
    got = wp.solve(plan, G, y, eps, 1.05 * nu, iters, levels).clone()
    plan.set_tuning("solve_graph", 0)
    plan.set_tuning("solve_streams", 2)
    want = wp.solve(plan, G, y, eps, 1.05 * nu, iters, levels)
    assert want.abs().max() > 0
    assert (torch.linalg.norm(got - want) / torch.linalg.norm(want)).item() < 1e-5
