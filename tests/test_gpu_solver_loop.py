"""The reconstruction loop's forms (one or two streams, coarse wavelet levels in one launch) against the oracle's iteration
over the same operator, and each other; solves from several threads on one plan.

Five iterations in single precision against double: 1e-4 of the image's norm, as for the tiny form.
"""
import threading

import numpy as np
import pytest

import synth
from oracle import solver

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1307_3424_amd as wp  # noqa: E402

L = synth.fov_L()


def problem(N, M):
    rng = np.random.default_rng([N, M, 3])
    u, v, w = synth.uvw(N, M, L, "gaussian", 0.25, 10 / (4 * L * L), rng)
    plan = wp.Plan(N, L)
    G = wp.build_G(plan, *(torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (u, v, w)), 0.99)
    x = np.zeros((N, N), np.complex64)
    x[N // 4:N // 2, N // 3:N // 2] = 1.0
    y = wp.apply_Phi(plan, G, torch.from_numpy(x.reshape(-1)).cuda())
    y = y + 0.01 * torch.from_numpy(synth.random_complex(M, rng).astype(np.complex64)).cuda()
    nu = 1.05 * wp.power_norm2(plan, G, torch.ones(N * N, dtype=torch.float32, device="cuda"), 20)
    return plan, G, y, 0.01 * float(np.sqrt(2 * M)), nu


# L0 of the coarse launch 64, 64, 32, 16; one to three levels in it; none
@pytest.mark.parametrize("N,levels", [(256, 4), (256, 3), (128, 4), (64, 4), (64, 2), (32, 3), (256, 1)])
@pytest.mark.parametrize("streams", [1, 2])
def test_early_iterates_match_the_oracle(N, levels, streams):
    plan, G, y, eps, nu = problem(N, 2000)

    def dev(a):
        return torch.from_numpy(np.ascontiguousarray(a.reshape(-1).astype(np.complex64))).cuda()

    want = solver.solve(y.cpu().numpy().astype(np.complex128),
                        lambda z: wp.apply_Phi(plan, G, dev(z)).cpu().numpy().astype(np.complex128),
                        lambda z: wp.apply_PhiT(plan, G, dev(z)).cpu().numpy().astype(np.complex128).reshape(N, N),
                        (N, N), eps, nu, 5, levels=levels)
    plan.set_tuning("solve_streams", streams)
    got = wp.solve(plan, G, y, eps, nu, 5, levels).cpu().numpy().reshape(N, N)
    assert np.linalg.norm(got - want) < 1e-4 * np.linalg.norm(want)


# the automatic choice's edges: visibilities, levels, iterations
@pytest.mark.parametrize("M,levels,iters", [(16384, 3, 20), (16383, 3, 20), (16384, 2, 20), (16384, 3, 19)])
def test_automatic_choice_gives_the_one_stream_image(M, levels, iters):
    plan, G, y, eps, nu = problem(256, M)
    got = wp.solve(plan, G, y, eps, nu, iters, levels).clone()
    plan.set_tuning("solve_streams", 1)
    want = wp.solve(plan, G, y, eps, nu, iters, levels)
    assert (torch.linalg.norm(got - want) / torch.linalg.norm(want)).item() < 1e-5


def test_threads_share_a_plan():
    """Each thread on its own stream: at most one uses the plan's second stream at a time, all give the same image."""
    plan, G, y, eps, nu = problem(256, 16384)
    want = wp.solve(plan, G, y, eps, nu, 30, 4).clone()
    torch.cuda.synchronize()
    got = [None] * 4

    def work(i):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for _ in range(3):
                got[i] = wp.solve(plan, G, y, eps, nu, 30, 4)
        s.synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    for g in got:
        assert (torch.linalg.norm(g - want) / torch.linalg.norm(want)).item() < 1e-5
