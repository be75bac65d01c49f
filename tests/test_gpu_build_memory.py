"""Device memory of a build: what stays is G itself, and a batch's workspaces are not all held at once."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1307_3424_amd as wp  # noqa: E402

L = synth.fov_L()
SLACK = 1 << 20                            # the allocator's rounding of some ten tensors


def coordinates(N, M, seed):
    rng = np.random.default_rng(seed)
    u, v = rng.uniform(-0.9 * N, 0.9 * N, (2, M)) / (2 * L)
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (u, v, np.zeros(M))]


@pytest.mark.parametrize("kw", [dict(transpose=False), dict(transpose=False, stored=False, factors=True), dict()])
def test_a_built_G_holds_its_own_bytes_only(kw):
    plan = wp.Plan(32, L)
    uvw = coordinates(32, 50000, 1)
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    G = wp.build_G(plan, *uvw, 0.5, **kw)
    assert torch.cuda.memory_allocated() - before <= G.nbytes() + SLACK


def test_a_batch_holds_a_bounded_workspace(monkeypatch):
    P, M = 6, 50000
    plans = [wp.Plan(32, L)] * P
    cs = [coordinates(32, M, p) for p in range(P)]
    one = [wp.build_G(plans[p], *cs[p], 0.5, transpose=False) for p in range(P)]
    limit = 256 << 20                      # two of these problems' workspaces
    monkeypatch.setattr(wp, "BATCH_WORKSPACE", limit, raising=False)
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    torch.cuda.reset_peak_memory_stats()
    Gs = wp.build_G_batch(plans, *([c[i] for c in cs] for i in range(3)), [0.5] * P, transpose=False)
    held = sum(G.nbytes() for G in Gs)
    assert torch.cuda.memory_allocated() - before <= held + SLACK
    assert torch.cuda.max_memory_allocated() - before <= held + limit + SLACK
    for a, b in zip(one, Gs):
        assert a.nnz == b.nnz and torch.equal(a.perm, b.perm) and torch.equal(a.col, b.col)
        assert torch.equal(torch.view_as_real(a.val), torch.view_as_real(b.val))
    with pytest.raises(wp.WprojError):
        wp.build_G_batch([], [], [], [], [])
