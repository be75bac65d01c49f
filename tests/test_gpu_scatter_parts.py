"""Gridding from the factor records where few work items are split over workgroups: short rows into as many as run at
once, long rows (512 bytes of record or more) into twice as many.

Reference: the stored taps in FP64.  A tap from the records and the stored one differ by their products' roundings, a
cell's sum of n terms in FP32 (the window's sums are exact, its flushes are added in FP32): at most n + 16 roundings of
2^-24 on every term, so |error| <= 2 (n + 16) 2^-24 sum |g| |y|.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1307_3424_amd as wp  # noqa: E402

L = synth.fov_L()


# rows of one item and of a few, items at and past the number that is split, each with short and with long rows
SIZES = [(64, 1), (64, 5), (64, 40), (64, 1500), (128, 7071)]


@pytest.mark.parametrize("N,M,long", [(N, M, long) for N, M in SIZES for long in (False, True)] + [(256, 16000, False)])
@pytest.mark.parametrize("order", [wp.WP_ORDER_CALLER, wp.WP_ORDER_SORTED])
def test_split_items(N, M, long, order):
    spread, E = (40, 0.9999) if long else (6, 0.99)
    rng = np.random.default_rng([N, M, spread])
    u, v, _ = synth.uvw(N, M, L, "uniform", 0.25, 0.0, rng)
    w = np.linspace(0.9, 1.0, M) * spread / (4 * L * L)
    plan = wp.Plan(N, L)
    uvw = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (u, v, w)]
    full = wp.build_G(plan, *uvw, E, transpose=False)
    G = wp.build_G(plan, *uvw, E, factors=True, transpose=False, stored=False)
    assert (G.fdat.numel() >= 512 * M) == long
    y = torch.from_numpy(synth.random_complex(M, rng).astype(np.complex64)).cuda()
    ys = wp.to_sorted(G, y)
    G.order = order
    got = wp.grid_scatter(plan, G, ys if order == wp.WP_ORDER_SORTED else y).reshape(-1)
    cells = plan.Ng ** 2
    row = torch.repeat_interleave(torch.arange(M, device="cuda"), full.rowptr[1:] - full.rowptr[:-1])
    col = full.col.long()
    t = full.val.to(torch.complex128).conj() * ys.to(torch.complex128)[row]
    ref = torch.zeros(cells, dtype=torch.complex128, device="cuda").index_add_(0, col, t)
    mag = torch.zeros(cells, dtype=torch.float64, device="cuda").index_add_(0, col, t.abs())
    n = torch.bincount(col, minlength=cells)
    assert bool(((got - ref).abs() <= 2 * (n + 16) * 2.0 ** -24 * mag).all())
