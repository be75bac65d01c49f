"""The blocked gather is compiled once for visibilities in the caller's order and once for sorted ones; a batch tells them
apart at run time.  All read the same taps and add in the same order, so their grids are equal bit for bit.

Reference of the cells: the stored taps in FP64.  A cell sums n products, each of four terms, in FP32: at most n + 8
roundings of 2^-24 on every term, so |error| <= 2 (n + 8) 2^-24 sum |g| |y|.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1307_3424_amd as wp  # noqa: E402

L = synth.fov_L()


# one visibility: blocks of few entries; more of them: chunks that end anywhere; more than the image has pixels
@pytest.mark.parametrize("N,M", [(32, 1), (32, 57), (32, 1025), (64, 4097)])
@pytest.mark.parametrize("taps", [wp.WP_TAPS_C64, wp.WP_TAPS_BF16, wp.WP_TAPS_I16])
def test_caller_order_equals_sorted(N, M, taps):
    rng = np.random.default_rng([N, M, 11])
    u, v, w = synth.uvw(N, M, L, "uniform", 0.25, 12 / (4 * L * L), rng)
    plan = wp.Plan(N, L)
    G = wp.build_G(plan, *(torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (u, v, w)), 0.99, taps=taps)
    cells = plan.Ng ** 2
    assert G.n_tblk > 0 and G.nnz < 512 * cells                   # the blocked form
    y = torch.from_numpy(synth.random_complex(M, rng).astype(np.complex64)).cuda()
    ys = wp.to_sorted(G, y)
    first = None
    for chunk in (0, 256, 512, 768, 1024):
        plan.set_tuning("gather_chunk", chunk)
        G.order = wp.WP_ORDER_CALLER
        caller = wp.grid_gather(plan, G, y)
        G.order = wp.WP_ORDER_SORTED
        assert torch.equal(wp.grid_gather(plan, G, ys), caller)
        first = caller if first is None else first
    if taps == wp.WP_TAPS_C64:
        row = torch.repeat_interleave(torch.arange(M, device="cuda"), G.rowptr[1:] - G.rowptr[:-1])
        col = G.col.long()
        t = G.val.to(torch.complex128).conj() * ys.to(torch.complex128)[row]
        ref = torch.zeros(cells, dtype=torch.complex128, device="cuda").index_add_(0, col, t)
        mag = torch.zeros(cells, dtype=torch.float64, device="cuda").index_add_(0, col, t.abs())
        n = torch.bincount(col, minlength=cells)
        for got in (first, caller):
            assert bool(((got.reshape(-1) - ref).abs() <= 2 * (n + 8) * 2.0 ** -24 * mag).all())
    # the batch kernel, whose chunk is 512: each problem in its own order
    G.order = wp.WP_ORDER_CALLER
    plan.set_tuning("gather_chunk", 0)
    Gs = wp.build_G(plan, *(torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (u, v, w)), 0.99, taps=taps)
    Gs.order = wp.WP_ORDER_SORTED
    batch = wp.Batch(plan, [G, Gs])
    x, _, grids = batch.new_buffers()
    x = batch.apply_PhiT(torch.cat([y, ys]), x, grids).reshape(2, -1)
    assert torch.equal(x[0], x[1])
