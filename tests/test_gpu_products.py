"""Products from stored taps where one form hands over to another: few long rows (a workgroup each), and the adjoint in
caller order with its visibilities sorted first.

Reference of the rows: the stored taps in FP64.  A row sums n products, each of four terms, in FP32: at most n + 8
roundings of 2^-24 on every term, so |error| <= 2 (n + 8) 2^-24 sum |g| |x|.  The sorted adjoint adds the same terms in
the same order as the unsorted one, so their images are equal bit for bit.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1307_3424_amd as wp  # noqa: E402

L = synth.fov_L()


def build(N, M, spread, taps=wp.WP_TAPS_C64):
    rng = np.random.default_rng([N, M, 7])
    u, v, _ = synth.uvw(N, M, L, "uniform", 0.25, 0.0, rng)
    w = np.linspace(0.9, 1.0, M) * spread / (4 * L * L)           # every row long
    plan = wp.Plan(N, L)
    uvw = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (u, v, w)]
    return plan, wp.build_G(plan, *uvw, 0.99, taps=taps), rng


def c64(n, rng):
    return torch.from_numpy(synth.random_complex(n, rng).astype(np.complex64)).cuda()


@pytest.mark.parametrize("M", [1, 3, 820, 16384])
@pytest.mark.parametrize("taps", [wp.WP_TAPS_C64, wp.WP_TAPS_BF16, wp.WP_TAPS_I16])
@pytest.mark.parametrize("order", [wp.WP_ORDER_CALLER, wp.WP_ORDER_SORTED])
def test_long_rows(M, taps, order):
    plan, G, rng = build(32, M, 60, taps)
    assert G.nnz >= 768 * M
    G.order = order
    X = c64(plan.Ng ** 2, rng)
    got = wp.degrid(plan, G, X)
    plan.set_tuning("degrid_lanes", 64)                           # a wavefront per row
    wave = wp.degrid(plan, G, X)
    plan.set_tuning("degrid_lanes", 0)
    if taps == wp.WP_TAPS_C64:
        at = G.perm.long() if order == wp.WP_ORDER_CALLER else torch.arange(M, device="cuda")
        n = G.rowptr[1:] - G.rowptr[:-1]
        row = torch.repeat_interleave(torch.arange(M, device="cuda"), n)
        t = G.val.to(torch.complex128) * X[G.col.long()].to(torch.complex128)
        ref = torch.zeros(M, dtype=torch.complex128, device="cuda").index_add_(0, row, t)
        mag = torch.zeros(M, dtype=torch.float64, device="cuda").index_add_(0, row, t.abs())
        for y in (got, wave):
            assert bool(((y[at] - ref).abs() <= 2 * (n + 8) * 2.0 ** -24 * mag).all())
    # the same taps and values in another order of sums: as close to each other as either is to the reference
    assert (torch.linalg.norm(got - wave) / torch.linalg.norm(wave)).item() <= 1e-6


# 3 M taps is where the sort pays; as many visibilities as the image has pixels, and more than it can hold
@pytest.mark.parametrize("N,M,spread", [(64, 820, 120), (64, 4096, 60), (64, 4097, 60), (32, 200, 60)])
def test_adjoint_in_caller_order(N, M, spread):
    plan, G, rng = build(N, M, spread)
    y = c64(M, rng)
    n = N * N
    want = wp.apply_PhiT(plan, G, y)                              # caller order
    G.order = wp.WP_ORDER_SORTED
    assert torch.equal(wp.apply_PhiT(plan, G, wp.to_sorted(G, y)), want)
    G.order = wp.WP_ORDER_CALLER
    # x next to y on either side, and over its first or last value: y is read before x is written
    for x0, y0 in ((0, n), (0, n - 1), (M, 0), (M, 1)):
        buf = torch.zeros(n + M + 1, dtype=torch.complex64, device="cuda")
        buf[y0:y0 + M] = y
        wp.apply_PhiT(plan, G, buf[y0:y0 + M], x=buf[x0:x0 + n])
        assert torch.equal(buf[x0:x0 + n], want)
