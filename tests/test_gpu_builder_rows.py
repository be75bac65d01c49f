"""The builder's band rows, whole-axis rows and cell sorts at the sizes where one hands over to another:
kept sets, values and the transposed copy against the oracle's rows.

Tolerances: kept sets are bit-exact except for taps tied with the row threshold within FP64 rounding (1e-9
relative); a complex64 tap is its FP64 value rounded once, 2^-24 relative per component, so 1e-6 of the row's
largest tap leaves an order of magnitude.
"""
import numpy as np
import pytest

import synth
from oracle.wproj import Setup, energy_threshold, kernel_row

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1307_3424_amd as wp  # noqa: E402

L = synth.fov_L()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def build(N, u, v, w, E, W=4, **kw):
    plan = wp.Plan(N, L, kb_W=W)
    G = wp.build_G(plan, dev(u), dev(v), dev(w), E, **kw)
    torch.cuda.synchronize()
    return G


# (N, spread of the chirp in cells, E, W): the band inside the axis; as wide as the axis; too wide for the lists or
# the registers; the second, wider threshold range; every window width; all entries
@pytest.mark.parametrize("N,spread,E,W", [
    (32, 0, 0.99, 4), (32, 28, 0.99, 4), (32, 60, 0.999, 4), (64, 28, 0.99999, 4), (64, 120, 0.99, 4),
    (128, 28, 0.99, 2), (128, 240, 0.999, 4), (256, 28, 0.99, 4), (256, 60, 0.9999, 8), (256, 300, 0.9, 4),
    (512, 60, 0.99, 16), (512, 140, 0.99, 4), (1024, 28, 0.999, 4), (2048, 28, 0.99, 4), (2048, -28, 0.5, 4),
    (32, 20, 1.0, 4)])
def test_rows_at_the_edges_of_the_band(N, spread, E, W):
    M = 12 if N <= 256 else 5
    rng = np.random.default_rng([N, abs(spread), W])
    B = N / (2 * L)
    u, v = rng.uniform(-B, B, (2, M))
    w = spread / (4 * L * L) * rng.uniform(0.6, 1.0, M)
    # the corners of the grid: the band wraps
    u[0], v[0] = -B * (1 - 1e-5), B * (1 - 3e-5)
    u[1], v[1] = B * (1 - 2e-4), -B * (1 - 1e-4)
    G = build(N, u, v, w, E, W, transpose=False)
    s = Setup(N=N, L=L, W=W)
    rp, col, val, perm = (t.cpu().numpy() for t in (G.rowptr, G.col, G.val, G.perm))
    cell = 1.0 / (2 * L)
    for r in range(M):
        k = perm[r]
        g = kernel_row(u[k] / cell, v[k] / cell, w[k], s).ravel()
        e = (g * g.conj()).real
        tau, _ = energy_threshold(e, E)
        c = col[rp[r]:rp[r + 1]]
        assert np.all(np.diff(c) > 0)
        kept = np.zeros(g.size, dtype=bool)
        kept[c] = True
        # E = 1 keeps what is not zero: entries below 1e-25 of the largest may round to zero on one side
        tied = np.abs(e - tau) <= 1e-9 * tau if E < 1 else e <= 1e-25 * e.max()
        assert np.array_equal(kept | tied, (e >= tau) | tied), (k, int((kept != (e >= tau)).sum()))
        assert np.abs(val[rp[r]:rp[r + 1]] - g[c]).max() <= 1e-6 * np.abs(g).max()


# visibilities per cell around one point of a 64-cell grid: cells of a few entries, of up to 64, 256, and 4096
# entries and longer
@pytest.mark.parametrize("M,taps", [(40, wp.WP_TAPS_C64), (300, wp.WP_TAPS_BF16), (1500, wp.WP_TAPS_C64),
                                    (20000, wp.WP_TAPS_C64), (20000, wp.WP_TAPS_I16)])
def test_transposed_cells_of_every_length(M, taps):
    N = 32
    rng = np.random.default_rng(M)
    u, v = rng.normal(0, 3.0 / (2 * L), (2, M))
    w = 12 / (4 * L * L) * rng.uniform(0, 1, M)
    G = build(N, u, v, w, 0.99, taps=taps)
    rp, col, val = (t.cpu().numpy() for t in (G.rowptr, G.col, G.val))
    row = np.repeat(np.arange(M), np.diff(rp))
    order = np.lexsort((row, col))
    cp = np.concatenate([[0], np.cumsum(np.bincount(col, minlength=4 * N * N))])
    assert np.array_equal(G.tcolptr.cpu().numpy(), cp)
    assert np.array_equal(G.trow.cpu().numpy(), row[order])
    assert np.array_equal(G.tval.cpu().numpy(), val[order])


# the rows' sort: stable, whatever the number of tiles of pairs
@pytest.mark.parametrize("M", [1, 63, 4096, 4097, 70001])
def test_rows_sorted_by_cell_stably(M):
    N = 64
    rng = np.random.default_rng(M)
    u, v = rng.uniform(-N, N, (2, M)) / (2 * L) * 0.999
    G = build(N, u, v, np.zeros(M), 0.9, transpose=False)
    cu, cv = (np.floor(x * 2 * L).astype(np.int64) + N for x in (u, v))
    key = sum((((cu >> b) & 1) << (2 * b)) | (((cv >> b) & 1) << (2 * b + 1)) for b in range(12))
    assert np.array_equal(G.perm.cpu().numpy(), np.argsort(key, kind="stable"))
