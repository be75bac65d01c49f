"""Rows of the linear chirp near the edges of the band they are made from, against the oracle's rows.

A kept set is compared but for entries tied with the row's threshold: energies within 1e-9 of it, and entries where the
running sum of the energies, largest first, comes within 1e-13 of the row's energy of the fraction kept (FP64 sums of up
to 65536 energies err by some 1e-15 of it; a kept entry's energy is above 1e-12 of it at every E used here).  A complex64
tap is its FP64 value rounded once, so 1e-6 of the row's largest tap leaves an order of magnitude.
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


def rows_of(G):
    """(columns, values) of each visibility's row."""
    rp, perm = G.rowptr.cpu().numpy(), G.perm.cpu().numpy()
    col, val = G.col.cpu().numpy(), G.val.cpu().numpy()
    return {int(k): (col[rp[r]:rp[r + 1]], val[rp[r]:rp[r + 1]]) for r, k in enumerate(perm)}


def check_rows(N, W, reach, E, M, **kw):
    """M rows whose chirps reach up to reach cells (2 |w| L^2), uniform over the plane."""
    rng = np.random.default_rng([N, W, int(10 * reach)])
    B = N / (2 * L)
    u, v = rng.uniform(-B, B, (2, M))
    w = reach / (2 * L * L) * rng.uniform(0.5, 1.0, M)
    plan = wp.Plan(N, L, kb_W=W)
    G = wp.build_G(plan, dev(u), dev(v), dev(w), E, transpose=False, **kw)
    s = Setup(N=N, L=L, W=W)
    rp, col, val, perm = (t.cpu().numpy() for t in (G.rowptr, G.col, G.val, G.perm))
    for r in range(M):
        k = perm[r]
        g = kernel_row(u[k] * 2 * L, v[k] * 2 * L, w[k], s).ravel()
        e = (g * g.conj()).real
        tau, _ = energy_threshold(e, E)
        order = np.argsort(-e, kind="stable")
        run = np.empty(e.size, dtype=np.longdouble)
        run[order] = np.cumsum(e[order].astype(np.longdouble))
        total = run[order[-1]]
        tied = (np.abs(e - tau) <= 1e-9 * tau) | (np.abs(run - E * total) <= 1e-13 * total)
        c = col[rp[r]:rp[r + 1]]
        assert np.all(np.diff(c) > 0)
        kept = np.zeros(g.size, dtype=bool)
        kept[c] = True
        assert np.array_equal(kept | tied, (e >= tau) | tied), (k, int((kept != (e >= tau)).sum()))
        assert np.abs(val[rp[r]:rp[r + 1]] - g[c]).max() <= 1e-6 * np.abs(g).max()


# more candidates along u than a wavefront has lanes: the row's offsets are carried from one 64 to the next
@pytest.mark.parametrize("N,W,reach,E", [(64, 4, 20, 0.99999), (128, 4, 40, 0.9999), (256, 4, 40, 0.9999)])
def test_rows_of_more_candidates_than_lanes(N, W, reach, E):
    check_rows(N, W, reach, E, 6)


# a band that reads every h(d) and yet leaves a few cells of the axis out: E so close to 1 that those are kept, or that
# the band's energies alone cannot reach it
@pytest.mark.parametrize("N,W,reach,E", [(64, 6, 0.95, 1 - 1e-8), (64, 6, 0.95, 1 - 4e-8), (64, 8, 0.95, 1 - 1e-8),
                                         (64, 16, 4, 1 - 1e-8), (128, 4, 62.5, 1 - 1e-8), (128, 8, 62.5, 1 - 1e-8)])
def test_rows_whose_band_is_nearly_the_axis(N, W, reach, E):
    check_rows(N, W, reach, E, 40 if N == 64 else 10)


# the widest bands the registers hold (a reach of 63 cells and beyond goes to the whole axis) and wide windows, whose
# cells next to the band read most of their values from inside it
@pytest.mark.parametrize("N,W,reach,E", [(256, 4, 66, 0.99), (256, 16, 75, 0.999), (512, 16, 40, 0.9999), (512, 2, 20, 0.9999)])
def test_rows_at_the_widest_band(N, W, reach, E):
    check_rows(N, W, reach, E, 6)


# more rows for the whole-axis kernels than these have workgroups: every row is made, and the same as in a build of few
@pytest.mark.parametrize("N,reach,M,E", [(512, 90, 1500, 0.5), (128, 120, 2000, 0.5)])
def test_more_whole_axis_rows_than_workgroups(N, reach, M, E):
    rng = np.random.default_rng(N)
    B = N / (2 * L)
    u, v = rng.uniform(-B, B, (2, M))
    w = reach / (2 * L * L) * rng.uniform(0.9, 1.0, M)
    plan = wp.Plan(N, L)
    rows = rows_of(wp.build_G(plan, dev(u), dev(v), dev(w), E, transpose=False))
    assert sorted(rows) == list(range(M))
    for k in rng.choice(M - 40, 3, replace=False):
        few = rows_of(wp.build_G(plan, dev(u[k:k + 40]), dev(v[k:k + 40]), dev(w[k:k + 40]), E, transpose=False))
        for i in range(40):
            assert len(rows[k + i][0]) > 0
            assert np.array_equal(rows[k + i][0], few[i][0]) and np.array_equal(rows[k + i][1], few[i][1])
    check_rows(N, 4, reach, E, 4)
