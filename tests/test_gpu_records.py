"""Products from the factor records where one form hands over to another: few and many rows, rows too long for the
packed lanes, taps outside the tile's window, rows at the grid's edges, and values the fixed-point window cannot hold.

The reference is the stored taps of the same G in FP64.  Tolerance: a product sums at most a few thousand terms in
FP32, each with a handful of roundings of 2^-24, errors adding as their square root: below 1e-6 of the result's norm.
"""
import numpy as np
import pytest
import scipy.sparse as sp

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1307_3424_amd as wp  # noqa: E402

L = synth.fov_L()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def problem(N, M, spread, seed=0):
    rng = np.random.default_rng([N, M, seed])
    u, v, w = synth.uvw(N, M, L, "gaussian" if M > 64 else "uniform", 0.25, spread / (4 * L * L), rng)
    B = N / (2 * L)
    u[0], v[0] = -B * (1 - 1e-6), B * (1 - 1e-6)                  # the record wraps around both axes
    plan = wp.Plan(N, L)
    full = wp.build_G(plan, dev(u), dev(v), dev(w), 0.99, transpose=False)
    G = wp.build_G(plan, dev(u), dev(v), dev(w), 0.99, factors=True, transpose=False, stored=False)
    Ng = plan.Ng
    A = sp.csr_matrix((full.val.cpu().numpy().astype(np.complex128), full.col.cpu().numpy(),
                       full.rowptr.cpu().numpy()), shape=(M, Ng * Ng))
    return plan, G, A, G.perm.cpu().numpy(), rng


# 24576 rows is where packed lanes take over; one row; rows of up to 10000 taps, one to a wavefront; supports beyond
# the window's halo
@pytest.mark.parametrize("N,M,spread", [(32, 1, 28), (64, 3, 120), (32, 24575, 20), (32, 24576, 28), (256, 30001, 28),
                                        (64, 24576, 100), (512, 2000, 60), (1024, 700, 28)])
@pytest.mark.parametrize("order", [wp.WP_ORDER_CALLER, wp.WP_ORDER_SORTED])
def test_record_products_match_stored_taps(N, M, spread, order):
    plan, G, A, perm, rng = problem(N, M, spread)
    G.order = order
    X = synth.random_complex(plan.Ng ** 2, rng)
    y = synth.random_complex(M, rng)
    at = perm if order == wp.WP_ORDER_CALLER else np.arange(M)    # row r's entry of a visibility vector
    z = wp.degrid(plan, G, dev(X.astype(np.complex64))).cpu().numpy()[at]
    ref = A @ X.astype(np.complex64)
    assert np.linalg.norm(z - ref) <= 1e-6 * np.linalg.norm(ref)
    g = wp.grid_scatter(plan, G, dev(y.astype(np.complex64))).cpu().numpy()
    ref = A.conj().T @ y.astype(np.complex64)[at]
    assert np.linalg.norm(g - ref) <= 1e-6 * np.linalg.norm(ref)


@pytest.mark.parametrize("scale", [0.0, 1e-34, 1e30])
def test_scatter_of_very_small_and_large_values(scale):
    plan, G, A, perm, rng = problem(64, 500, 28)
    y = (scale * synth.random_complex(500, rng)).astype(np.complex64)
    g = wp.grid_scatter(plan, G, dev(y)).cpu().numpy().astype(np.complex128)
    ref = A.conj().T @ y[perm].astype(np.complex128)
    assert np.linalg.norm(g - ref) <= 1e-6 * np.linalg.norm(ref)


def test_scatter_keeps_a_value_that_is_not_finite():
    plan, G, A, perm, rng = problem(64, 500, 28)
    y = synth.random_complex(500, rng).astype(np.complex64)
    y[perm[250]] = np.inf
    g = wp.grid_scatter(plan, G, dev(y)).cpu().numpy()
    hit = A.indices[A.indptr[250]:A.indptr[251]]
    rest = np.setdiff1d(np.arange(g.size), hit)
    y[perm[250]] = 0
    ref = A.conj().T @ y[perm].astype(np.complex128)
    assert not np.isfinite(g[hit]).any()
    assert np.linalg.norm(g[rest] - ref[rest]) <= 1e-6 * np.linalg.norm(ref[rest])
