"""A faint visibility beside bright ones of the same tile, gridded from the factor records: the window's fixed-point unit
is at most 2^-61 of the sum over the rows of |y| times the row's largest tap.

Bound on a cell's error: half a unit a tap that falls on it, and FP32 rounding, six roundings of 2^-24 a term (the two
products of two terms each, the sum, the value flushed).
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


@pytest.mark.parametrize("W", [2, 4, 16])
@pytest.mark.parametrize("faint", [1e-9, 1e-13])
def test_faint_beside_bright(W, faint):
    N, M = 64, 96
    rng = np.random.default_rng(W)
    at = rng.uniform(-27, -26, (2, M))                           # grid coordinates: one tile, cells -32 .. -1
    at[:, 50] = -8.3, -7.6                                       # far enough for cells of its own
    plan = wp.Plan(N, L, kb_W=W)
    uvw = [dev(a) for a in (at[0] / (2 * L), at[1] / (2 * L), np.zeros(M))]
    full = wp.build_G(plan, *uvw, 0.99, transpose=False)
    G = wp.build_G(plan, *uvw, 0.99, factors=True, transpose=False, stored=False)
    A = sp.csr_matrix((full.val.cpu().numpy().astype(np.complex128), full.col.cpu().numpy(),
                       full.rowptr.cpu().numpy()), shape=(M, plan.Ng ** 2))
    y = synth.random_complex(M, rng).astype(np.complex64)
    y[50] *= np.float32(faint)
    got = wp.grid_scatter(plan, G, dev(y)).cpu().numpy().astype(np.complex128)
    ys = y[G.perm.cpu().numpy()].astype(np.complex128)
    ref = A.conj().T @ ys
    peak = np.maximum.reduceat(np.abs(A.data), A.indptr[:-1])
    unit = 2.0 ** -61 * float(np.abs(ys) @ peak)
    taps = np.asarray((A != 0).sum(0)).ravel()
    bound = 0.5 * unit * taps + 6 * 2.0 ** -24 * (abs(A).T @ np.abs(ys))
    err = np.maximum(np.abs((got - ref).real), np.abs((got - ref).imag))
    own = (taps == 1) & (np.abs(ref) > 0) & (np.abs(ref) < 1e-6 * np.abs(ref).max())
    assert own.any()                                             # cells of the faint one alone
    assert np.all(err <= bound)
