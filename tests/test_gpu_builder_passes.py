"""The two passes of the builder called one by one: the fill pass makes rows of the coordinates that it is given and of the
threshold that the last count pass on the workspace left, whatever an earlier one left there, and fails where a row's
length is another than the one counted."""
import ctypes as C

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1307_3424_amd as wp  # noqa: E402
from paper_1307_3424_amd import WprojError  # noqa: E402

L = synth.fov_L()
N, M = 64, 200


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def coordinates(seed):
    rng = np.random.default_rng(seed)
    u, v = rng.uniform(-0.8 * N, 0.8 * N, (2, M)) / (2 * L)
    return u, v, 10 / (4 * L * L) * rng.uniform(0, 1, M)


class Passes:
    def __init__(self):
        self.plan = wp.Plan(N, L)
        b = C.c_int64()
        wp.check(wp.load().wp_build_workspace_bytes(self.plan.handle, M, C.byref(b)), "workspace")
        self.ws = torch.zeros(b.value, dtype=torch.uint8, device="cuda")

    def count(self, uvw, E):
        nnz, nwork = C.c_int64(), C.c_int64()
        t = [dev(a) for a in uvw]
        wp.check(wp.load().wp_build_G_count(self.plan.handle, M, *(C.c_void_p(a.data_ptr()) for a in t), float(E),
                                            C.c_void_p(self.ws.data_ptr()), C.byref(nnz), C.byref(nwork),
                                            C.c_void_p(torch.cuda.current_stream().cuda_stream)), "count")
        return nnz.value, nwork.value

    def fill(self, uvw, E, counted):
        t = [dev(a) for a in uvw]
        G = wp._new_G(self.plan, M, *counted, wp.WP_TAPS_C64, False, t[0].device)
        d = G.desc()
        wp.check(wp.load().wp_build_G_fill(self.plan.handle, M, *(C.c_void_p(a.data_ptr()) for a in t), float(E),
                                           C.c_void_p(self.ws.data_ptr()), C.byref(d),
                                           C.c_void_p(torch.cuda.current_stream().cuda_stream)), "fill")
        return rows_of(G)

    def build(self, uvw, E):
        return rows_of(wp.build_G(self.plan, *(dev(a) for a in uvw), E, transpose=False))


def rows_of(G):
    rp, perm = G.rowptr.cpu().numpy(), G.perm.cpu().numpy()
    col, val = G.col.cpu().numpy(), G.val.cpu().numpy()
    return {int(k): (col[rp[r]:rp[r + 1]], val[rp[r]:rp[r + 1]]) for r, k in enumerate(perm)}


def same(a, b):
    return sorted(a) == sorted(b) and all(np.array_equal(x, y) for k in a for x, y in zip(a[k], b[k]))


# moved by whole cells the rows are as long, but for the entry that is the threshold itself: its energy differs by rounding
@pytest.mark.parametrize("moved", [lambda u, v, w: (u, v, 0.3 * w), lambda u, v, w: (u + 3 / (2 * L), v - 5 / (2 * L), w)],
                         ids=["w", "cells"])
def test_other_coordinates_than_counted_fail(moved):
    p, uvw = Passes(), coordinates(1)
    n = p.count(uvw, 0.99)
    with pytest.raises(WprojError):
        p.fill(moved(*uvw), 0.99, n)
    n = p.count(uvw, 0.99)
    assert same(p.fill(uvw, 0.99, n), p.build(uvw, 0.99))


@pytest.mark.parametrize("before", [None, 0.9])
def test_all_entries_counted_and_filled_under_another_fraction(before):
    p, uvw = Passes(), coordinates(3)
    if before:
        p.count(uvw, before)               # leaves its candidates in the workspace
    n = p.count(uvw, 1.0)
    assert same(p.fill(uvw, 0.9, n), p.build(uvw, 1.0))
    n = p.count(uvw, 0.9)
    assert same(p.fill(uvw, 1.0, n), p.build(uvw, 0.9))


# a workspace sized for rows with a beam has always served the plan's own rows too
@pytest.mark.parametrize("n", [32, 64, 256, 512, 2048])
def test_a_workspace_for_rows_with_a_beam_holds_rows_without(n):
    plan = wp.Plan(n, L)
    for m in (1, 1000, 300000):
        b = [C.c_int64(), C.c_int64()]
        wp.check(wp.load().wp_build_workspace_bytes(plan.handle, m, C.byref(b[0])), "plain")
        wp.check(wp.load().wp_build_dde_workspace_bytes(plan.handle, m, C.byref(b[1])), "beam")
        assert b[1].value >= b[0].value
