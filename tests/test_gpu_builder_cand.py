"""The builder's fill pass at the row from which the count pass leaves no candidates: the same visibility on either
side of it gives the same row, bit for bit, in taps of every kind and in the factor records."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_1307_3424_amd as wp  # noqa: E402

L = synth.fov_L()
ROWS = 1 << 18                                                    # rows with room for their candidates


@pytest.mark.parametrize("taps", [wp.WP_TAPS_C64, wp.WP_TAPS_BF16, wp.WP_TAPS_I16])
@pytest.mark.parametrize("spread,extra", [(6, 300), (50, 1)])
def test_rows_past_the_room_for_candidates(taps, spread, extra):
    N = 32
    rng = np.random.default_rng(spread)
    u, v = rng.uniform(-N, N, (2, ROWS)) / (2 * L) * 0.999
    w = np.full(ROWS, 1.0) * 4 / (4 * L * L)
    w[:extra] = spread / (4 * L * L) * rng.uniform(0.5, 1.0, extra)
    u, v, w = (torch.from_numpy(np.concatenate([a, a[:extra]])).cuda() for a in (u, v, w))
    plan = wp.Plan(N, L)
    G = wp.build_G(plan, u, v, w, 0.9, taps=taps, transpose=False, factors=taps == wp.WP_TAPS_C64)
    rp, perm = G.rowptr.cpu().numpy(), G.perm.cpu().numpy()
    at = np.empty(ROWS + extra, dtype=np.int64)
    at[perm] = np.arange(ROWS + extra)                            # sorted row of a visibility
    val = torch.view_as_real(G.val) if G.val.is_complex() else G.val
    for k in range(extra):
        a, b = at[k], at[ROWS + k]
        assert rp[a + 1] - rp[a] == rp[b + 1] - rp[b] > 0
        sa, sb = slice(rp[a], rp[a + 1]), slice(rp[b], rp[b + 1])
        assert torch.equal(G.col[sa], G.col[sb]) and torch.equal(val[sa], val[sb])
        if taps == wp.WP_TAPS_I16:
            assert G.rscale[a] == G.rscale[b]
        if G.frec is not None:
            f = [int(G.frec[i]) for i in (a, a + 1, b, b + 1)]
            assert torch.equal(G.fdat[f[0]:f[1]], G.fdat[f[2]:f[3]])
