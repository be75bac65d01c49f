"""Grid transforms at every supported size (each has its own radices, rows and columns per block) against numpy in
double precision.

Tolerance.  A transform of Ng x Ng points is 2 log2(Ng) levels of additions, each rounding every value once by at most
u = 2^-24 of its size and independently, and fewer twiddle products than that with two roundings each (value and
twiddle): relative error in the 2-norm at most sqrt(2 log2(Ng) (1 + 2)) u, and the apodisation's product another u.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_1307_3424_amd as wp  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("aphys", [wp.WP_APHYS_ONE, wp.WP_APHYS_INV_N])
@pytest.mark.parametrize("N", [32, 64, 128, 256, 512, 1024, 2048])
def test_grid_transforms(N, aphys):
    plan = wp.Plan(N, 0.4, aphys=aphys)
    Ng = 2 * N
    rng = np.random.default_rng(N)

    def cplx(*s):
        return (rng.standard_normal(s) + 1j * rng.standard_normal(s)).astype(np.complex64)

    # the adjoint of a unit value in the grid's centre is the apodisation itself, with no rounding
    d = torch.zeros(Ng, Ng, dtype=torch.complex64, device="cuda")
    d[N, N] = 1
    a = wp.grid_adjoint(plan, d).cpu().numpy().reshape(N, N)
    assert np.all(a.imag == 0) and a.real.max() > 0
    a = a.real.astype(np.float64)
    tol = (np.sqrt(6 * np.log2(Ng)) + 1) * 2.0 ** -24

    x = cplx(N, N)
    z = np.zeros((Ng, Ng), np.complex128)
    z[N // 2:N // 2 + N, N // 2:N // 2 + N] = x * a
    want = np.fft.fftshift(np.fft.fft2(np.fft.ifftshift(z)))
    got = wp.grid_forward(plan, torch.from_numpy(x).cuda()).cpu().numpy().reshape(Ng, Ng)
    assert np.linalg.norm(got - want) <= tol * np.linalg.norm(want)

    g = cplx(Ng, Ng)
    want = np.fft.fftshift(np.fft.ifft2(np.fft.ifftshift(g.astype(np.complex128)))) * Ng * Ng
    want = want[N // 2:N // 2 + N, N // 2:N // 2 + N] * a
    got = wp.grid_adjoint(plan, torch.from_numpy(g).cuda()).cpu().numpy().reshape(N, N)
    assert np.linalg.norm(got - want) <= tol * np.linalg.norm(want)
