"""GPU test that the adjoint's line kernels take exponentials that are good to an ulp.

With eps = 1 nothing scatters and dL/deps = a (B - J), a the sum of q (1 - e^-dtau) over the lines through a voxel.  In
the top layer of a medium of one opacity, with 2 x 4 angles, a is 4 (1 - e^-x)(1 + e^-x) g: every line has two halves
there.  The depths x are those where a table of 2^(j/16) alone is off by up to 2.7e-15.  About 19 roundings (the exponential's
two, x, eight terms and their sum, five on the way to nu, three in the result) of at most 1.1e-16, spread evenly: 2.8e-16
rms, and 1.2e-15 is four times that."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_gradient_of_thin_segments():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1107_5719_amd import rt3d as R

    nx, ny, nz = 5, 4, 3
    length = 0.5 / abs(R.rt3d_quadrature(2, 4)[0][0])
    one = np.ones((nz, ny, nx))
    worst = 0.0
    for x in np.linspace(0.02167, 0.0225, 24):
        chi = x / length
        with R.Solver(nx, ny, nz, 2, 4, bottom_bc=1) as s:
            s.set_medium(one * chi, one, one)
            s.solve(1e-14, 10, 2)
            J = s.get_J()
            _, deps, status, *_ = s.adjoint(np.ones((4, ny, nx)), 1e-14, 10, 2)
        dt = np.longdouble(chi) * np.longdouble(length)
        a = 4 * -np.expm1(-dt) * (1 + np.exp(-dt))
        ref = a * (np.longdouble(1.0) - J[-1].astype(np.longdouble))
        worst = max(worst, float(np.max(np.abs(deps[-1] / ref - 1))))
    assert status == R.RT3D_OK and worst <= 1.2e-15, worst
