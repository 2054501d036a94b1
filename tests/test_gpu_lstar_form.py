"""GPU test that the form of Lambda* depends on the problem alone: with few direction pairs (4, 8, 12 and 16), whose
partial planes take more or less memory as pairs are split or not, the sweep shapes and a member of a large batch (which
splits none of the small grid's pairs) build the entries of a single context bit by bit; and that the tiles end where lines can
wrap back onto a neighbour within two layers."""
import numpy as np
import pytest

from lstar_bar import close_lstar
from paper_1107_5719_amd.inputs import random_medium

pytestmark = pytest.mark.gpu

CASES = [((33, 33, 33), 2, 12), ((20, 20, 20), 6, 4), ((12, 12, 12), 2, 12), ((17, 18, 19), 2, 8), ((20, 20, 20), 2, 4), ((9, 20, 21), 8, 4)]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}-{c[1]}x{c[2]}" for c in CASES])
def test_lstar_has_one_form(case):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1107_5719_amd import rt3d as R

    (nz, ny, nx), nt, nph = case
    m = random_medium(nx, ny, nz, seed=nx, chi_range=(1e-3, 3e1), eps_range=(1e-3, 0.3))
    out = {}
    for shape in (0, 1):
        with R.Solver(nx, ny, nz, nt, nph) as s:
            s.set_sweep_shape(shape)
            s.set_medium(m["chi"], m["eps"], m["B"])
            s.set_J(m["B"])
            s.build_lstar()
            L = s.get_lstar()
            s.solve(tol=10.0, max_iter=2, inner_sweeps=3)
            out[shape] = (L, s.get_J())
    big = {"nx": 97, "ny": 97, "nz": 97, "n_theta": nt, "n_phi": nph}
    with R.Batch([dict(big, nx=nx, ny=ny, nz=nz)] + [big] * 3) as b:
        one = torch.ones((97, 97, 97), dtype=torch.float64, device="cuda")
        for i in range(1, 4):
            b.set_medium(i, one, one * 0.1, one)
        b.set_medium(0, m["chi"], m["eps"], m["B"])
        b.set_J(0, m["B"])
        b.solve(tol=10.0, max_iter=2, inner_sweeps=3)
        J = b.get_J(0)
    assert np.array_equal(out[0][0], out[1][0])
    assert np.array_equal(out[0][1], out[1][1])
    assert np.array_equal(out[0][1], J)


@pytest.mark.parametrize("nt,nph,axis", [(8, 8, 0), (8, 8, 1), (4, 12, 0)])
def test_tiles_end_where_lines_wrap(orc, nt, nph, axis):
    """Rows (columns) of more than twice the largest drift per layer and four hold tiles, one column less does not."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.zeros(1, device="cuda")
    from paper_1107_5719_amd import rt3d as R

    mu, ox, oy, _ = R.rt3d_quadrature(nt, nph)
    least = int(np.floor(2.0 * np.max(np.abs((ox, oy)[axis] / mu)) + 4.0)) + 1
    for n, form in ((least, "tiles"), (least - 1, "symmetric")):
        shape = [3, 31, 31]
        shape[2 - axis] = n
        nz, ny, nx = shape
        m = random_medium(nx, ny, nz, seed=n, chi_range=(1e-4, 1e2))
        with R.Solver(nx, ny, nz, nt, nph) as s:
            assert s.stats()["lstar_form"] == form
            s.set_medium(m["chi"], m["eps"], m["B"])
            s.build_lstar()
            close_lstar(s.get_lstar(), orc.lstar(m["chi"], nt, nph), m["chi"], nt)
    with R.Solver(31, 31, 3, 2, 8) as s:
        assert s.stats()["lstar_form"] == "full"
