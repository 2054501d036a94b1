"""GPU test of the tiled form of Lambda* (grids whose lines cannot wrap back within two layers, at least 16
direction pairs) against the oracle, at the edges of its tiles (254 threads with a halo of one column to each
side): one tile and several, rows that end a tile and rows that start one, the thinnest grid; and next to it a grid
that is one column too narrow for it.  Bars as in the other Lambda* tests; the lower neighbours' entries and half
of the in-plane ones come from the symmetry of chi_v Lambda*_vu, which costs two roundings more.
"""
import numpy as np
import pytest

from lstar_bar import close_lstar
from paper_1107_5719_amd.inputs import random_medium

pytestmark = pytest.mark.gpu

CASES = [
    # (nz, ny, nx), n_theta, n_phi, precision; lines of 8 polar angles drift at most 5.4 columns per layer
    ((3, 15, 15), 8, 8, 0),
    ((3, 15, 14), 8, 8, 0),      # too narrow: voxel by voxel
    ((5, 16, 31), 8, 8, 1),
    ((4, 18, 62), 8, 8, 0),
    ((3, 29, 65), 8, 16, 0),
    ((6, 16, 130), 8, 8, 0),
    ((4, 26, 27), 16, 16, 0),
]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}-{c[1]}x{c[2]}-{c[3]}" for c in CASES])
def test_lstar_tile(orc, case):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.zeros(1, device="cuda")
    from paper_1107_5719_amd import rt3d as R

    (nz, ny, nx), nt, nph, precision = case
    m = random_medium(nx, ny, nz, seed=nx + ny, chi_range=(1e-4, 1e2))
    with R.Solver(nx, ny, nz, nt, nph, precision=precision) as s:
        s.set_medium(m["chi"], m["eps"], m["B"])
        s.build_lstar()
        L = s.get_lstar()
        with R.Batch([{"nx": nx, "ny": ny, "nz": nz, "n_theta": nt, "n_phi": nph}], precision=precision) as b:
            b.set_medium(0, m["chi"], m["eps"], m["B"])
            b.set_J(0, m["B"])
            s.set_J(m["B"])
            b.solve(tol=10.0, max_iter=2, inner_sweeps=3)
            s.solve(tol=10.0, max_iter=2, inner_sweeps=3)
            assert np.array_equal(b.get_J(0), s.get_J())
    close_lstar(L, orc.lstar(m["chi"], nt, nph), m["chi"], nt)
