"""GPU tests of the column form of the sweep (rows of up to 512 columns) and its reduction at the edges of their tiles.

Rows around one, two and eight wavefronts and the first row length that takes the other form; bands whose last
one holds 1, 2, 3 or 4 line rows; pairs split into single line rows (the small grids; shape 1 splits none), whole,
and both in one launch (33 x 34 with 16 x 16 angles).  Split or whole, and whatever the workgroup's size, the sums
have one order, so shapes agree bitwise; float64 is compared with the oracle at rel 1e-10, float32 at N 2^-22 of
the largest intensity, N the most segments of a line: each adds about four roundings of at most 2^-24 (chi, S, the
exponential, the sum) to the intensity it carries on.
"""
import numpy as np
import pytest

from paper_1107_5719_amd.inputs import random_medium

pytestmark = pytest.mark.gpu

CASES = [
    # (nz, ny, nx), n_theta, n_phi, I_top, bottom_bc
    ((4, 3, 3), 16, 16, 0.3, 0),
    ((3, 6, 16), 8, 8, 0.0, 0),
    ((5, 9, 17), 8, 8, 0.2, 1),
    ((5, 34, 33), 16, 16, 0.1, 0),
    ((3, 5, 63), 16, 8, 0.0, 0),
    ((3, 7, 64), 8, 16, 0.4, 0),
    ((4, 8, 65), 16, 16, 0.2, 0),
    ((3, 11, 128), 8, 8, 0.1, 0),
    ((3, 10, 129), 8, 8, 0.0, 1),
    ((3, 5, 512), 8, 8, 0.2, 0),
    ((3, 5, 513), 8, 8, 0.2, 0),
    # the reduction's chunks of pairs: 3 pairs, 18 in chunks of 4, 200 in chunks of 16; rows of even and odd length
    ((4, 7, 10), 2, 12, 0.1, 0),
    ((5, 12, 11), 6, 12, 0.2, 0),
    ((3, 6, 8), 20, 20, 0.0, 1),
]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}-{c[1]}x{c[2]}" for c in CASES])
def test_column_sweep(orc, case):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.zeros(1, device="cuda")
    from paper_1107_5719_amd import rt3d as R

    (nz, ny, nx), nt, nph, I_top, bbc = case
    m = random_medium(nx, ny, nz, seed=nx, chi_range=(1e-3, 3e1))
    S = np.random.default_rng(nx).uniform(0.1, 3.0, (nz, ny, nx))
    I_bot = m["B"][0] if bbc != 1 else None
    J_orc, Iem_orc = orc.formal_solution(m["chi"], S, nt, nph, I_top=I_top, I_bot=I_bot, want_emergent=True)
    mu, ox, oy, _ = orc.quadrature(nt, nph)
    n_seg = nz * (1 + np.max((np.abs(ox) + np.abs(oy)) / np.abs(mu))) + 2
    top = max(3.0, I_top, 0.0 if I_bot is None else float(np.max(I_bot)))
    for precision in (0, 1):
        first = None
        for shape in (0, 1, 5) if nx <= 512 else (0, 1):   # (shape 5 refuses rows of more than 512 columns)
            with R.Solver(nx, ny, nz, nt, nph, I_top=I_top, bottom_bc=bbc, precision=precision) as s:
                s.set_sweep_shape(shape)
                s.set_medium(m["chi"], m["eps"], m["B"])
                J, Iem = s.formal_solution(S), s.emergent_top()
            for got, ref in ((J, J_orc), (Iem, Iem_orc)):
                lim = 1e-10 * np.abs(ref) + 1e-300 if precision == 0 else n_seg * 2.0**-22 * top
                assert np.all(np.abs(got - ref) <= lim), (precision, shape, np.max(np.abs(got - ref)))
            if first is None:
                first = (J, Iem)
            elif nx <= 512:
                assert np.array_equal(J, first[0]) and np.array_equal(Iem, first[1]), (precision, shape)
