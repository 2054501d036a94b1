"""GPU test of the Jacobi launches that do two sweeps: OS steps of even and odd numbers of sweeps agree bitwise with single
sweeps (which the layouts of RT3D_JACOBI_XCD other than the default one take), on grids of one tile, of tiles that
divide the axes and of ragged last ones, thin in each direction, and on both sides of the size limit for float
coefficients (3 * 2^16 voxels)."""
import numpy as np
import pytest

from paper_1107_5719_amd.inputs import random_medium

pytestmark = pytest.mark.gpu

CASES = [((3, 3, 3), 0), ((3, 4, 5), 1), ((17, 17, 17), 0), ((10, 9, 37), 0), ((5, 70, 6), 1), ((40, 3, 11), 0), ((3, 5, 200), 1),
         ((33, 65, 40), 0), ((58, 58, 58), 1), ((59, 58, 58), 1)]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}-{c[1]}" for c in CASES])
def test_two_sweeps_are_two_sweeps(case, monkeypatch):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.zeros(1, device="cuda")
    from paper_1107_5719_amd import rt3d as R

    (nz, ny, nx), precision = case
    m = random_medium(nx, ny, nz, seed=nx, chi_range=(1e-3, 3e1), eps_range=(1e-4, 0.3))
    out = []
    for layout in ("4", "2"):
        monkeypatch.setenv("RT3D_JACOBI_XCD", layout)
        with R.Solver(nx, ny, nz, 2, 8, precision=precision) as s:
            s.set_medium(m["chi"], m["eps"], m["B"])
            s.set_J(m["B"] * 0.5 + 0.25)
            cs = [s.os_step(n) for n in (1, 2, 5, 8)]
            s.set_timing(2)
            cs += [s.os_step(n) for n in (2, 5, 8)]
            out.append((s.get_J(), cs, s.stats()["kernels"]["jacobi"]["launches"]))
    assert np.array_equal(out[0][0], out[1][0])
    assert out[0][1] == out[1][1] and out[0][2] == out[1][2]
