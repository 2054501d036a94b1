"""GPU test that timing every launch (mode 1) times the launches that an untimed step makes: as many of two Jacobi sweeps,
each counted as two, and the same iterates."""
import numpy as np
import pytest

from paper_1107_5719_amd.inputs import random_medium

pytestmark = pytest.mark.gpu


def test_timing_changes_no_launch():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.zeros(1, device="cuda")
    from paper_1107_5719_amd import rt3d as R

    m = random_medium(17, 16, 15, seed=3)
    out = []
    for mode in (0, 1, 2):
        with R.Solver(17, 16, 15, 4, 8) as s:
            s.set_medium(m["chi"], m["eps"], m["B"])
            s.set_timing(mode)
            for sweeps in (6, 7):
                s.os_step(sweeps)
            st = s.stats()
            k = st["kernels"]["jacobi"]
            assert k["launches"] == 13 and k["timed"] == (0, 13, 9)[mode] and (k["total_ms"] > 0) == (mode > 0)
            out.append((s.get_J(), st["jacobi_pairs"]))
    # 6 sweeps are three pairs, 7 one sweep and three pairs; mode 2: the first and the last apart
    assert [n for _, n in out] == [6, 6, 4]
    assert all(np.array_equal(J, out[0][0]) for J, _ in out)
