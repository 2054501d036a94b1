"""GPU test of the autotuner with the sweep's column form: entries of the window form in a cache (which older files hold
for the same grids) do not decide, and shapes that run the same kernels are timed once, so that the choice between them is
not left to noise."""
import json

import numpy as np
import pytest

from paper_1107_5719_amd.inputs import random_medium

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [False, True])
def test_autotune_of_the_column_form(batch, tmp_path):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    torch.zeros(1, device="cuda")
    from paper_1107_5719_amd import rt3d as R

    nx, ny, nz = 17, 18, 19
    m = random_medium(nx, ny, nz, seed=1)
    grid = {"nx": nx, "ny": ny, "nz": nz, "n_theta": 8, "n_phi": 8}
    path = str(tmp_path / "cache.json")

    def handle():
        h = R.Batch([grid, grid]) if batch else R.Solver(**grid)
        for i in range(2 if batch else 1):
            h.set_medium(*((i,) if batch else ()), m["chi"], m["eps"], m["B"])
        return h

    with handle() as h:
        shape, ms = h.autotune(path)[:2]
    ms = np.array(ms)
    # 512 x 2, 1024 x 2 and 256 x 2 split the same pairs, the other three none, in workgroups of single waves
    assert ms[0] == ms[3] == ms[5] > 0 and ms[1] == ms[2] == ms[4] > 0 and shape in (0, 1)
    (key, entry), = json.load(open(path)).items()
    assert key.endswith("|columns")
    with open(path, "w") as f:
        f.write('{\n"%s": {"shape": 4}\n}\n' % key[:-len("|columns")])
    with handle() as h:
        shape, ms = h.autotune(path)[:2]
        assert np.all(np.array(ms) > 0) and shape in (0, 1)
    with handle() as h:
        again, ms = h.autotune(path)[:2]
        assert again == shape and np.all(np.array(ms) < 0)
    assert len(json.load(open(path))) == 2
