"""GPU test of Lambda* on tall grids with lines through voxel edges (n_phi = 12, 20): rounding leaves slivers between
the x and the y face there, which may lie in the voxel of the segment before and which opposite directions need not share.

The medium has one opacity, so an entry depends on its layer alone and a walk over the library's own segment tables gives
it.  Both sides take the same products chi * length, so they differ by the exponentials' rounding: at most four factors,
each off by an ulp of its optical depth (below 400 here, so 1e-13) or by 3e-15, in sums of terms of one sign.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

CASES = [
    # (nz, ny, nx), n_theta, n_phi, chi, layers
    ((3000, 15, 15), 8, 20, 30.0, range(100, 125)),      # two segments in one voxel
    ((3000, 15, 15), 8, 20, 30.0, (0, 9, 2998, 2999)),
    ((1200, 11, 12), 4, 12, 30.0, range(250, 265)),      # slivers in a voxel of their own
    ((4000, 15, 15), 8, 4, 10.0, range(340, 350)),       # walks of more than three steps
    ((2700, 7, 6), 16, 4, 30.0, range(45, 60)),          # lines wrap back within two layers
]


def _walks(R, nx, ny, nz, nt, nph, chi, k):
    """The 27 entries of a voxel of layer k: over the segments in it, back along the line to those before."""
    desc = R._desc(nx, ny, nz, nt, nph)
    mu, _, _, w = R.rt3d_quadrature(nt, nph)
    L = np.zeros(27)
    for d in range(nt * nph):
        wmu, up = w[d] * abs(mu[d]), k + 1 if mu[d] < 0 else k - 1
        line = []
        for kk in (up, k):
            if 0 <= kk < nz:
                line += [(i, j, kk, l) for i, j, l in zip(*R.rt3d_segment_table(desc, d, kk))]
        n_up = sum(1 for s in line if s[2] == up)
        for q in range(n_up, len(line)):
            i, j, _, length = line[q]
            x = chi * length
            em1 = np.expm1(-x)
            L[13] += wmu * (x + em1 if x > 0.5 else sum((-1) ** n * x**n / np.prod(np.arange(1.0, n + 1)) for n in range(18, 1, -1)))
            T = 1.0
            for bi, bj, kk, bl in reversed(line[:q]):
                di, dj = int(bi - i), int(bj - j)
                oi = [o for o in (-1, 0, 1) if (di - o) % nx == 0]
                oj = [o for o in (-1, 0, 1) if (dj - o) % ny == 0]
                if oi and oj:
                    L[9 * (kk - k + 1) + 3 * (oj[0] + 1) + oi[0] + 1] += wmu * em1 * np.expm1(-chi * bl) * T
                T *= np.exp(-chi * bl)
                if T < 1e-250:
                    break
    return L / chi


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}-{c[1]}x{c[2]}-{min(c[4])}" for c in CASES])
def test_lstar_of_tall_grids(case):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1107_5719_amd import rt3d as R

    (nz, ny, nx), nt, nph, chi, layers = case
    one = torch.ones((nz, ny, nx), dtype=torch.float64, device="cuda")
    out = torch.empty((27, nz, ny, nx), dtype=torch.float64, device="cuda")
    with R.Solver(nx, ny, nz, nt, nph) as s:
        s.set_medium(one * chi, one * 0.1, one)
        s.build_lstar()
        s.get_lstar(out)
    for k in layers:
        got, ref = out[:, k].cpu().numpy(), _walks(R, nx, ny, nz, nt, nph, chi, k)[:, None, None]
        assert np.all(np.abs(got - ref) <= 1e-12 * np.abs(ref) + 1e-290), \
            (k, np.max(np.abs(got / np.where(ref == 0.0, 1.0, ref) - 1.0), axis=(1, 2)))
