"""GPU test of the allocation-free formal solution on grids whose partial planes do not fit its workspace at once: parts of
layers, with bands of 1 to 4 rows, pairs split and whole, sums of chunks of pairs carried on (up to 2^19 voxels) or not,
and fewer pairs at a time near the largest grid.  Bitwise what a context gives.  A slab of three layers of very many rows
takes the window form there, whose sums differ by rounding: N 2^-52 with N = 100 roundings in a line of 30 segments and
the sum of its deposits."""
import pytest

pytestmark = pytest.mark.gpu

CASES = [
    # (nz, ny, nx), n_theta, n_phi, I_top, bottom_bc, bitwise
    ((81, 80, 79), 16, 16, 0.3, 0, True),
    ((60, 65, 129), 16, 16, 0.0, 1, True),
    ((300, 34, 33), 16, 16, 0.2, 0, True),
    ((129, 130, 131), 8, 8, 0.1, 0, True),
    ((9, 300, 511), 8, 20, 0.0, 0, True),
    ((160, 199, 200), 8, 8, 0.0, 0, True),        # 102 of 128 MiB hold the medium
    ((130, 300, 3), 16, 16, 0.2, 0, True),
    ((40, 60, 600), 8, 8, 0.1, 0, True),          # rows of more than 512 columns: parts of pairs
    ((3, 109056, 16), 8, 8, 0.1, 0, False),
]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}-{c[1]}x{c[2]}" for c in CASES])
def test_noalloc_in_parts(case):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1107_5719_amd import rt3d as R

    (nz, ny, nx), nt, nph, I_top, bbc, bitwise = case
    gen = torch.Generator(device="cuda").manual_seed(nx)

    def field(lo, hi):
        return lo + (hi - lo) * torch.rand((nz, ny, nx), generator=gen, dtype=torch.float64, device="cuda")

    chi, S, B = 10.0 ** field(-3.0, 1.0), field(0.1, 3.0), field(0.5, 1.5)
    ref, out = torch.empty_like(chi), torch.full_like(chi, float("nan"))
    with R.Solver(nx, ny, nz, nt, nph, I_top=I_top, bottom_bc=bbc) as s:
        s.set_medium(chi, torch.full_like(chi, 0.1), B)
        s.formal_solution(S, ref)
    for _ in range(2):
        R.rt3d_formal_solution_noalloc(nx, ny, nz, nt, nph, chi, S, B[0].contiguous(), out, I_top=I_top, bottom_bc=bbc)
        worst = float(((out - ref).abs() / ref).max())
        assert torch.equal(out, ref) if bitwise else worst <= 100 * 2.0**-52, worst
        out.fill_(float("nan"))
