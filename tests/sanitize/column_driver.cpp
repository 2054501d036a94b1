// Host-side code of the sweep's column form under AddressSanitizer / UndefinedBehaviorSanitizer, on grids of
// ordinary heights and tall ones: the segment lists in sweep order against the tables that they are made from.
// Built with g++ by tests/test_column_plan.py.
#include <cstdio>
#include <cstdlib>
#include <string>
#include <vector>

#include "../../paper_1107_5719_amd/csrc/geometry.h"

namespace {

struct Grid { int nx, ny, nz, nt, np; bool same_voxel; };   // same_voxel: neighbouring segments of a line share a voxel

int check_segments(const rt3d::SweepPlan &P, const rt3d::AngleSet &A, bool &same_voxel)
{
    size_t at = 0;
    for (const rt3d::PairInfo &pi : P.pairs) {
        if (pi.c_off != int(at)) return 10;
        const size_t end = at + size_t(pi.n_seg);
        int i = 0, j = 0;
        for (int st = 0; st < P.nz; ++st) {
            const size_t ka = size_t(pi.dA) * P.nz + (pi.down ? P.nz - 1 - st : st);
            for (int s = 0; s < P.seg_n[ka]; ++s, ++at) {
                const int o = P.seg_off[ka] + s;
                if (at >= end || P.cseg[at].len != P.seg_len[o]) return 11;
                if (((P.cseg[at].flags & rt3d::kLayerEnd) != 0) != (s + 1 == P.seg_n[ka])) return 12;
                if (st > 0 || s > 0) {
                    // at most one column and one row on, always in the direction that the line drifts to
                    const int di = P.seg_ai[o] - i, dj = P.seg_bi[o] - j, f = P.cseg[at - 1].flags;
                    if (di != ((f & rt3d::kNextColumn) ? pi.xsgn : 0) || dj != ((f & rt3d::kNextRow) ? pi.ysgn : 0)) return 13;
                    same_voxel = same_voxel || f == 0;
                }
                i = P.seg_ai[o];
                j = P.seg_bi[o];
            }
        }
        if (at != end || (P.cseg[at - 1].flags & ~rt3d::kLayerEnd)) return 14;
        if (A.ox[pi.dA] * pi.xsgn <= 0.0 || A.oy[pi.dA] * pi.ysgn <= 0.0) return 15;
    }
    return at == P.cseg.size() ? 0 : 16;
}

}  // namespace

int main()
{
    const Grid grids[] = {{3, 3, 3, 2, 4, false}, {17, 17, 17, 8, 8, false}, {65, 5, 65, 16, 16, false}, {9, 12, 500, 8, 20, false},
                          {12, 11, 1200, 4, 12, false}, {15, 15, 3000, 8, 20, true}, {15, 15, 4000, 8, 4, true}, {6, 7, 2700, 16, 4, true}};
    for (const Grid &g : grids) {
        rt3d::AngleSet A;
        rt3d::SweepPlan P;
        std::string err;
        if (!rt3d::make_angle_set(g.nt, g.np, A) ||
            !rt3d::build_sweep_plan(g.nx, g.ny, g.nz, A, 1024, 8192, 48 * 1024, P, err))
            return 1;
        bool same = false, shortest = false;
        int rc = check_segments(P, A, same);
        for (double l : P.seg_len) shortest = shortest || l < 1e-11;
        // Lambda* by tiles and by symmetry asks for a plan without slivers
        if (!rc && (same != g.same_voxel || (same && !P.slivers) || (shortest && !P.slivers) || (g.nz <= 500 && P.slivers))) rc = 17;
        if (rc) {
            std::printf("%dx%dx%d %dx%d: %d\n", g.nx, g.ny, g.nz, g.nt, g.np, rc);
            return rc;
        }
    }
    std::printf("column driver ok\n");
    return 0;
}
