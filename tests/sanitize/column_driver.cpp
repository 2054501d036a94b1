// Host-side code of the sweep's column form under AddressSanitizer / UndefinedBehaviorSanitizer, on grids of
// ordinary heights and tall ones: the segment lists in sweep order against the tables that they are made from, the
// partial planes' places (whole and in parts) against the rows that the lines come through, and the Jacobi tiles.
// Built with g++ by tests/test_column_plan.py.
#include <algorithm>
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

// The rows of nx elements that the lines of pair q store in its layers of a part: each in a place of its own, all within
// n_elems.
int check_places(const rt3d::SweepPlan &P, const rt3d::SweepPart &part, int64_t n_elems)
{
    std::vector<char> taken(size_t(n_elems / P.nx), 0);
    for (int q = part.q0; q < part.q1; ++q) {
        const rt3d::PairInfo &pi = P.pairs[q];
        const int rows = pi.split ? 1 : rt3d::kColumnRows, n = (P.ny + rows - 1) / rows;
        for (int step = part.step0; step < part.step0 + part.layers; ++step) {
            const int k = pi.down ? P.nz - 1 - step : step;
            const size_t ka = size_t(pi.dA) * P.nz + k;
            const rt3d::LayerBlock &lb = P.blocks[size_t(k) * P.n_pair + q];
            int moves = 0, lowest = P.seg_bi[P.seg_off[ka]];
            for (int s = 1; s < P.seg_n[ka]; ++s) {
                moves += P.seg_bi[P.seg_off[ka] + s] != P.seg_bi[P.seg_off[ka] + s - 1];
                lowest = std::min(lowest, P.seg_bi[P.seg_off[ka] + s]);
            }
            // a store at every row move and one for each row at the layer's end
            if (moves != lb.span || lb.wmu != pi.wmu || lb.rmin != ((lowest % P.ny) + P.ny) % P.ny) return 20;
            if (((lb.flags & rt3d::kBlockSplit) != 0) != (pi.split != 0) || ((lb.flags & rt3d::kBlockDown) != 0) != (pi.ysgn < 0)) return 21;
            for (int b = 0; b < n; ++b)
                for (int r = 0; r < rows + moves; ++r) {
                    const int64_t at = lb.off + (int64_t(b) * lb.stride + r) * P.nx;
                    if (at < 0 || at % P.nx || at + P.nx > n_elems || taken[size_t(at / P.nx)]++) return 22;
                }
        }
    }
    return 0;
}

int check_plan(rt3d::SweepPlan P, const rt3d::AngleSet &A)
{
    for (const int *shape : {(const int[]){512, 2}, (const int[]){256, 8}, (const int[]){1024, 2}}) {
        if (!rt3d::make_column_plan(A, shape[0], shape[1], rt3d::column_load(P.nx, P.ny, P.nz, A), P)) return 30;
        if (int rc = check_places(P, rt3d::SweepPart{0, P.n_pair, 0, P.nz}, P.p_elems)) return rc;
        // the work items hold every band of every pair once, in workgroups of the stated size
        std::vector<std::vector<char>> band(P.n_pair);
        for (const rt3d::WorkItem &it : P.items) {
            const int rows = P.pairs[it.pair].split ? 1 : rt3d::kColumnRows;
            band[it.pair].resize(size_t((P.ny + rows - 1) / rows), 0);
            if (it.rows < 1 || it.rows * P.nx > P.block_threads || it.j0 != it.band * rows) return 31;
            for (int b = it.band; b < it.band + it.rows; ++b)
                if (b >= int(band[it.pair].size()) || band[it.pair][b]++) return 32;
        }
        for (const auto &b : band)
            for (char seen : b)
                if (!seen) return 33;
        // in parts of every size from what the plan takes down to one layer of one pair
        const std::vector<rt3d::LayerStart> start = rt3d::layer_starts(P);
        int smallest = 0;
        for (int64_t room = P.p_elems + 1000; room > 0; room = room * 5 / 8) {
            rt3d::SweepPlan Q = P;
            const std::vector<rt3d::SweepPart> parts = rt3d::layer_parts(Q, room);
            if (parts.empty()) break;
            std::vector<int> step(P.n_pair, 0), pairs(P.nz, 0);
            for (const rt3d::SweepPart &part : parts) {
                const int64_t n = rt3d::lay_out(Q, part);
                if (n + rt3d::line_elems(Q, part) > room) return 40;
                if (int rc = check_places(Q, part, n)) return rc;
                for (int q = part.q0; q < part.q1; ++q) {
                    // every layer of every pair once, the layers in sweep order and a layer's pairs in theirs
                    if (step[q] != part.step0 || (P.pairs[q].down != 0) != part.down) return 41;
                    step[q] += part.layers;
                    for (int st = part.step0; st < part.step0 + part.layers; ++st)
                        if (pairs[part.down ? P.nz - 1 - st : st]++ != q) return 42;
                    const int k = part.down ? P.nz - 1 - part.step0 : part.step0;
                    const rt3d::LayerStart ls = start[size_t(k) * P.n_pair + q];
                    if (part.step0 == 0 ? ls.seg != P.pairs[q].c_off || ls.row != P.pairs[q].row0
                                        : !(P.cseg[ls.seg - 1].flags & rt3d::kLayerEnd))
                        return 43;
                }
            }
            for (int s : step)
                if (s != P.nz) return 44;
            smallest = int(parts.size());
        }
        if (smallest < P.n_pair) return 45;
    }
    return 0;
}

int check_tile(int nx, int ny, int nz)
{
    const rt3d::JacobiTile t = rt3d::choose_jacobi_tile(nx, ny, nz);
    if (t.tx < 1 || t.ty < 1 || t.z < 1 || t.tx > nx || t.ty > ny || t.z > nz) return 50;
    if (t.tx * t.ntx < nx || t.ty * t.nty < ny || t.z * t.ntz < nz) return 51;
    if (t.tx * (t.ntx - 1) >= nx || t.ty * (t.nty - 1) >= ny || t.z * (t.ntz - 1) >= nz) return 52;
    return t.threads() <= rt3d::kPairThreads && t.cells0() <= rt3d::kPairLoads * t.threads() ? 0 : 53;
}

}  // namespace

int main()
{
    const Grid grids[] = {{3, 3, 3, 2, 4, false}, {17, 17, 17, 8, 8, false}, {65, 5, 65, 16, 16, false}, {9, 12, 500, 8, 20, false}, {5, 7, 4, 8, 4, false},
                          {33, 34, 9, 16, 16, false},
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
        if (!rc && g.nz <= 500) rc = check_plan(P, A);
        if (!rc) rc = check_tile(g.nx, g.ny, g.nz);
        if (rc) {
            std::printf("%dx%dx%d %dx%d: %d\n", g.nx, g.ny, g.nz, g.nt, g.np, rc);
            return rc;
        }
    }
    for (int nx : {3, 4, 5, 17, 40, 200, 513, 1000})
        for (int ny : {3, 4, 18, 65, 300})
            for (int nz : {3, 7, 33, 129})
                if (int rc = check_tile(nx, ny, nz)) {
                    std::printf("tile of %dx%dx%d: %d\n", nx, ny, nz, rc);
                    return rc;
                }
    std::printf("column driver ok\n");
    return 0;
}
