// Host-side geometry of the HIP library: the angle set, the per-direction segment tables of the
// line family and the band plan of the sweep kernel.
//
// Every line of a direction is the same line translated by an integer number of columns (the lines
// go through the voxel centres (i+1/2, j+1/2) on the top plane and the grid is uniform and periodic
// in x,y), so one table per (direction, layer) describes every line: the column offsets of its
// segments relative to the line's own top column, and their lengths.
#include "geometry.h"

#include <algorithm>
#include <cmath>
#include <limits>
#include <numeric>

namespace rt3d {

namespace {

// Number of eigenvalues below x of the symmetric tridiagonal matrix with zero diagonal and squared
// off-diagonals b2[1..n-1] (LDL^T pivots of T - x I; Sylvester's law of inertia).
int sturm_count(int n, const std::vector<double> &b2, double x)
{
    int cnt = 0;
    double piv = -x;
    if (piv < 0.0) ++cnt;
    for (int k = 1; k < n; ++k) {
        if (piv == 0.0) piv = 1e-300;
        piv = -x - b2[k] / piv;
        if (piv < 0.0) ++cnt;
    }
    return cnt;
}

}  // namespace

bool gauss_legendre(int n, std::vector<double> &x, std::vector<double> &w)
{
    if (n < 2) return false;
    // Jacobi matrix of the Legendre polynomials: zero diagonal, off-diagonal k / sqrt(4k^2 - 1).
    std::vector<double> b2(n, 0.0);
    for (int k = 1; k < n; ++k) b2[k] = double(k) * k / (4.0 * k * k - 1.0);
    x.assign(n, 0.0);
    w.assign(n, 0.0);
    for (int r = 0; r < n; ++r) {
        double lo = -1.0, hi = 1.0;
        for (int it = 0; it < 200; ++it) {
            double mid = 0.5 * (lo + hi);
            if (mid == lo || mid == hi) break;
            if (sturm_count(n, b2, mid) > r) hi = mid; else lo = mid;
        }
        x[r] = 0.5 * (lo + hi);
    }
    // exact mirror symmetry of the node set
    for (int r = 0; r < n / 2; ++r) {
        double m = 0.5 * (x[n - 1 - r] - x[r]);
        x[r] = -m;
        x[n - 1 - r] = m;
    }
    // Christoffel numbers: 1 / sum_{k<n} (k + 1/2) P_k(x)^2 (orthonormal Legendre polynomials)
    for (int r = 0; r < n; ++r) {
        double p_prev = 1.0, p = x[r];
        double s = 0.5 * p_prev * p_prev + 1.5 * p * p;
        for (int k = 1; k + 1 < n; ++k) {
            double p_next = ((2.0 * k + 1.0) * x[r] * p - k * p_prev) / (k + 1.0);
            p_prev = p;
            p = p_next;
            s += (k + 1.5) * p * p;
        }
        w[r] = 1.0 / s;
    }
    return true;
}

int mirror_x(int b, int n_phi)
{
    return (b < n_phi / 2) ? n_phi / 2 - 1 - b : 3 * n_phi / 2 - 1 - b;
}

bool make_angle_set(int n_theta, int n_phi, AngleSet &out)
{
    if (n_theta < 2 || (n_theta % 2) != 0 || n_phi < 4 || (n_phi % 4) != 0) return false;
    std::vector<double> x, w;
    if (!gauss_legendre(n_theta, x, w)) return false;
    out.n_theta = n_theta;
    out.n_phi = n_phi;
    out.n_dir = n_theta * n_phi;
    out.mu.resize(out.n_dir);
    out.ox.resize(out.n_dir);
    out.oy.resize(out.n_dir);
    out.w.resize(out.n_dir);
    const double two_pi = 2.0 * M_PI;
    for (int a = 0; a < n_theta; ++a) {
        const double sin_t = std::sqrt(1.0 - x[a] * x[a]);
        for (int b = 0; b < n_phi; ++b) {
            const int d = a * n_phi + b;
            const double phi = two_pi * (b + 0.5) / n_phi;
            out.mu[d] = x[a];
            out.ox[d] = sin_t * std::cos(phi);
            out.oy[d] = sin_t * std::sin(phi);
            out.w[d] = w[a] / (2.0 * n_phi);
        }
        // exact mirror symmetry x -> -x (phi -> pi - phi): the mirror of b is
        // n_phi/2 - 1 - b for b < n_phi/2 and 3 n_phi/2 - 1 - b otherwise
        for (int b = 0; b < n_phi; ++b) {
            const int bm = mirror_x(b, n_phi);
            if (bm > b) {
                out.ox[a * n_phi + bm] = -out.ox[a * n_phi + b];
                out.oy[a * n_phi + bm] = out.oy[a * n_phi + b];
            }
        }
    }
    return true;
}

namespace {

// Heights in (z_lo, z_hi) where X(z) = x0 + (z - nz) t is an integer, ordered along the travel
// direction (descending z when going down).
void face_crossings(int nz, double x0, double t, double z_in, double z_out, std::vector<double> &z)
{
    z.clear();
    const double lo = std::min(z_in, z_out), hi = std::max(z_in, z_out);
    const double Xa = x0 + (lo - nz) * t, Xb = x0 + (hi - nz) * t;
    const double m_lo = std::floor(std::min(Xa, Xb)) + 1.0;
    for (double m = m_lo; m < std::max(Xa, Xb); m += 1.0) {
        double zc = nz + (m - x0) / t;
        zc = std::min(std::max(zc, lo), hi);
        z.push_back(zc);
    }
    // in the order of m the heights rise or fall with the sign of t (rounding keeps the order)
    if ((t < 0.0) != (z_out < z_in)) std::reverse(z.begin(), z.end());
}

}  // namespace

void layer_segments(int nz, double mu, double ox, double oy, int k, LayerSegments &out)
{
    const double tx = ox / mu, ty = oy / mu;                  // horizontal drift per unit height
    const double z_in = (mu < 0.0) ? k + 1.0 : double(k);
    const double z_out = (mu < 0.0) ? double(k) : k + 1.0;
    std::vector<double> &zx = out.zx, &zy = out.zy, &zb = out.zb;
    face_crossings(nz, 0.5, tx, z_in, z_out, zx);
    face_crossings(nz, 0.5, ty, z_in, z_out, zy);
    // merge the two ordered crossing lists along the travel direction; crossings closer than
    // kCornerTol in height are one crossing through a voxel edge (a line through an edge would
    // otherwise leave a rounding-sized sliver between the x and the y crossing)
    constexpr double kCornerTol = 1e-12;
    const bool down = z_out < z_in;
    zb.clear();
    zb.push_back(z_in);
    size_t p = 0, q = 0;
    while (p < zx.size() || q < zy.size()) {
        bool take_x;
        if (p == zx.size()) take_x = false;
        else if (q == zy.size()) take_x = true;
        else take_x = down ? (zx[p] >= zy[q]) : (zx[p] <= zy[q]);
        const double z = take_x ? zx[p++] : zy[q++];
        if (std::fabs(z - zb.back()) > kCornerTol) zb.push_back(z);
    }
    if (zb.size() > 1 && std::fabs(z_out - zb.back()) <= kCornerTol) zb.back() = z_out;
    else zb.push_back(z_out);
    out.di.clear();
    out.dj.clear();
    out.len.clear();
    const double inv_amu = 1.0 / std::fabs(mu);
    for (size_t s = 0; s + 1 < zb.size(); ++s) {
        const double dz = std::fabs(zb[s + 1] - zb[s]);
        if (!(dz > 0.0)) continue;
        const double zm = 0.5 * (zb[s] + zb[s + 1]);
        out.di.push_back(int(std::floor(0.5 + (zm - nz) * tx)));
        out.dj.push_back(int(std::floor(0.5 + (zm - nz) * ty)));
        out.len.push_back(dz * inv_amu);
    }
}

void direction_segments(int nz, const AngleSet &A, int d, int k, LayerSegments &out)
{
    const int a = d / A.n_phi, b = d % A.n_phi;
    const int bm = mirror_x(b, A.n_phi);
    if (bm >= b) {
        layer_segments(nz, A.mu[d], A.ox[d], A.oy[d], k, out);
        return;
    }
    const int dm = a * A.n_phi + bm;
    layer_segments(nz, A.mu[dm], A.ox[dm], A.oy[dm], k, out);
    for (int &x : out.di) x = -x;
}

static int pos_mod(int a, int n)
{
    int r = a % n;
    return r < 0 ? r + n : r;
}

// dispatch the most expensive work items first
static void sort_work(std::vector<std::pair<double, WorkItem>> &work, SweepPlan &P)
{
    std::stable_sort(work.begin(), work.end(),
                     [](const std::pair<double, WorkItem> &x, const std::pair<double, WorkItem> &y) {
                         return x.first > y.first;
                     });
    P.items.clear();
    P.items.reserve(work.size());
    for (auto &w : work) P.items.push_back(w.second);
}

namespace {

// The pairs' segments in sweep order, with what follows each (the rows that a band touches are the column
// plan's to add)
void append_column_segments(SweepPlan &P)
{
    P.cseg.clear();
    for (PairInfo &pi : P.pairs) {
        pi.c_off = int(P.cseg.size());
        int prev_i = 0, prev_j = 0;
        for (int st = 0; st < P.nz; ++st) {
            const size_t ka = size_t(pi.dA) * P.nz + (pi.down ? P.nz - 1 - st : st);
            const int o = P.seg_off[ka], n = P.seg_n[ka];
            for (int s = o; s < o + n; ++s) {
                if (st > 0 || s > o) {
                    if (P.seg_ai[s] != prev_i) P.cseg.back().flags |= kNextColumn;
                    if (P.seg_bi[s] != prev_j) P.cseg.back().flags |= kNextRow;
                }
                P.cseg.push_back(ColumnSeg{P.seg_len[s], s + 1 == o + n ? kLayerEnd : 0, 0});
                prev_i = P.seg_ai[s];
                prev_j = P.seg_bi[s];
            }
        }
        pi.n_seg = int(P.cseg.size()) - pi.c_off;
    }
}

// Rows, less one, that a line of the pair comes through in layer k
int layer_span(const SweepPlan &P, const PairInfo &pi, int k)
{
    const size_t ka = size_t(pi.dA) * P.nz + k;
    const auto first = P.seg_bi.begin() + P.seg_off[ka];
    const auto mm = std::minmax_element(first, first + P.seg_n[ka]);
    return *mm.second - *mm.first;
}

}  // namespace

void segment_plan(int nx, int ny, int nz, const AngleSet &A, SweepPlan &P)
{
    P = SweepPlan();
    P.nx = nx;
    P.ny = ny;
    P.nz = nz;
    P.n_dir = A.n_dir;
    const size_t n_dk = size_t(A.n_dir) * nz;
    P.seg_off.resize(n_dk);
    P.seg_n.resize(n_dk);
    P.row_min.resize(n_dk);
    P.dirs.resize(A.n_dir);
    // heights of crossings are rounded to a few eps nz
    const double sliver = 64.0 * std::numeric_limits<double>::epsilon() * nz;
    LayerSegments L;
    for (int d = 0; d < A.n_dir; ++d) {
        P.dirs[d].wmu = A.w[d] * std::fabs(A.mu[d]);
        P.dirs[d].down = A.mu[d] < 0.0 ? 1 : 0;
        P.dirs[d].pad = 0;
        P.dirs[d].mu = A.mu[d];
        const int b = d % A.n_phi, bm = mirror_x(b, A.n_phi);
        if (bm < b) {
            // the second of a pair mirrored in x has the first one's table with negated columns (direction_segments)
            const size_t k0 = size_t(d - b + bm) * nz, k1 = size_t(d) * nz, at = P.seg_len.size();
            const size_t s0 = size_t(P.seg_off[k0]), n = size_t(P.seg_off[k0 + nz - 1] + P.seg_n[k0 + nz - 1]) - s0;
            for (int k = 0; k < nz; ++k) {
                P.seg_off[k1 + k] = P.seg_off[k0 + k] + int(at - s0);
                P.seg_n[k1 + k] = P.seg_n[k0 + k];
                P.row_min[k1 + k] = P.row_min[k0 + k];
            }
            P.seg_ai.resize(at + n);
            P.seg_bi.resize(at + n);
            P.seg_len.resize(at + n);
            for (size_t s = 0; s < n; ++s) {
                P.seg_ai[at + s] = -P.seg_ai[s0 + s];
                P.seg_bi[at + s] = P.seg_bi[s0 + s];
                P.seg_len[at + s] = P.seg_len[s0 + s];
            }
            continue;
        }
        for (int k = 0; k < nz; ++k) {
            direction_segments(nz, A, d, k, L);
            const size_t dk = size_t(d) * nz + k;
            P.seg_off[dk] = int(P.seg_len.size());
            P.seg_n[dk] = int(L.di.size());
            P.row_min[dk] = pos_mod(*std::min_element(L.dj.begin(), L.dj.end()), ny);
            P.seg_ai.insert(P.seg_ai.end(), L.di.begin(), L.di.end());
            P.seg_bi.insert(P.seg_bi.end(), L.dj.begin(), L.dj.end());
            P.seg_len.insert(P.seg_len.end(), L.len.begin(), L.len.end());
            for (double l : L.len) P.slivers = P.slivers || l * std::fabs(A.mu[d]) < sliver;
        }
    }
    P.mean_segments = double(P.seg_len.size()) / (double(A.n_dir) * nz);
    for (int a = 0; a < A.n_theta; ++a)
        for (int b = 0; b < A.n_phi; ++b) {
            const int bm = mirror_x(b, A.n_phi);
            if (bm < b) continue;
            PairInfo pi{};
            pi.dA = a * A.n_phi + b;
            pi.dB = a * A.n_phi + bm;
            pi.wmu = P.dirs[pi.dA].wmu;
            pi.down = P.dirs[pi.dA].down;
            pi.mu = A.mu[pi.dA];
            pi.xsgn = A.ox[pi.dA] > 0.0 ? 1 : -1;
            pi.ysgn = A.oy[pi.dA] > 0.0 ? 1 : -1;
            P.pairs.push_back(pi);
        }
    P.n_pair = int(P.pairs.size());
    append_column_segments(P);
}

bool window_row_fits(int lines_per_wg, int nx, std::string &err)
{
    if (nx <= lines_per_wg) return true;
    err = "nx exceeds the lines one sweep workgroup can hold";
    return false;
}

bool window_bands(int lines_per_wg, int target_seg_per_wg, size_t lds_bytes_max, SweepPlan &P, std::string &err)
{
    const int nx = P.nx, ny = P.ny, nz = P.nz;
    if (!window_row_fits(lines_per_wg, nx, err)) return false;
    const int max_rows = lines_per_wg / nx;
    P.lines_per_wg = lines_per_wg;
    P.max_win_rows = 0;
    // the Lambda* kernel takes the pairs as two runs, all of one vertical direction, then the other
    for (int p = 1, changes = 0; p < P.n_pair; ++p)
        if (P.pairs[p].down != P.pairs[p - 1].down && ++changes > 1) {
            err = "direction pairs are not ordered by their vertical direction";
            return false;
        }
    for (PairInfo &pi : P.pairs) {
        int span = 0;
        for (int k = 0; k < nz; ++k) span = std::max(span, layer_span(P, pi, k));
        // Band height: about target_seg_per_wg line-segments per layer for the two directions,
        // never thinner than the window's halo, within the line and LDS budgets.
        const double seg_per_layer = double(pi.n_seg) / nz;
        int rows = int(std::lround(target_seg_per_wg / (2.0 * nx * seg_per_layer)));
        rows = std::max(rows, std::max(1, span));
        rows = std::min(rows, max_rows);
        auto lds = [&](int r) {
            return std::max(sweep_lds_bytes(r + span, r, nx, false), sweep_lds_bytes(r + span, r, nx, true));
        };
        while (rows > 1 && lds(rows) > lds_bytes_max) --rows;
        rows = std::min(rows, ny);
        if (lds(rows) > lds_bytes_max) {
            err = "the deposit window of one band exceeds the LDS budget";
            return false;
        }
        pi.band_rows = rows;
        pi.n_bands = (ny + rows - 1) / rows;
        pi.win_rows = rows + span;
        P.max_win_rows = std::max(P.max_win_rows, pi.win_rows);
    }
    return true;
}

void window_plan(SweepPlan &P)
{
    const int nx = P.nx, ny = P.ny, nz = P.nz;
    int64_t off = 0;
    std::vector<std::pair<double, WorkItem>> work;
    P.blocks.resize(size_t(P.n_pair) * nz);
    for (int p = 0; p < P.n_pair; ++p) {
        PairInfo &pi = P.pairs[p];
        pi.p_off = off;
        pi.band_stride = int64_t(nz) * pi.win_rows * nx;
        off += pi.n_bands * pi.band_stride;
        const size_t pl0 = P.player.size();
        for (int k = 0; k < nz; ++k) {
            const size_t ka = size_t(pi.dA) * nz + k;
            const int o = P.seg_off[ka], n = P.seg_n[ka];
            const int bmin = *std::min_element(P.seg_bi.begin() + o, P.seg_bi.begin() + o + n);
            P.player.push_back(PairLayer{int(P.pseg.size()), n, P.row_min[ka], 0});
            for (int s = o; s < o + n; ++s) {
                PairSeg ps{};
                ps.saA = pos_mod(P.seg_ai[s], nx);
                ps.shB = 0;
                ps.smnx = pos_mod(P.seg_bi[s] - bmin, ny) * nx;
                ps.sbnx = (P.seg_bi[s] - bmin) * nx;
                ps.len = P.seg_len[s];
                ps.len32 = float(P.seg_len[s]);
                P.pseg.push_back(ps);
            }
            P.blocks[size_t(k) * P.n_pair + p] =
                LayerBlock{pi.p_off + int64_t(k) * pi.win_rows * nx, pi.wmu, P.row_min[ka],
                           pi.win_rows - pi.band_rows, nz * pi.win_rows, pi.band_rows << kBlockRows};
        }
        // moves of the B lines: a slot holds the B line whose top column is its A line's plus
        // 2 dA, so when dA changes by delta to the next segment in sweep order (layers top down
        // for downward pairs) the B line moves by -2 delta columns
        PairSeg *before = nullptr;
        int dA = 0;
        for (int st = 0; st < nz; ++st) {
            const int k = pi.down ? nz - 1 - st : st;
            const int o = P.seg_off[size_t(pi.dA) * nz + k];
            for (int s = 0; s < P.player[pl0 + k].ns; ++s) {
                if (before) before->shB = pos_mod(-2 * (P.seg_ai[o + s] - dA), nx);
                before = &P.pseg[P.player[pl0 + k].off + s];
                dA = P.seg_ai[o + s];
            }
        }
        for (int b = 0; b < pi.n_bands; ++b) {
            WorkItem it;
            it.pair = p;
            it.band = b;
            it.j0 = b * pi.band_rows;
            it.rows = std::min(pi.band_rows, ny - it.j0);
            work.push_back({it.rows * double(pi.n_seg) / nz, it});
        }
    }
    P.p_elems = off;
    sort_work(work, P);
}

bool build_sweep_plan(int nx, int ny, int nz, const AngleSet &A, int lines_per_wg, int target_seg_per_wg,
                      size_t lds_bytes_max, SweepPlan &P, std::string &err)
{
    segment_plan(nx, ny, nz, A, P);
    if (!window_bands(lines_per_wg, target_seg_per_wg, lds_bytes_max, P, err)) return false;
    window_plan(P);
    return true;
}

namespace {

// Whether a pair with n_seg segments is split into single line rows.  A sweep lasts at least as long as the
// chain of the longest lines: with R rows a wavefront alone takes about 450 + 165 R cycles per segment
// (measured on 17^3 and 65^3 grids, where nothing else runs beside the shallowest directions), of which the
// rows share the first term, so single rows make the chain short and four make the sum of all work (and
// the partial planes) small.  A pair is split where the chain of four rows would take longer than 1.2 times
// the launch's whole work (about 150 cycles per wavefront and segment) spread over all SIMDs.
bool column_split(double n_seg, double load)
{
    return n_seg * column_segment_cycles(kColumnRows) > 1.2 * load * 150.0 / 1024.0;
}

// Bands of one workgroup: a thread per column, so G bands of nx columns fill G nx of its lanes.  The
// waves of a workgroup go to the four SIMDs of a CU in turn, the first always to the first one, so 5 waves
// load a SIMD as much as 8 do (129 columns: 5, 7 and 9 waves 2.33, 1.98 and 2.41 ms at 129^3 x 256).  G
// maximises the lanes in use over that, less a little per wave, since large workgroups wait longer at
// their barriers.  A grid that leaves the chip short of waves (fill: waves per SIMD with one row per
// thread) takes single waves instead (33^3 x 64: 63 us against 72 with 4 waves).
// Every G on 26 grids with rows of 3 to 400 columns, both precisions: what is taken here is within 5% of the best in 42 of
// the 52 (fill below 3, 17^3 x 64 to 40^3 x 256, us with G = 1, 2, 4, 8: 32 32 34 36, 62 65 68 80, 109 117 118 140, 132 142
// 140 169; between 3 and 12, 65^3 x 64 with 1 to 4: 147 145 136 154, rule 144, 97^3 x 64 with 1 to 5: 276
// 249 288 246 248, rule 250; above, 65^3 x 256 with 1 to 7: 393 336 280 364 343 297 307, rule 287, 97^3 x 256 with 1 to 5: 852 840
// 1028 888 752, rule 761); the worst are 97 x 41 x 58 x 128 (151 against 133) and 161 x 100 x 60 x 256 in float32 (510 against 435, where
// single bands do better than the float64 pattern that the table follows).
int column_bands(int nx, int n_bands, double fill, int max_waves)
{
    const int most = std::max(1, std::min({1024 / nx, n_bands, 64 * max_waves / nx}));
    if (fill < 3.0) return std::min(most, std::max(1, 64 / nx));
    static const double load[8] = {1.3, 2.5, 3.3, 4.0, 8.0, 8.0, 7.5, 8.0};
    const double per_wave = fill < 12.0 ? 0.04 : 0.02;
    int best = 1;
    double best_score = -1e9;
    for (int G = 1; G <= most; ++G) {
        const int w = (G * nx + 63) / 64;
        const double l = load[(w - 1) % 8] + 8.0 * ((w - 1) / 8);
        const double score = G * nx / (64.0 * l) - per_wave * w;
        if (score > best_score) {
            best = G;
            best_score = score;
        }
    }
    return best;
}

}  // namespace

double column_load(int nx, int ny, int nz, const AngleSet &A)
{
    // 1 + tan(theta) (|cos phi| + |sin phi|) segments per layer on average
    double seg = 0.0;
    for (int d = 0; d < A.n_dir; ++d) seg += 1.0 + (std::fabs(A.ox[d]) + std::fabs(A.oy[d])) / std::fabs(A.mu[d]);
    return 0.5 * seg * nz * (double(nx) * ny / 64.0);
}

bool make_column_plan(const AngleSet &A, int threads, int lines, double load, SweepPlan &P)
{
    const int nx = P.nx, ny = P.ny, nz = P.nz;
    if (nx > kColumnMaxNx) return false;
    std::vector<PairInfo> pairs = P.pairs;
    std::vector<LayerBlock> blocks(size_t(P.n_pair) * nz);
    std::vector<std::pair<double, WorkItem>> work;
    int max_cover = 0, block_threads = 64, col_rows = 1;
    // waves per SIMD of the launch, if its other members are like this one
    const double fill = double(nx) * ny / 64.0 * P.n_pair / 1024.0 * load / column_load(nx, ny, nz, A);
    int64_t off = 0;
    for (int p = 0; p < P.n_pair; ++p) {
        PairInfo &pi = pairs[p];
        pi.split = lines <= 2 && column_split(pi.n_seg, load) ? 1 : 0;
        const int rows = pi.split ? 1 : kColumnRows;
        const int n_parts = (ny + rows - 1) / rows;       // bands, or line rows
        const int G = column_bands(nx, n_parts, fill, std::max(1, threads / 64));
        block_threads = std::max(block_threads, (G * nx + 63) / 64 * 64);
        col_rows = std::max(col_rows, rows);
        pi.band_rows = kColumnRows;
        pi.n_bands = (ny + kColumnRows - 1) / kColumnRows;
        pi.win_rows = 0;
        pi.row0 = pos_mod(P.seg_bi[P.seg_off[size_t(pi.dA) * nz + (pi.down ? nz - 1 : 0)]], ny);
        const size_t ka_end = size_t(pi.dA) * nz + (pi.down ? 0 : nz - 1);
        pi.sa_last = pos_mod(P.seg_ai[P.seg_off[ka_end] + P.seg_n[ka_end] - 1], nx);
        int64_t block = 0;
        size_t end = size_t(pi.c_off);         // end of the layer in the segment list
        for (int st = 0; st < nz; ++st) {
            const int k = pi.down ? nz - 1 - st : st;
            const size_t ka = size_t(pi.dA) * nz + k;
            const int span = layer_span(P, pi, k), cover = rows + span;
            if (st == 0) pi.cover0 = cover;
            else P.cseg[end - 1].cover = cover;
            end += size_t(P.seg_n[ka]);
            pi.win_rows = std::max(pi.win_rows, cover);
            blocks[size_t(k) * P.n_pair + p] =
                LayerBlock{off + block, pi.wmu, P.row_min[ka], span, 0,
                           (kColumnRows << kBlockRows) | (pi.split ? kBlockSplit : 0) | (pi.ysgn < 0 ? kBlockDown : 0)};
            block += int64_t(cover) * nx;
        }
        pi.band_stride = block;
        for (int k = 0; k < nz; ++k) blocks[size_t(k) * P.n_pair + p].stride = int(block / nx);
        pi.p_off = off;
        off += n_parts * block;
        // the kernel addresses a workgroup's bands with 32-bit byte offsets
        if (G * block * int64_t(sizeof(double)) >= (int64_t(1) << 32) - 16) return false;
        max_cover = std::max(max_cover, pi.win_rows);
        for (int b = 0; b < n_parts; b += G) {
            WorkItem it;
            it.pair = p;
            it.band = b;
            it.j0 = b * rows;
            it.rows = std::min(G, n_parts - b);
            work.push_back({pi.n_seg * column_segment_cycles(rows), it});
        }
    }
    P.columns = true;
    P.pairs = std::move(pairs);
    P.blocks = std::move(blocks);
    P.max_win_rows = max_cover;
    P.block_threads = block_threads;
    P.col_rows = col_rows;
    P.p_elems = off;
    sort_work(work, P);
    return true;
}

namespace {

// Elements of pair q's partial planes of the layer at a step (column form)
int64_t layer_elems(const SweepPlan &P, int q, int step)
{
    const PairInfo &pi = P.pairs[q];
    const int rows = pi.split ? 1 : kColumnRows, k = pi.down ? P.nz - 1 - step : step;
    return int64_t(rows + P.blocks[size_t(k) * P.n_pair + q].span) * P.nx * ((P.ny + rows - 1) / rows);
}

}  // namespace

SweepKind::SweepKind(const SweepPlan &plan) : columns(plan.columns), block_threads(plan.block_threads)
{
    for (const PairInfo &pi : plan.pairs) split.push_back(pi.split);
    for (const WorkItem &it : plan.items) items.insert(items.end(), {it.pair, it.band, it.rows});
}

std::vector<LayerStart> layer_starts(const SweepPlan &P)
{
    std::vector<LayerStart> start(P.blocks.size());
    for (int q = 0; q < P.n_pair; ++q) {
        int s = P.pairs[q].c_off;
        for (int step = 0; step < P.nz; ++step) {
            const int k = P.pairs[q].down ? P.nz - 1 - step : step;
            const size_t ka = size_t(P.pairs[q].dA) * P.nz + k;
            start[size_t(k) * P.n_pair + q] = LayerStart{s, pos_mod(P.seg_bi[P.seg_off[ka]], P.ny)};
            s += P.seg_n[ka];
        }
    }
    return start;
}

int64_t lay_out(SweepPlan &P, const SweepPart &part)
{
    int64_t off = 0;
    if (!P.columns) {
        for (int q = part.q0; q < part.q1; ++q) {
            PairInfo &pi = P.pairs[q];
            for (int k = 0; k < P.nz; ++k) P.blocks[size_t(k) * P.n_pair + q].off += off - pi.p_off;
            pi.p_off = off;
            off += pi.n_bands * pi.band_stride;
        }
        return off;
    }
    for (int q = part.q0; q < part.q1; ++q) {
        PairInfo &pi = P.pairs[q];
        const int rows = pi.split ? 1 : kColumnRows, n = (P.ny + rows - 1) / rows;
        int64_t block = 0;
        for (int pass = 0; pass < 2; ++pass) {
            // first the rows of a band (line row) in all layers, then every layer's place
            int64_t at = 0;
            for (int step = part.step0; step < part.step0 + part.layers; ++step) {
                LayerBlock &lb = P.blocks[size_t(pi.down ? P.nz - 1 - step : step) * P.n_pair + q];
                if (pass == 1) {
                    lb.off = off + at;
                    lb.stride = int(block / P.nx);
                }
                at += int64_t(rows + lb.span) * P.nx;
            }
            block = at;
        }
        if (part.layers == P.nz) {
            pi.p_off = off;
            pi.band_stride = block;
        }
        off += n * block;
    }
    return off;
}

std::vector<SweepPart> layer_parts(const SweepPlan &P, int64_t room)
{
    std::vector<SweepPart> parts;
    for (int run0 = 0; run0 < P.n_pair;) {
        int run1 = run0;
        while (run1 < P.n_pair && P.pairs[run1].down == P.pairs[run0].down) ++run1;
        for (int group = run1 - run0;; group = (group + 1) / 2) {
            const size_t before = parts.size();
            const int64_t free = room - int64_t(group) * 2 * P.nx * P.ny;
            bool fits = true;
            for (int q0 = run0; q0 < run1 && fits; q0 += group) {
                const int q1 = std::min(q0 + group, run1);
                std::vector<int64_t> elems(P.nz, 0);
                int64_t sum = 0;
                for (int step = 0; step < P.nz; ++step) {
                    for (int q = q0; q < q1; ++q) elems[step] += layer_elems(P, q, step);
                    sum += elems[step];
                }
                if (sum <= room) {
                    parts.push_back(SweepPart{q0, q1, 0, P.nz, P.pairs[q0].down != 0});
                    continue;
                }
                for (int step = 0; step < P.nz && fits;) {
                    int n = 0;
                    int64_t used = 0;
                    while (step + n < P.nz && used + elems[step + n] <= free) used += elems[step + n++];
                    fits = n >= (group > 1 ? std::min(2, P.nz - step) : 1);
                    parts.push_back(SweepPart{q0, q1, step, n, P.pairs[q0].down != 0});
                    step += n;
                }
            }
            if (fits) break;
            parts.resize(before);
            if (group == 1) return {};
        }
        run0 = run1;
    }
    return parts;
}

std::vector<SweepPart> pair_parts(const SweepPlan &P, int64_t room)
{
    std::vector<SweepPart> parts;
    for (int q = 0; q < P.n_pair;) {
        int q1 = q;
        for (int64_t used = 0; q1 < P.n_pair; ++q1) {
            used += P.pairs[q1].n_bands * P.pairs[q1].band_stride;
            if (used > room) break;
        }
        if (q1 == q) return {};
        parts.push_back(SweepPart{q, q1, 0, P.nz});
        q = q1;
    }
    return parts;
}

JacobiTile choose_jacobi_tile(int nx, int ny, int nz)
{
    // A launch takes about 2 us, 3 more for each round of workgroups (24 wavefronts of a CU at once), and for each
    // wavefront of the fullest CU 0.1 us, as much for every previous iterate per thread and 0.8 / tx for the loads of
    // rows that end within it (fitted to 17^3 .. 72^3, for instance 65^3 with tiles of 13 x 5 x 5 / 17 x 4 x 4 / 6 x 6 x 6 /
    // 5 x 5 x 11: 19.6 / 21.6 / 21.3 / 27.3 us for two sweeps).
    JacobiTile best{};
    double best_us = 1e300;
    // the next tile size that divides an axis of n into fewer nearly equal parts
    auto next = [](int n, int t) {
        const int parts = (n + t - 1) / t;
        return parts == 1 ? n + 1 : (n + parts - 2) / (parts - 1);
    };
    for (int tx = 1; tx <= nx && (tx + 2) * 9 <= kPairThreads; tx = next(nx, tx))
        for (int ty = 1; ty <= ny && (tx + 2) * (ty + 2) * 3 <= kPairThreads; ty = next(ny, ty))
            for (int z = 1; z <= nz && (tx + 2) * (ty + 2) * (z + 2) <= kPairThreads; z = next(nz, z)) {
                JacobiTile t;
                t.tx = tx;
                t.ty = ty;
                t.z = z;
                t.ntx = (nx + tx - 1) / tx;
                t.nty = (ny + ty - 1) / ty;
                t.ntz = (nz + z - 1) / z;
                if (t.cells0() > kPairLoads * t.threads()) continue;
                const int w = t.threads() / 64, at_once = 256 * (24 / w);
                // (a workgroup that has a CU to itself waits at its barriers with nothing else to run)
                const int b = t.blocks();
                const double waves = (b <= 512 ? (b + 255) / 256 : b / 256.0) * w * (24 / w == 1 ? 1.25 : 1.0);
                const double us = 2.0 + (0.1 + 0.8 / tx + 0.1 * t.cells0() / t.cells()) * waves +
                                  3.0 * ((t.blocks() + at_once - 1) / at_once);
                if (us < best_us) {
                    best_us = us;
                    best = t;
                }
            }
    return best;
}

}  // namespace rt3d
