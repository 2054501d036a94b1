// Host-side geometry of the HIP library: angle set, per-direction segment tables and the work plan
// of the line sweep.  Internal to the library (not part of the C ABI).
#pragma once

#include <cstdint>
#include <string>
#include <vector>

namespace rt3d {

struct AngleSet {
    int n_theta = 0, n_phi = 0, n_dir = 0;
    std::vector<double> mu, ox, oy, w;   // per direction d = a * n_phi + b
};

// Gauss-Legendre nodes (ascending) by Sturm-sequence bisection on the Jacobi matrix of the Legendre
// polynomials, weights by the Christoffel sum 1 / sum_k (k + 1/2) P_k(x)^2.
bool gauss_legendre(int n, std::vector<double> &x, std::vector<double> &w);
bool make_angle_set(int n_theta, int n_phi, AngleSet &out);

// Segments of the reference line (through (1/2, 1/2, nz)) of one direction inside layer k, in travel
// order: column offsets (di, dj) relative to the line's top column and path lengths.
struct LayerSegments {
    std::vector<int> di, dj;
    std::vector<double> len;
    std::vector<double> zx, zy, zb;      // working space: crossings of the x and y faces, and all of them
};
void layer_segments(int nz, double mu, double ox, double oy, int k, LayerSegments &out);

// Index of the azimuth mirrored in x (phi -> pi - phi).
int mirror_x(int b, int n_phi);

// The segments of direction d of an angle set inside layer k.  Of an x-mirrored pair of azimuths
// the lower index is cut by layer_segments and the other is its exact mirror (columns negated):
// lines that pass through voxel edges (every line when n_phi = 4) leave rounding-sized slivers whose
// voxel would otherwise depend on the rounding of each direction separately.
void direction_segments(int nz, const AngleSet &A, int d, int k, LayerSegments &out);

// Per-direction metadata (plain old data, copied to the device).
struct DirInfo {
    double wmu;        // W_d * |mu_d|
    int down;          // 1 if mu < 0 (sweep from the top layer down)
    int pad;
    double mu;         // direction cosine with the z axis
};

// A pair of directions mirrored in x, (mu, phi) and (mu, pi - phi).  Their lines cross the same
// faces at the same heights: the segment lengths and row offsets are identical and the column
// offsets are negated, so one workgroup sweeps both through the same band and one partial plane
// holds both.  W |mu| is the same for both.
struct PairInfo {
    double wmu;        // W |mu| of either direction
    int dA, dB;        // the two directions; dA owns the shared tables
    int down;          // 1 if mu < 0
    int band_rows;     // Bj: line rows per band (last band may be shorter)
    int n_bands;       // nb
    int win_rows;      // Hw = Bj + span: rows of the deposit window of one band
    int64_t p_off;     // element offset of this pair's partial planes in P
    double mu;         // direction cosine with the z axis (the same for both)
    int64_t band_stride;   // elements of P per band
    // column form: bands of kColumnRows line rows, either each held by one thread per column, or (split) each
    // line row by a thread of its own with partial planes of its own (band_stride is then a line row's)
    int split;
    int c_off, n_seg;  // the pair's segments in the list: first entry, count
    int xsgn, ysgn;    // signs of direction A's column moves and of both directions' row moves
    int row0;          // row offset of the first segment modulo ny
    int cover0;        // rows that a band (split: a line row) touches in the first layer
    int sa_last;       // direction A's column offset at the last segment modulo nx
};

// A segment as the column form of the sweep reads it, in sweep order: its length, what follows it, and,
// where its layer ends, the rows that a band (split: a line row) touches in the next layer.
enum { kNextColumn = 1, kNextRow = 2, kLayerEnd = 4 };   // the lines change columns / rows, the layer ends
struct ColumnSeg {
    double len;
    int flags, cover;
};

// Where the reduction finds a pair's partial planes of one layer, as one 32-byte scalar load: the block of band
// (split: line row) n starts n * stride rows of nx elements after element off of P, and holds the rows from
// the band's first plus rmin (modulo ny) on, span more than the band has.
enum { kBlockSplit = 1, kBlockDown = 2, kBlockRows = 2 };     // flags; the rows of a full band << kBlockRows
struct alignas(32) LayerBlock {
    int64_t off;
    double wmu;
    int rmin, span, stride, flags;
};

// Segment s of a pair in one layer, packed for one scalar load: the column offset of direction A
// (modulo nx; B's is its negative), the move of the B lines between the slots of their row after
// this segment (-2 times the change of A's column offset to the next segment in sweep order, modulo
// nx; 0: none), the row offset modulo ny times nx (global row step), the row offset within the band
// window times nx (LDS row step), and the length in both precisions.
struct PairSeg {
    int saA, shB, smnx, sbnx;
    double len;
    float len32;
    int pad;
};

// Per (pair, layer): first entry in the packed segment list, segment count, window origin row.
struct PairLayer {
    int off, ns, rmin, pad;
};

// One workgroup of the sweep: direction pair p, band of line rows [j0, j0 + rows); in the column form the
// rows bands from band on, the first starting at line row j0.
struct WorkItem {
    int pair, band, j0, rows;
};

struct SweepPlan {
    int nx = 0, ny = 0, nz = 0, n_dir = 0, n_pair = 0;
    int lines_per_wg = 0;                 // lines of one direction in one workgroup
    // segment tables, flat; index of (d, k) is d * nz + k
    std::vector<int> seg_off, seg_n;      // per (d, k)
    std::vector<int> seg_ai, seg_bi;      // column / row offsets from the line's top column
    std::vector<double> seg_len;
    std::vector<int> row_min;             // per (d, k): minimum row offset modulo ny
    std::vector<DirInfo> dirs;
    std::vector<PairInfo> pairs;
    std::vector<PairSeg> pseg;            // packed per-pair segments
    std::vector<PairLayer> player;        // per (pair, layer): index pair * nz + k
    std::vector<LayerBlock> blocks;       // per (layer, pair): index k * n_pair + pair
    // column form (it has no pseg and player)
    bool columns = false;
    int col_rows = 0;                     // most rows per thread of any pair
    int block_threads = 0;                // threads of a workgroup
    std::vector<ColumnSeg> cseg;
    // a segment so short that rounding made it (a line through voxel edges: n_phi = 4, 12, 20, ... and about 1000
    // layers or more).  Opposite directions need not share it, and it may lie in the voxel of its neighbour.
    bool slivers = false;
    std::vector<WorkItem> items;          // in dispatch order (most expensive first)
    int64_t p_elems = 0;                  // size of the partial-plane buffer P in elements
    int max_win_rows = 0;
    double mean_segments = 0.0;           // per voxel and angle
};

// LDS of one sweep workgroup for a band of band_rows line rows and a deposit window of win_rows rows:
// the window and two exchange buffers of one value per line, in the sweep's precision.
inline size_t sweep_lds_bytes(int win_rows, int band_rows, int nx, bool f32)
{
    const size_t cells = size_t(win_rows) * size_t(nx), lines = size_t(band_rows) * size_t(nx);
    return (cells + 2 * lines) * (f32 ? sizeof(float) : sizeof(double));
}

// A plan is made in three steps: the segment tables and direction pairs (which every form of the sweep, Lambda* and the
// adjoint read), the window form's bands, which decide what grids are accepted, and then the tables of one of the two forms.
void segment_plan(int nx, int ny, int nz, const AngleSet &A, SweepPlan &plan);
// lines_per_wg bounds the lines of one direction in one band; lds_bytes_max bounds a band's LDS in either
// precision (sweep_lds_bytes).  May be called again with other limits.
bool window_row_fits(int lines_per_wg, int nx, std::string &err);
bool window_bands(int lines_per_wg, int target_seg_per_wg, size_t lds_bytes_max, SweepPlan &plan, std::string &err);
void window_plan(SweepPlan &plan);
// All three for the window form
bool build_sweep_plan(int nx, int ny, int nz, const AngleSet &A, int lines_per_wg, int target_seg_per_wg,
                      size_t lds_bytes_max, SweepPlan &plan, std::string &err);

// The column form's tables: a thread per column of a band (or, where the pair is split, of a line
// row), workgroups of at most about threads threads that hold several bands (line rows) of a pair; a work
// item's band and rows count those.  load: what the launch that sweeps this plan has to do (this plan's own,
// or the sum over the members of a batch), see column_load.  lines > 2: no pair is split.  The sums of a
// voxel's deposits have the same order whether a pair is split or not.  Rows of more than kColumnMaxNx
// columns keep the window form (false is returned and the plan's bands left as they are): there one row fills
// a workgroup by itself.
constexpr int kColumnMaxNx = 512;
constexpr int kColumnRows = 4;
bool make_column_plan(const AngleSet &A, int threads, int lines, double load, SweepPlan &plan);
// Wavefronts times segments of a grid's sweep, one line row per thread
double column_load(int nx, int ny, int nz, const AngleSet &A);
// Cycles per segment of a wavefront of the column form that has its SIMD to itself, with rows line rows
inline double column_segment_cycles(int rows) { return 450.0 + 165.0 * rows; }

// What the launches of a column plan depend on; two shapes whose plans agree in it run the same kernels.
struct SweepKind {
    bool columns = false;
    int block_threads = 0;
    std::vector<int> split, items;
    explicit SweepKind(const SweepPlan &plan);
    bool operator==(const SweepKind &o) const
    {
        return columns && o.columns && block_threads == o.block_threads && split == o.split && items == o.items;
    }
};

// A part of a sweep whose partial planes do not all fit a buffer: layers [step0, step0 + layers), counted in sweep order, of
// direction pairs [q0, q1); its work items in a list.
struct SweepPart {
    int q0, q1, step0, layers;
    bool down = false;
    int item0 = 0, n_items = 0;
};
// Parts of layers (column form) of as many pairs of one vertical direction as leave room for two layers (one, where it is a
// single pair); empty where that does not fit.  room: elements for the partial planes and the lines' intensities.
std::vector<SweepPart> layer_parts(const SweepPlan &plan, int64_t room);
// Parts of pairs, all their layers (window form)
std::vector<SweepPart> pair_parts(const SweepPlan &plan, int64_t room);
// Gives the partial planes of a part's pairs and layers their places from the start of the buffer on; their elements.
int64_t lay_out(SweepPlan &plan, const SweepPart &part);
// Elements that the intensities of its lines take between parts
inline int64_t line_elems(const SweepPlan &plan, const SweepPart &part)
{
    return part.layers < plan.nz ? int64_t(part.q1 - part.q0) * 2 * plan.nx * plan.ny : 0;
}
// Per (layer, pair) as SweepPlan::blocks: the layer's first segment in cseg and its row offset modulo ny
struct LayerStart { int seg, row; };
std::vector<LayerStart> layer_starts(const SweepPlan &plan);

// The tile of a launch that does two Jacobi sweeps: a workgroup puts out tx x ty x z voxels.
struct JacobiTile {
    int tx, ty, z;
    int ntx, nty, ntz;
    // its first sweep has a voxel more to each side, the previous iterates two
    constexpr int cells() const { return (tx + 2) * (ty + 2) * (z + 2); }
    constexpr int cells0() const { return (tx + 4) * (ty + 4) * (z + 4); }
    constexpr int threads() const { return (cells() + 63) / 64 * 64; }
    constexpr int blocks() const { return ntx * nty * ntz; }
    constexpr size_t lds() const { return size_t(cells0() + cells()) * sizeof(double); }
};
constexpr int kPairThreads = 1024;      // most threads of its workgroup
constexpr int kPairLoads = 3;           // most previous iterates that a thread brings
JacobiTile choose_jacobi_tile(int nx, int ny, int nz);

}  // namespace rt3d
