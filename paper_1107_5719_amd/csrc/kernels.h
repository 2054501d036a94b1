// kernels.h -- HIP device code of the 3D radiative-transfer hot path (gfx950).  Included by the
// single-problem ABI (rt3d.hip) and the batched ABI (batch.hip).  The kernels that batching applies
// to are device functions taking an argument struct, with a single-problem wrapper here and a
// batched wrapper in batch.hip, so both run the same arithmetic.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <type_traits>

#include "geometry.h"

using rt3d::DirInfo;
using rt3d::WorkItem;

namespace {

// Sweep workgroup shapes (threads, lines per thread and direction); the context picks one.  The column form
// takes from a shape only the threads that a workgroup may have and, with more than 2 lines, never splits
// a pair into single rows.
struct SweepShape { int threads, lines; };
// Measured on MI355X at 129^3 x 256 in the window form: 512 x 2 is fastest (64 VGPRs, 8 waves/SIMD; the sweep is
// latency-bound, so occupancy beats lines per thread and prefetching).
constexpr SweepShape kSweepShapes[] = {{512, 2}, {512, 4}, {256, 8}, {1024, 2}, {256, 4}, {256, 2}};
// Calls f(NT, LPT) (as integral constants) for the sweep shape with the given index.
template <int NT, int LPT> struct ShapeTag {
    static constexpr int threads = NT, lines = LPT;
};
template <typename F>
inline void with_sweep_shape(int shape, F &&f)
{
    switch (shape) {
    case 1: f(ShapeTag<512, 4>{}); break;
    case 2: f(ShapeTag<256, 8>{}); break;
    case 3: f(ShapeTag<1024, 2>{}); break;
    case 4: f(ShapeTag<256, 4>{}); break;
    case 5: f(ShapeTag<256, 2>{}); break;
    default: f(ShapeTag<512, 2>{}); break;
    }
}
constexpr size_t kWindowBytes = 48 * 1024;   // LDS budget of a band (deposit window and exchange)
// Grids whose windows do not fit kWindowBytes (wide rows, shallow angle sets) take up to this much of
// the 160 KB of LDS a gfx950 workgroup may use (the rest holds the kernel's static LDS): one workgroup
// per CU then, but no width limit below the line budget of a workgroup.
constexpr size_t kWindowBytesWide = 156 * 1024;
// LDS elements that one thread of a column sweep passes its lines through at an x-face: two buffers of both
// lines of every row, padded so that the lanes' 16-byte accesses meet no bank twice.
template <typename real> __host__ __device__ constexpr int column_edge(int rows) { return 4 * rows + 16 / int(sizeof(real)); }
// Dynamic LDS of a sweep workgroup.  Column form: column_edge of every thread.  Window form: the largest window
// and exchange buffers of any direction pair's bands (each band lays out its own within this).
inline size_t sweep_smem_bytes(const rt3d::SweepPlan &plan, bool f32)
{
    if (plan.columns)
        return size_t(plan.block_threads) *
               (f32 ? column_edge<float>(plan.col_rows) * sizeof(float) : column_edge<double>(plan.col_rows) * sizeof(double));
    size_t bytes = 0;
    for (const rt3d::PairInfo &pi : plan.pairs)
        bytes = std::max(bytes, rt3d::sweep_lds_bytes(pi.win_rows, pi.band_rows, plan.nx, f32));
    return bytes;
}
constexpr int kPlaneThreads = 256;   // voxel-parallel kernels: one thread per voxel of a k-plane

template <typename real> struct Vec2;
template <> struct Vec2<double> { using type = double2; };
template <> struct Vec2<float> { using type = float2; };

// e^x - 1 for x <= 0 (the argument is always -dtau).  No range branches: x is clamped where e^x
// vanishes.
//
// float64, Tang's table method with N = 16: x = (16 k + j) ln2/16 + r with 0 <= j < 16 and
// |r| <= ln2/32, so e^x - 1 = 2^k T_j (1 + r p(r)) - 1 with T_j = 2^(j/16) read from a table and p the
// Taylor polynomial of (e^r - 1)/r through r^6 (truncation below 1e-16 relative).  The multiple
// n = 16 k + j is the nearest integer to x 16/ln2, taken from the rounding of x 16/ln2 + 1.5 * 2^52
// (the spacing of doubles there is 1, so the low word of the sum is n in two's complement).
// 2^k T_j - 1 is exact when 2^k T_j >= 1/2 and is far from zero otherwise; the rounding of T_j bounds
// the relative error by a few 1e-15 where the result is small (|x| a few times ln2/32), and below
// ln2/32 the result is r p(r) itself.  The sweep reduces with one fma on the rounded ln2/16: its error
// in r, |n| times half an ulp of ln2/16, moves e^x by at most 1e-16 |x| e^x relative (below 3e-17
// absolute).  exp_pair_tab splits ln2/16 into a high part whose product with n is exact and a low
// part, so that e^x itself stays accurate to a few ulps for thick segments.  The table (128 bytes,
// in LDS) is small enough that the lanes' lookups never meet in an LDS bank: a 128-entry table with
// the polynomial through r^4 took 2-3% longer per sweep (host emulation against long-double expm1 over
// 3e7 samples of x in [-2000, -1e-14]: at most 2.7e-15 relative here, 3.9e-15 with 128 entries).
constexpr int kExpTabLog2 = 4;
constexpr int kExpTab = 1 << kExpTabLog2;
constexpr double kExpInvStep = 184.66496523378731 / 8;            // 16 / ln2 (128 / ln2, exactly scaled)
constexpr double kExpStep = 0.0054152123481245725 * 8;             // ln2 / 16
constexpr double kExpStepHi = 6.93147180369123816490e-01 / 16;    // 21 trailing zero bits
constexpr double kExpStepLo = 1.90821492927058770002e-10 / 16;
constexpr double kExpRound = 6755399441055744.0;                   // 1.5 * 2^52

// The table as exp_scale reads it: T_j = 2^(j/kExpTab) rounded to float64 from the 64-bit-mantissa long double
// exp2, less j << (20 - kExpTabLog2) in the high word; after these, what the rounding took, over T_j (exp_pair_ulp).
constexpr int kExpTabSize = 2 * kExpTab;
inline void exp_table(double *tab)
{
    for (int j = 0; j < kExpTab; ++j) {
        const long double exact = std::exp2(static_cast<long double>(j) / kExpTab);
        const double t = double(exact);
        tab[kExpTab + j] = double((exact - t) / t);
        uint64_t bits;
        std::memcpy(&bits, &t, sizeof bits);
        bits -= uint64_t(j) << (52 - kExpTabLog2);
        std::memcpy(&tab[j], &bits, sizeof bits);
    }
}

// a * b + c as one VOP3 v_fma_f64 with c in an SGPR pair.  For a constant addend the compiler would
// otherwise keep c in VGPRs and copy it into the destination of a two-address v_fmac_f64 at every
// use (a v_mov_b64 per polynomial step of every exponential in the sweep's segment loop).
__device__ inline double fma3(double a, double b, double c)
{
    double d;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
    return d;
}

// (e^r - 1 - r) / r^2
__device__ inline double expm1_poly_rest(double r)
{
    double p = fma3(r, 1.0 / 5040.0, 1.0 / 720.0);
    p = fma3(p, r, 1.0 / 120.0);
    p = fma3(p, r, 1.0 / 24.0);
    p = fma3(p, r, 1.0 / 6.0);
    return fma(p, r, 0.5);
}
__device__ inline double expm1_poly(double r) { return fma(expm1_poly_rest(r), r, 1.0) * r; }

// 2^k T_j for n = 16 k + j (k >= -1022): the table holds T_j with j << 16 taken off its high word, so
// that one shift-and-add of n puts k into the exponent field.
__device__ inline double exp_scale(int n, const double *tab)
{
    const double t = tab[n & (kExpTab - 1)];
    return __hiloint2double(__double2hiint(t) + int(unsigned(n) << (20 - kExpTabLog2)), __double2loint(t));
}

__device__ inline double expm1_nonpos_tab(double x, const double *tab)
{
    x = fmax(x, -708.0);
    const double kr = fma(x, kExpInvStep, kExpRound);
    const double kf = kr - kExpRound;
    const int n = __double2loint(kr);
    const double q = expm1_poly(fma(-kf, kExpStep, x));
    const double s = exp_scale(n, tab);
    return fma(s, q, s - 1.0);
}

// Both e^x and e^x - 1 for x <= 0 from one table evaluation: with s = 2^k T_j and q = r p(r),
// e^x = s (1 + q) and e^x - 1 = s q + (s - 1), each to a few ulps relative (the first also for
// thick segments, where 1 + (e^x - 1) would lose all of it).
__device__ inline void exp_pair_tab(double x, const double *tab, double &e, double &em1)
{
    x = fmax(x, -708.0);
    const double kr = fma(x, kExpInvStep, kExpRound);
    const double kf = kr - kExpRound;
    const int n = __double2loint(kr);
    const double q = expm1_poly(fma(-kf, kExpStepLo, fma(-kf, kExpStepHi, x)));
    const double s = exp_scale(n, tab);
    e = fma(s, q, s);
    em1 = fma(s, q, s - 1.0);
}

// exp_pair_tab with the rounding of T_j taken back in q: tab[kExpTab + j] is the rest of 2^(j/16) over T_j, so e^x and
// e^x - 1 are good to one ulp (2.2e-16 and 1.2e-16 against long double over 3e7 samples of x in [-1000, -1e-14]), as the
// library's expm1 and exp are.
__device__ inline void exp_pair_ulp(double x, const double *tab, double &e, double &em1)
{
    x = fmax(x, -708.0);
    const double kr = fma(x, kExpInvStep, kExpRound);
    const double kf = kr - kExpRound;
    const int n = __double2loint(kr);
    const double r = fma(-kf, kExpStepLo, fma(-kf, kExpStepHi, x));
    const double q = r + fma(expm1_poly_rest(r) * r, r, tab[kExpTab + (n & (kExpTab - 1))]);
    const double s = exp_scale(n, tab);
    e = fma(s, q, s);
    em1 = fma(s, q, s - 1.0);
}
__device__ inline double expm1_ulp(double x, const double *tab)
{
    double e, em1;
    exp_pair_ulp(x, tab, e, em1);
    return em1;
}

// float32: x = k ln2 + r with |r| <= ln2/2; e^x - 1 = 2^k (e^r - 1) + (2^k - 1), and e^r - 1 is its
// Taylor series through r^8 (truncation below 1e-9 relative).
__device__ inline float expm1_nonpos(float x)
{
    x = fmaxf(x, -87.0f);
    const float kf = rintf(x * 1.44269504089f);
    float r = fmaf(-kf, 0.693145751953125f, x);
    r = fmaf(-kf, 1.42860682e-06f, r);
    float p = 1.0f / 40320.0f;
    p = fmaf(p, r, 1.0f / 5040.0f);
    p = fmaf(p, r, 1.0f / 720.0f);
    p = fmaf(p, r, 1.0f / 120.0f);
    p = fmaf(p, r, 1.0f / 24.0f);
    p = fmaf(p, r, 1.0f / 6.0f);
    p = fmaf(p, r, 0.5f);
    p = fmaf(p, r, 1.0f);
    const float two_k = ldexpf(1.0f, int(kf));
    return fmaf(two_k, p * r, two_k - 1.0f);
}

// ------------------------------------------------------------------------------------------------
// S update
// ------------------------------------------------------------------------------------------------

// S_given: the source itself.  Ja (difference mode of the FP32 form): the source change since the
// anchor iterate, (1 - eps)(J - Ja), whose formal solution is added to the anchor's.  scatter_only:
// the scattering part (1 - eps) J alone (the adjoint solve, whose thermal term enters as a base).
struct SourceArgs {
    int nx, ny, nz;
    int scatter_only;
    const double *chi, *eps, *B, *J, *S_given, *Ja;
    void *cs;                     // Vec2<real>
    unsigned long long *clear;    // the step's three scalars, set to 0 (may be null); spares a memset launch
};

template <typename real>
__device__ inline void source_body(const SourceArgs &a, int p, int k)
{
    if (p >= a.nx * a.ny) return;
    if (a.clear && k == 0 && p < 3) a.clear[p] = 0;
    const long v = long(k) * a.nx * a.ny + p;
    double S;
    if (a.S_given) S = a.S_given[v];
    else if (a.Ja) S = (1.0 - a.eps[v]) * (a.J[v] - a.Ja[v]);
    else if (a.scatter_only) S = (1.0 - a.eps[v]) * a.J[v];
    else S = a.eps[v] * a.B[v] + (1.0 - a.eps[v]) * a.J[v];
    typename Vec2<real>::type c;
    c.x = real(a.chi[v]);
    c.y = real(S);
    static_cast<typename Vec2<real>::type *>(a.cs)[v] = c;
}

template <typename real>
__global__ __launch_bounds__(kPlaneThreads) void source_kernel(SourceArgs a)
{
    source_body<real>(a, blockIdx.x * kPlaneThreads + threadIdx.x, blockIdx.y);
}

// ------------------------------------------------------------------------------------------------
// FS sweep
// ------------------------------------------------------------------------------------------------

struct SweepArgs {
    int nx, ny, nz, n_down;
    const rt3d::PairSeg *pseg;        // window form
    const rt3d::PairLayer *player;    // window form
    const rt3d::ColumnSeg *cseg;      // column form
    const rt3d::PairInfo *pairs;
    const WorkItem *items;
    const void *cs;               // Vec2<real>
    const double *Ibot;           // [ny][nx] intensities at the bottom plane, or null (zero)
    const double *Islope;         // [ny][nx] LTE-diffusion gradient: upward lines add mu * Islope (or null)
    double I_top;
    void *P;                      // real
    double *Iem;                  // [n_up][ny][nx] or null
    const double *Iem_base;       // added to Iem in difference mode (or null)
    const double *xtab;           // [kExpTab] 2^(j/kExpTab), the float64 exponential's table
};

__device__ inline double expm1_sweep(double x, const double *tab) { return expm1_nonpos_tab(x, tab); }
__device__ inline float expm1_sweep(float x, const double *) { return expm1_nonpos(x); }

template <typename real> __device__ inline real seg_length(const rt3d::PairSeg &g);
template <> __device__ inline double seg_length<double>(const rt3d::PairSeg &g) { return g.len; }
template <> __device__ inline float seg_length<float>(const rt3d::PairSeg &g) { return g.len32; }

// x mod n for 0 <= x < 2n, as min(x, x - n) on unsigned integers (x - n wraps when x < n)
__device__ inline unsigned wrap_once(unsigned x, unsigned n) { return min(x, x - n); }

// One workgroup sweeps the lines of one band for both directions A and B of an x-mirrored pair.  The
// two directions' segments have equal lengths and row offsets and negated column offsets, so at every
// segment index a line of A and a line of B cross the same voxel: slot q = (row, column c) of the band
// holds the A line whose top column is c and the B line whose top column is c + 2 dA (mod nx), dA
// being A's column offset at that segment; both are in voxel column c + dA.  The pair then shares the
// voxel's chi,S, the exponential of its optical depth and the deposit cell.  Where dA changes between
// consecutive segments the B lines move between the slots of their row, through a double-buffered
// LDS array (the barrier that ends every segment index orders the write before the read).  Thread t
// owns slots q = t + i*NT (i < LPT).  Per segment index the slots deposit into pairwise distinct cells
// of the band's LDS window, so the window is updated with a plain read-add-write.
template <typename real, int NT, int LPT>
__device__ __forceinline__ void sweep_body(const SweepArgs &a, const WorkItem &it, unsigned char *smem_raw)
{
    using real2 = typename Vec2<real>::type;
    const rt3d::PairInfo pi = a.pairs[it.pair];
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const unsigned plane = unsigned(nx) * unsigned(ny);
    const int nlines = it.rows * nx;
    const int wsize = pi.win_rows * nx;
    const real2 *cs = static_cast<const real2 *>(a.cs);
    // LDS: the band's deposit window, then the two exchange buffers of the B lines
    real *win = reinterpret_cast<real *>(smem_raw);
    real *xch = win + wsize;                                   // [2][nlines]
    real *P = static_cast<real *>(a.P) + pi.p_off + long(it.band) * nz * wsize;

    for (int e = threadIdx.x; e < wsize; e += NT) win[e] = real(0);
    __shared__ double xtab[kExpTab];
    if (std::is_same<real, double>::value && threadIdx.x < kExpTab) xtab[threadIdx.x] = a.xtab[threadIdx.x];

    real IA[LPT], IB[LPT];
    int li[LPT], lj[LPT];
    unsigned lbase[LPT];
#pragma unroll
    for (int t = 0; t < LPT; ++t) {
        const int q = threadIdx.x + t * NT;
        const int qq = q < nlines ? q : 0;
        lj[t] = qq / nx;
        li[t] = q < nlines ? qq - lj[t] * nx : -1;   // -1 marks an unused slot
        lbase[t] = unsigned(lj[t] * nx);
        IA[t] = real(a.I_top);
        IB[t] = real(a.I_top);
    }
    __syncthreads();

    int xpar = 0;              // exchange buffer of the last move of the B lines
    bool moved = false;        // the B lines were written to it before the last barrier
    unsigned sa_last = 0;      // A's column offset at the last segment (the B lines' top columns)
    for (int step = 0; step < nz; ++step) {
        const int k = pi.down ? nz - 1 - step : step;
        const rt3d::PairLayer L = a.player[it.pair * nz + k];
        const real2 *csk = cs + long(k) * plane;
        unsigned grow0[LPT];
#pragma unroll
        for (int t = 0; t < LPT; ++t) {
            unsigned r = unsigned(it.j0 + lj[t] + L.rmin);
            r = wrap_once(wrap_once(r, ny), ny);
            grow0[t] = r * unsigned(nx);
        }
        if (!pi.down && step == 0) {
            // upward lines enter through the bottom plane: boundary light of the entry voxel, the
            // same voxel for the slot's A and B lines
            const rt3d::PairSeg g = a.pseg[L.off];
#pragma unroll
            for (int t = 0; t < LPT; ++t) {
                if (li[t] < 0) continue;
                const unsigned row = wrap_once(grow0[t] + unsigned(g.smnx), plane);
                const unsigned col = wrap_once(unsigned(li[t] + g.saA), nx);
                const double sl = a.Islope ? pi.mu * a.Islope[row + col] : 0.0;
                IA[t] = a.Ibot ? real(a.Ibot[row + col] + sl) : real(0);
                IB[t] = IA[t];
            }
        }
        rt3d::PairSeg g = a.pseg[L.off];
        for (int s = 0; s < L.ns; ++s) {
            // the next segment's descriptor is loaded one segment ahead, so its load latency is not
            // part of the chain of latencies of a segment index
            const rt3d::PairSeg gn = a.pseg[L.off + min(s + 1, L.ns - 1)];
            const real len = seg_length<real>(g);
            // gather of segment s: the voxel of each slot in the chi,S plane
            real2 cv[LPT];
            unsigned wc[LPT];
#pragma unroll
            for (int t = 0; t < LPT; ++t) {
                const unsigned col = wrap_once(unsigned(li[t] + g.saA), nx);
                wc[t] = lbase[t] + unsigned(g.sbnx) + col;
                const unsigned grow = wrap_once(grow0[t] + unsigned(g.smnx), plane);
                if (li[t] >= 0) cv[t] = csk[grow + col];
            }
            // the B lines that moved at the end of the previous segment
            if (moved) {
#pragma unroll
                for (int t = 0; t < LPT; ++t)
                    if (li[t] >= 0) IB[t] = xch[xpar * nlines + int(lbase[t]) + li[t]];
            }
            // At one segment index the slots deposit into distinct cells, so the window cells are
            // read first, ahead of the exponentials, and written after: one LDS wait per segment
            // index, not one per deposit.
            real o[LPT];
#pragma unroll
            for (int t = 0; t < LPT; ++t) o[t] = li[t] >= 0 ? win[wc[t]] : real(0);
#pragma unroll
            for (int t = 0; t < LPT; ++t) {
                if (li[t] < 0) continue;
                const real dtau = cv[t].x * len;
                const real em1 = expm1_sweep(-dtau, xtab);     // e^{-dtau} - 1
                const real dA = (IA[t] - cv[t].y) * em1;
                const real dB = (IB[t] - cv[t].y) * em1;
                IA[t] += dA;
                IB[t] += dB;
                const real sd = cv[t].y * dtau;
                win[wc[t]] = o[t] + ((sd - dA) + (sd - dB));   // chi * integral of I, both lines
            }
            // B lines move by -2 (change of dA) columns in their row before the next segment
            moved = g.shB != 0;
            if (moved) {
                xpar ^= 1;
#pragma unroll
                for (int t = 0; t < LPT; ++t)
                    if (li[t] >= 0)
                        xch[xpar * nlines + int(lbase[t] + wrap_once(unsigned(li[t] + g.shB), nx))] = IB[t];
            }
            sa_last = unsigned(g.saA);
            g = gn;
            __syncthreads();
        }
        real *Pk = P + long(k) * wsize;
        for (int e = threadIdx.x; e < wsize; e += NT) {
            Pk[e] = win[e];
            win[e] = real(0);
        }
        __syncthreads();
    }
    if (!pi.down && a.Iem) {
        const long ea0 = long(pi.dA - a.n_down) * plane, eb0 = long(pi.dB - a.n_down) * plane;
#pragma unroll
        for (int t = 0; t < LPT; ++t) {
            if (li[t] < 0) continue;
            // the B line in this slot entered the top at column li + 2 dA (mod nx)
            const unsigned colB = wrap_once(wrap_once(unsigned(li[t]) + sa_last, nx) + sa_last, nx);
            const long ea = ea0 + (it.j0 + lj[t]) * nx + li[t];
            const long eb = eb0 + (it.j0 + lj[t]) * nx + colB;
            const double baseA = a.Iem_base ? a.Iem_base[ea] : 0.0;
            const double baseB = a.Iem_base ? a.Iem_base[eb] : 0.0;
            a.Iem[ea] = baseA + double(IA[t]);
            a.Iem[eb] = baseB + double(IB[t]);
        }
    }
}

// Two slots per thread fit 64 VGPRs (59 in float64), which lets 8 waves share a SIMD (a band's LDS
// takes ~33 KB at 129 columns in float64, half that in float32, so 4 workgroups of 512 fit a CU); the
// segment loop waits on its gathers, and 8 waves hide that better than 6.  Shapes with more slots per
// thread keep the compiler's choice; the batched kernel has a bound of its own.
template <int LPT> constexpr int kSweepMinWaves = LPT <= 2 ? 8 : 1;

template <typename real, int NT, int LPT>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(kSweepMinWaves<LPT>))) void sweep_kernel(SweepArgs a)
{
    extern __shared__ unsigned char smem_raw[];
    sweep_body<real, NT, LPT>(a, a.items[blockIdx.x], smem_raw);
}

}  // namespace

#include "sweep_columns.h"

namespace {

// Launches n_items workgroups of one problem's sweep in the plan's form.
inline void launch_sweep_kernel(const SweepArgs &a, const rt3d::SweepPlan &plan, int shape, int n_items, bool f32,
                                hipStream_t stream)
{
    const size_t smem = sweep_smem_bytes(plan, f32);
    const dim3 grid(n_items);
    if (plan.columns) {
        const dim3 blk(plan.block_threads);
        if (f32) hipLaunchKernelGGL(column_sweep_kernel<float>, grid, blk, smem, stream, a);
        else hipLaunchKernelGGL(column_sweep_kernel<double>, grid, blk, smem, stream, a);
        return;
    }
    with_sweep_shape(shape, [&](auto tag) {
        using Tag = decltype(tag);
        if (f32)
            hipLaunchKernelGGL((sweep_kernel<float, Tag::threads, Tag::lines>), grid, dim3(Tag::threads), smem, stream, a);
        else
            hipLaunchKernelGGL((sweep_kernel<double, Tag::threads, Tag::lines>), grid, dim3(Tag::threads), smem, stream, a);
    });
}

// ------------------------------------------------------------------------------------------------
// Angle reduction of the partial planes
// ------------------------------------------------------------------------------------------------

struct ReduceArgs {
    int nx, ny, nz, n_pair;
    const rt3d::LayerBlock *blocks;
    const void *P;            // real
    const double *chi;
    const double *J;          // for r = J_fs - J (may be null)
    const double *base;       // difference mode: J_fs of the anchor, added (may be null)
    double *Jfs;
    double *rb;               // chi (J_fs - J), the right-hand side of the OS step (may be null)
    int chunk;                // direction pairs that are summed by themselves (reduce_chunk_pairs)
    int waves;                // wavefronts that share the chunks of a voxel (reduce_waves)
};

// The pairs of a voxel are summed in chunks of this many, and the chunks' sums added in order, so that
// wavefronts can share them.  Only a function of the problem: a batch's members and ranges of pairs
// sum as a single context does.  Grids beyond 2^19 voxels have wavefronts enough and take one chunk.
inline int reduce_chunk_pairs(long V, int n_pair)
{
    return V > (1L << 19) ? n_pair : std::max(4, (n_pair + 63) / 64 * 4);
}

// Wavefronts that share the chunks of the same voxels, a power of 2 of at most one per chunk and max_waves:
// as many as bring the launch (a wavefront takes 128 voxels) up to about 8 wavefronts per SIMD; a
// chain of pairs that each wait for memory is all that a small grid's reduction spends its time on (65^3 x 64 with
// limits of 2, 4, 8 and 16: 56, 52, 46 and 50 us).
// The window form's planes are wide: more waves on other pairs only take the caches from each other where the launch has
// waves enough (600 x 20 x 20 x 256, 1875 wavefronts of voxels: 218, 176, 207 and 254 us with 1, 2, 4 and 8; 513 x 20 x 40 x 256,
// 3206: 295, 313, 331, 421; 520 x 8 x 8 x 256, 260: 118, 61, 45, 35 and with 16 48), so it stops at 2 per SIMD.
inline int reduce_waves(long V, int n_pair, int chunk, int max_waves, bool columns)
{
    int w = 1;
    while (2 * w <= std::min(max_waves, (n_pair + chunk - 1) / chunk) && V / 128 * w < (columns ? 8192 : 2048)) w *= 2;
    return w;
}

// J_fs(v) = (1/chi_v) sum_pairs W|mu| sum over the bands whose deposit windows cover v.  The band of
// voxel row j at layer k is found from the row's offset to the layer's window origin; the previous
// bands (cyclically) still cover the row while the offset stays inside their windows.
__device__ inline rt3d::LayerBlock layer_block(const ReduceArgs &a, int q, int k)
{
    // q and k are the same in all lanes and the table is constant while kernels run: a scalar load
    typedef int v8i __attribute__((ext_vector_type(8)));
    const v8i w = *(const __attribute__((address_space(4))) v8i *)(uintptr_t)(a.blocks + (long(k) * a.n_pair + q));
    rt3d::LayerBlock lb;
    __builtin_memcpy(&lb, &w, sizeof(lb));
    return lb;
}

// Bands of lb's rows each (COL: kColumnRows), the last one of fewer
template <bool COL>
struct BandRow {
    int rows, nb, last;
    int b, off;                  // a band, and the row's offset to its first
    __device__ BandRow(const rt3d::LayerBlock &lb, int ny, int j)
    {
        rows = COL ? rt3d::kColumnRows : lb.flags >> rt3d::kBlockRows;
        int jj = j - lb.rmin;
        jj += (jj < 0) ? ny : 0;
        if (!COL && rows == 1) {
            // what the default shape leaves of a band in the window form: no divisions
            nb = ny;
            last = 1;
            b = jj;
            off = 0;
            return;
        }
        nb = (ny + rows - 1) / rows;
        last = ny - (nb - 1) * rows;
        b = jj / rows;
        off = jj - b * rows;
    }
    __device__ int rows_before() const { return b == 0 ? last : rows; }      // of the band before (cyclically)
    __device__ void back()
    {
        off += rows_before();
        b = (b == 0) ? nb - 1 : b - 1;
    }
    // a band of n rows has n + span: a band that one has stepped back to covers the row where this held before
    __device__ bool before(int span) const { return off < span; }
    __device__ long at(const rt3d::LayerBlock &lb, int nx) const { return long(unsigned(b * lb.stride + off)) * unsigned(nx); }
};

template <typename real> struct ReducePair;      // two neighbours of a row, at any element
template <> struct ReducePair<double> { typedef double type __attribute__((ext_vector_type(2), aligned(8))); };
template <> struct ReducePair<float> { typedef float type __attribute__((ext_vector_type(2), aligned(4))); };

// Adds the sums of the U unsplit pairs from q on, less those that repeat q1 - 1, for the voxels (i, j, k) and
// (i + 1, j, k) to acc0 and acc1, pair by pair in order.  A pair's bands are added in the order b, the one
// before, then earlier ones, for lines that drift down from the earliest on (as reduce_split).  The
// partials of the first two bands of all U pairs are loaded before any is summed (a pair whose row only
// one band covers loads the first band's again and does not add it), so a wave keeps that many loads in
// flight instead of waiting on each pair; the rare third and later bands are read where they are added.
template <typename real, bool COL, int U>
__device__ inline void reduce_group(const ReduceArgs &a, const rt3d::LayerBlock (&lb)[U], int n, int i, int j,
                                    double &acc0, double &acc1)
{
    using real2 = typename ReducePair<real>::type;
    real2 x[U], y[U];
    bool m1[U], more[U];
    const real *Pi = static_cast<const real *>(a.P) + i;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        BandRow<COL> r(lb[u], a.ny, j);
        const real *Pq = Pi + lb[u].off;
        const long o0 = r.at(lb[u], a.nx);
        m1[u] = r.before(lb[u].span);
        r.back();
        more[u] = r.before(lb[u].span);
        x[u] = *reinterpret_cast<const real2 *>(Pq + o0);
        y[u] = *reinterpret_cast<const real2 *>(Pq + (m1[u] ? r.at(lb[u], a.nx) : o0));
    }
    // keep the sums below the group's loads (the scheduler would otherwise interleave them and wait on each
    // pair's loads before issuing the next pair's)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (u >= n) break;
        double s0 = double(x[u].x), s1 = double(x[u].y);
        if (m1[u]) {
            s0 += double(y[u].x);
            s1 += double(y[u].y);
        }
        if (more[u]) {
            // bands thinner than the window halo: still earlier bands cover the row
            const real *Pq = Pi + lb[u].off;
            BandRow<COL> r(lb[u], a.ny, j);
            r.back();
            if (!COL || !(lb[u].flags & rt3d::kBlockDown)) {      // (the window form marks none)
                while (r.before(lb[u].span)) {
                    r.back();
                    const real2 z = *reinterpret_cast<const real2 *>(Pq + r.at(lb[u], a.nx));
                    s0 += double(z.x);
                    s1 += double(z.y);
                }
            } else {
                int m = 0;
                for (; r.before(lb[u].span); ++m) r.back();
                s0 = s1 = 0.0;
                for (; m > 0; --m) {
                    BandRow<COL> e(lb[u], a.ny, j);
                    for (int t = 0; t <= m; ++t) e.back();
                    const real2 z = *reinterpret_cast<const real2 *>(Pq + e.at(lb[u], a.nx));
                    s0 += double(z.x);
                    s1 += double(z.y);
                }
                s0 = (s0 + double(y[u].x)) + double(x[u].x);
                s1 = (s1 + double(y[u].y)) + double(x[u].y);
            }
        }
        acc0 = fma(lb[u].wmu, s0, acc0);
        acc1 = fma(lb[u].wmu, s1, acc1);
    }
}

// The same for a split pair: line row l of the grid has left its deposits for the row t above the layer's
// first in row t of its own block.  The line rows come through a row in the order of t, from 0 for lines that
// drift up and towards 0 for lines that drift down; those of one band are added to each other first, in the
// sweep's precision, which are the sums that a thread of an unsplit band makes.
template <typename real>
__device__ inline void reduce_split(const ReduceArgs &a, const rt3d::LayerBlock &lb, int i, int j, double &acc0,
                                    double &acc1)
{
    using real2 = typename ReducePair<real>::type;
    constexpr int U = 4;
    const real *Pq = static_cast<const real *>(a.P) + lb.off + i;
    const bool up = !(lb.flags & rt3d::kBlockDown);
    const int ny = a.ny, span = lb.span;
    // line row l of the step t, its row in its block, and where a line row is the first of its band
    const int l_step = up ? -1 : 1, t_step = up ? 1 : -1, first = up ? rt3d::kColumnRows - 1 : 0, last = up ? ny - 1 : 0;
    int t0 = up ? 0 : span, l = j - lb.rmin;
    l += (l < 0) ? ny : 0;
    l -= up ? 0 : span % ny;
    l += (l < 0) ? ny : 0;
    double s0 = 0.0, s1 = 0.0;
    real b0 = real(0), b1 = real(0);
    for (int tb = 0; tb <= span; tb += U, t0 += U * t_step) {
        real2 x[U];
        bool fresh[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            // (beyond the last step: the last one again)
            const int t = t0 + t_step * min(u, span - tb);
            x[u] = *reinterpret_cast<const real2 *>(Pq + long(unsigned(l * lb.stride + t)) * unsigned(a.nx));
            fresh[u] = l % rt3d::kColumnRows == first || l == last;
            const int next = l + (tb + u < span ? l_step : 0);
            l = next < 0 ? ny - 1 : next >= ny ? 0 : next;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (tb + u > span) break;
            s0 += fresh[u] ? double(b0) : 0.0;
            s1 += fresh[u] ? double(b1) : 0.0;
            b0 = (fresh[u] ? real(0) : b0) + x[u].x;
            b1 = (fresh[u] ? real(0) : b1) + x[u].y;
        }
    }
    acc0 = fma(lb.wmu, s0 + double(b0), acc0);
    acc1 = fma(lb.wmu, s1 + double(b1), acc1);
}

// The angle sum of the direction pairs [q0, q1) for voxels (i, j, k) and (i + 1, j, k), added to acc0 / acc1.
template <typename real, bool COL>
__device__ inline void reduce_pairs(const ReduceArgs &a, int i, int j, int k, int q0, int q1, double &acc0, double &acc1)
{
    constexpr int U = 4;
    for (int q = q0; q < q1; q += U) {
        rt3d::LayerBlock lb[U];
        int split = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            lb[u] = layer_block(a, min(q + u, q1 - 1), k);
            split |= lb[u].flags & rt3d::kBlockSplit;
        }
        if (!COL || !split) {
            reduce_group<real, COL, U>(a, lb, q1 - q, i, j, acc0, acc1);
            continue;
        }
        for (int u = 0; u < min(U, q1 - q); ++u) {
            const rt3d::LayerBlock one[1] = {layer_block(a, q + u, k)};
            if (one[0].flags & rt3d::kBlockSplit) reduce_split<real>(a, one[0], i, j, acc0, acc1);
            else reduce_group<real, COL, 1>(a, one, 1, i, j, acc0, acc1);
        }
    }
}

__device__ inline void reduce_finish(const ReduceArgs &a, long v, double acc)
{
    const double Jfs = a.base ? a.base[v] + acc / a.chi[v] : acc / a.chi[v];
    a.Jfs[v] = Jfs;
    if (a.rb) a.rb[v] = a.chi[v] * (Jfs - a.J[v]);
}

// Two neighbouring voxels of one row per thread (p2 indexes the (ny, (nx + 1) / 2) voxel pairs of
// plane k; the last pair of an odd row starts one voxel earlier): the band lookup is shared and the
// partials of both are read together.
struct ReduceVoxels {
    bool in;
    int i, j, t0;      // first voxel, and the first of the two that is this thread's to write
    long v;
};
__device__ inline ReduceVoxels reduce_voxels(const ReduceArgs &a, int p2, int k)
{
    const int hx = (a.nx + 1) / 2;
    ReduceVoxels r;
    r.in = p2 < hx * a.ny;
    p2 = min(p2, hx * a.ny - 1);
    r.j = p2 / hx;
    const int h = p2 - r.j * hx;
    r.i = min(2 * h, a.nx - 2);
    r.t0 = 2 * h - r.i;
    r.v = long(k) * a.nx * a.ny + long(r.j) * a.nx + r.i;
    return r;
}

// Block b of plane k: blockDim.x / a.waves voxel pairs, whose chunks the block's thread groups share
// (LDS: reduce_smem_bytes).  What bounds it: the partial planes' bytes on large grids (3.1 GB at 129^3 x 256, read at
// 4.8 TB/s; 4 pairs' loads in flight per wave, a row's address by one scalar load and a few integer operations per
// pair), the chain of pairs on small ones.  us per launch with one chain of pairs per voxel and the tables read
// by vector loads, and now: 17^3 x 64 45 and 7, 65^3 x 64 55 and 33, 65^3 x 256 193 and 159, 129^3 x 256 654 and 642,
// 129 x 129 x 193 x 256 in float32 746 and 645, the benchmark batch of 12 grids up to 97^3 417 and 290.  Window form (float64 /
// float32): 600 x 20 x 20 x 256 204 / 161 and 179 / 115, 600 x 200 x 40 x 64 719 / 463 and 716 / 416, 1000 x 30 x 30 x 64 174 / 92
// and 171 / 77, 1024 x 40 x 10 x 128 147 / 94 and 145 / 95, 513 x 64 x 64 x 256 1247 / 837 and 1292 / 759.
template <typename real, bool COL>
__device__ inline void reduce_body(const ReduceArgs &a, int b, int k, double2 *part)
{
    const int W = a.waves, n = int(blockDim.x) / W;          // voxel pairs of this block
    const int w = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / n), p = int(threadIdx.x) - w * n;
    const ReduceVoxels r = reduce_voxels(a, b * n + p, k);
    const int n_chunk = (a.n_pair + a.chunk - 1) / a.chunk, per = (n_chunk + W - 1) / W;
    double acc0 = 0.0, acc1 = 0.0;
    for (int c = w * per; c < min(n_chunk, (w + 1) * per); ++c) {
        double s0 = 0.0, s1 = 0.0;
        reduce_pairs<real, COL>(a, r.i, r.j, k, c * a.chunk, min(a.n_pair, (c + 1) * a.chunk), s0, s1);
        if (W > 1) part[c * n + p] = make_double2(s0, s1);
        acc0 += s0;
        acc1 += s1;
    }
    if (W > 1) {
        __syncthreads();
        if (w > 0) return;
        acc0 = acc1 = 0.0;
        for (int c = 0; c < n_chunk; ++c) {
            const double2 s = part[c * n + p];
            acc0 += s.x;
            acc1 += s.y;
        }
    }
    if (!r.in) return;
    if (r.t0 == 0) reduce_finish(a, r.v, acc0);
    reduce_finish(a, r.v + 1, acc1);
}

inline int reduce_threads(const ReduceArgs &a) { return std::max(kPlaneThreads, 64 * a.waves); }
inline size_t reduce_smem_bytes(const ReduceArgs &a, int threads)
{
    return a.waves > 1 ? size_t((a.n_pair + a.chunk - 1) / a.chunk) * (threads / a.waves) * sizeof(double2) : 0;
}
inline int reduce_blocks(const ReduceArgs &a, int threads)      // per plane
{
    const int n = threads / a.waves;
    return ((a.nx + 1) / 2 * a.ny + n - 1) / n;
}

template <typename real, bool COL>
__global__ __launch_bounds__(1024) void reduce_kernel_pair(ReduceArgs a)
{
    extern __shared__ double2 reduce_part[];
    reduce_body<real, COL>(a, blockIdx.x, blockIdx.y, reduce_part);
}

inline void launch_reduce_kernel(ReduceArgs &a, bool columns, bool f32, hipStream_t stream)
{
    const long V = long(a.nx) * a.ny * a.nz;
    a.chunk = reduce_chunk_pairs(V, a.n_pair);
    a.waves = reduce_waves(V, a.n_pair, a.chunk, 16, columns);
    const int threads = reduce_threads(a);
    const dim3 grid(reduce_blocks(a, threads), a.nz);
    const size_t smem = reduce_smem_bytes(a, threads);
    if (columns) {
        if (f32) hipLaunchKernelGGL((reduce_kernel_pair<float, true>), grid, dim3(threads), smem, stream, a);
        else hipLaunchKernelGGL((reduce_kernel_pair<double, true>), grid, dim3(threads), smem, stream, a);
    } else {
        if (f32) hipLaunchKernelGGL((reduce_kernel_pair<float, false>), grid, dim3(threads), smem, stream, a);
        else hipLaunchKernelGGL((reduce_kernel_pair<double, false>), grid, dim3(threads), smem, stream, a);
    }
}

// Direction pairs [q0, q1) and the layers from k0 on only: starts from 0 (first) or from what a range before left, the sum of the whole
// chunks in Jfs and of the chunk begun in carry (may be null where there is one chunk: Jfs holds its sum
// then), and finishes only when last, so ranges taken in order give bitwise the sum of one pass over all
// pairs.
template <bool COL>
__global__ __launch_bounds__(kPlaneThreads) void reduce_kernel_pair_range(ReduceArgs a, int q0, int q1, int k0, int first,
                                                                          int last, double *carry)
{
    const int k = k0 + int(blockIdx.y);
    const ReduceVoxels r = reduce_voxels(a, int(blockIdx.x) * kPlaneThreads + int(threadIdx.x), k);
    if (!r.in) return;
    const bool one = a.chunk >= a.n_pair;
    double *begun = one ? a.Jfs : carry;
    double acc[2] = {0.0, 0.0}, part[2] = {0.0, 0.0};
    for (int t = r.t0; t < 2 && !first; ++t) {
        acc[t] = one ? 0.0 : a.Jfs[r.v + t];
        part[t] = begun[r.v + t];
    }
    for (int q = q0; q < q1;) {
        const int qe = min(q1, (q / a.chunk + 1) * a.chunk);
        reduce_pairs<double, COL>(a, r.i, r.j, k, q, qe, part[0], part[1]);
        if (qe % a.chunk == 0 || qe == a.n_pair)
            for (int t = 0; t < 2; ++t) {
                acc[t] += part[t];
                part[t] = 0.0;
            }
        q = qe;
    }
    for (int t = r.t0; t < 2; ++t) {
        if (last) {
            reduce_finish(a, r.v + t, acc[t]);
        } else {
            if (!one) a.Jfs[r.v + t] = acc[t];
            begun[r.v + t] = part[t];
        }
    }
}


// ------------------------------------------------------------------------------------------------
// Lambda*
// ------------------------------------------------------------------------------------------------

struct LstarArgs {
    int nx, ny, nz, n_pair;
    int early_exit;                 // 1: no line can wrap back onto a neighbour within two layers
    const rt3d::PairInfo *pairs;    // x-mirrored direction pairs (the tables of direction dA are read)
    const int *seg_off, *seg_n, *seg_ai, *seg_bi;
    const double *seg_len;
    const rt3d::ColumnSeg *cseg;    // the pairs' segments in sweep order, with what follows each
    const double *chi;
    double *L;                      // [27][V]
    double *T;                      // [18][V] scratch for the sums of the downward pairs (null: all pairs into L)
    int tx, ty;                     // tile of the tiled form (0: not taken)
    const double *xtab;             // [kExpTab] 2^(j/kExpTab), the float64 exponential's table
};

// x + expm1(-x) = e^{-x} - 1 + x for x >= 0 (em1 = e^{-x} - 1 given); below 1/2 by Horner on x^2
// (1/2! - x/3! + x^2/4! - ...) through x^15/17!, which avoids the cancellation of the direct form for
// thin segments.
__device__ inline double self_term(double x, double em1)
{
    if (x >= 0.5) return x + em1;
    constexpr double inv_fact[18] = {
        1.0, 1.0, 1.0 / 2, 1.0 / 6, 1.0 / 24, 1.0 / 120, 1.0 / 720, 1.0 / 5040, 1.0 / 40320,
        1.0 / 362880, 1.0 / 3628800, 1.0 / 39916800, 1.0 / 479001600, 1.0 / 6227020800.0,
        1.0 / 87178291200.0, 1.0 / 1307674368000.0, 1.0 / 20922789888000.0,
        1.0 / 355687428096000.0};
    double r = inv_fact[17];
#pragma unroll
    for (int n = 16; n >= 2; --n) r = inv_fact[n] - x * r;
    return x * x * r;
}

__device__ inline int wrap_small(int a, int n)
{
    // a may be any integer; returns a mod n in [0, n)
    int r = a % n;
    return r < 0 ? r + n : r;
}

// Lambda*_{vu} = sum_d W_d |mu_d| / chi_v * sum over the segments s of direction d inside v of
//   delta_uv (dtau_s + em1_s) - em1_s * sum over earlier segments s' in u of c_{s'->s},
//   c_{s'->s} = (1 - e_{s'}) prod_{s' < s'' < s} e_{s''},  e = exp(-dtau).
// The lines through v are the reference line shifted so that its segment s lies in v; walking that
// line backwards through the current and the previous layer reaches every earlier segment that can
// lie in the 3x3x3 block (lines are monotone in z).  The two directions of an x-mirrored pair have
// equal segment lengths and row offsets and negated column offsets, so one walk over direction A's
// table serves both (B's voxels at the mirrored columns), and their self terms are equal.
// One wavefront per workgroup, small workgroups letting many of them share a CU to hide the latency of
// the gathers along the lines (measured at 129^3 x 256: 31.7 ms with 256 threads, 29.2 ms with 128,
// 26.4 ms with 64).  The accumulators live in LDS.  A walk reaches the voxel's own layer and the one it
// came from: layer k + 1 for the downward pairs, k - 1 for the upward ones, and the pairs come in two
// runs (all of one vertical direction, then all of the other; the plan checks this).  So a thread
// keeps 18 accumulators, its own layer's 9 and those of the run's other layer, which are stored and
// cleared between the runs: every entry sums the same terms in the same order as with 27.
// With a.T only the downward pairs are walked, chi_v times their part goes there and the rest follows by symmetry
// (see lstar_tile_body, which grids that cannot wrap take instead): half the time.
constexpr int kLstarThreads = 64;
// Columns p (p = j nx + i; p >= nx ny: none) of plane k; the whole block calls this.
__device__ inline void lstar_body(const LstarArgs &a, int p, int k)
{
    __shared__ double acc[18][kLstarThreads];   // [0, 9): layer k; [9, 18): the current run's other layer
    __shared__ double xtab[kExpTab];
    for (int q = threadIdx.x; q < kExpTab; q += kLstarThreads) xtab[q] = a.xtab[q];
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const bool valid = p < nx * ny;
    const int j = valid ? p / nx : 0, i = valid ? p - (p / nx) * nx : 0;
    const long plane = long(nx) * ny;
    const long V = plane * nz;
    const long v = k * plane + long(j) * nx + i;
    for (int o = 0; o < 18; ++o) acc[o][threadIdx.x] = 0.0;
    __syncthreads();
    const double chiv = a.chi[v];
    // 3x3x3 block index of a column offset m (mod n) from v: 0 for -1, 1 for 0, 2 for +1, -1 outside
    auto block_col = [](int m, int n) { return (m == 0) ? 1 : (m == 1) ? 2 : (m == n - 1) ? 0 : -1; };
    // the other layer's 9 entries of the 27-point row (entries 0..8 for k - 1, 18..26 for k + 1)
    auto store_other = [&](int down) {
        const int o0 = down ? 18 : 0;
        if (valid)
            for (int o = 0; o < 9; ++o) a.L[(o0 + o) * V + v] = acc[9 + o][threadIdx.x];
        for (int o = 0; o < 9; ++o) acc[9 + o][threadIdx.x] = 0.0;
    };
    int run_down = a.n_pair > 0 ? a.pairs[0].down : 0;
    bool stored_up = false, stored_down = false;    // the layers k - 1 and k + 1 have been written
    for (int q = 0; q < a.n_pair; ++q) {
        const rt3d::PairInfo pi = a.pairs[q];
        if (a.T && !pi.down) continue;
        if (pi.down != run_down && !a.T) {
            store_other(run_down);
            stored_down = stored_down || run_down;
            stored_up = stored_up || !run_down;
            run_down = pi.down;
        }
        const double fac = a.T ? pi.wmu : pi.wmu / chiv;
        const int d = pi.dA;
        const int dk = d * nz + k;
        const int off = a.seg_off[dk], n = a.seg_n[dk];
        const int ku = pi.down ? k + 1 : k - 1;
        const bool has_up = ku >= 0 && ku < nz;
        const int offu = has_up ? a.seg_off[d * nz + ku] : 0;
        const int nu = has_up ? a.seg_n[d * nz + ku] : 0;
        for (int s = 0; s < n; ++s) {
            const int as = a.seg_ai[off + s], bs = a.seg_bi[off + s];
            const double dtau = chiv * a.seg_len[off + s];
            const double em1 = expm1_nonpos_tab(-dtau, xtab);
            acc[4][threadIdx.x] += 2.0 * (fac * self_term(dtau, em1));
            const double g = -fac * em1;
            double prodA = 1.0, prodB = 1.0;
            // walk back: current layer s-1 .. 0, then the previous layer from its last segment
            const int total = s + nu;
            for (int w = 0; w < total; ++w) {
                int idx, base;
                if (w < s) { idx = off + s - 1 - w; base = 0; }
                else { idx = offu + nu - 1 - (w - s); base = 9; }
                const int dA = a.seg_ai[idx] - as, dB = a.seg_bi[idx] - bs;
                if (a.early_exit && (dA > 1 || dA < -1 || dB > 1 || dB < -1)) break;
                // with early exit the offsets are -1, 0 or 1 here
                const int mA = a.early_exit ? dA + (dA < 0 ? nx : 0) : wrap_small(dA, nx);
                const int mB = a.early_exit ? dB + (dB < 0 ? ny : 0) : wrap_small(dB, ny);
                const int mAm = (mA == 0) ? 0 : nx - mA;      // direction B's column offset, -dA mod nx
                int colA = i + mA, colB = i + mAm;
                colA -= (colA >= nx) ? nx : 0;
                colB -= (colB >= nx) ? nx : 0;
                int row = j + mB;
                row -= (row >= ny) ? ny : 0;
                const long ub = long(base ? ku : k) * plane + long(row) * nx;
                const double len = a.seg_len[idx];
                double eA, em1A, eB, em1B;
                exp_pair_tab(-a.chi[ub + colA] * len, xtab, eA, em1A);
                exp_pair_tab(-a.chi[ub + colB] * len, xtab, eB, em1B);
                const int oj = block_col(mB, ny);
                const int oiA = block_col(mA, nx), oiB = block_col(mAm, nx);
                if (oiA >= 0 && oj >= 0) acc[base + 3 * oj + oiA][threadIdx.x] += g * (-em1A * prodA);
                if (oiB >= 0 && oj >= 0) acc[base + 3 * oj + oiB][threadIdx.x] += g * (-em1B * prodB);
                prodA *= eA;
                prodB *= eB;
            }
        }
    }
    if (a.T) {
        if (valid)
            for (int o = 0; o < 18; ++o) a.T[o * V + v] = acc[o][threadIdx.x];
        return;
    }
    store_other(run_down);
    stored_down = stored_down || run_down;
    stored_up = stored_up || !run_down;
    // a layer no run reached (all pairs of one vertical direction) has no entries
    if (valid && !stored_up)
        for (int o = 0; o < 9; ++o) a.L[o * V + v] = 0.0;
    if (valid && !stored_down)
        for (int o = 0; o < 9; ++o) a.L[(18 + o) * V + v] = 0.0;
    if (valid)
        for (int o = 0; o < 9; ++o) a.L[(9 + o) * V + v] = acc[o][threadIdx.x];
}

// Tiled form, for grids whose lines cannot wrap back (early_exit).
// K_vu = chi_v Lambda*_vu is symmetric, and the walk of an upward line from v to u is that of the reversed
// downward line from u to v, so the downward pairs alone give all of it: with D the part that they add,
// K_vu = D_vu + D_uv for voxels of one layer and K_vu = D_vu, K_uv = D_vu for u in the layer above.
// A walk crosses at most one face of each axis, so it has at most three steps, and the exponential of a voxel
// and segment is the same for every walk that comes through it.  So a workgroup takes tx x ty columns of a layer,
// a thread for each and for one more to each side: for one segment index after another (the last three
// of the layer above, then the layer's own) each thread computes its voxel's exponential once and leaves it
// in LDS, where the neighbours' walks find it up to three segments later.  Pairs with the same sign of
// the y drift follow each other, and of a pair P is the line that drifts to larger x, M the other, so
// the neighbour that a step reaches is known but for which axes it has crossed: 12 sums in registers.
// What bounds it: float64 arithmetic, one exponential (about 30 instructions) and one self term per voxel
// and segment index, and beside it the scalar unit (the walk's branches and addresses; a segment is one 16-byte
// scalar load: with three loads and the crossings worked out here 561 us at 65^3 x 256 against 495).  us before (a walk
// per thread, each step with two exponentials and gathers of its own, both vertical directions) and now, with the
// fold: 17^3 x 64 222 and 75, 65^3 x 256 1936 and 517, 129^3 x 256 10950 and 3350, the benchmark batch of 12 grids up to
// 97^3 6845 and 2280.  Workgroups of up to 512, 768 or 1024 threads, with less halo, waited longer at their barriers
// (65^3 x 256: 790, 980 and 790 us against 561 at 256), smaller ones had more halo (192: 678, 128: 687); two segments per
// barrier 583.
constexpr int kLstarTileThreads = 256;
// acc += x y on a tied operand: in the cases of a switch the compiler would copy all sums to merge the paths
__device__ __forceinline__ void fma_to(double &acc, double x, double y)
{
    asm volatile("v_fma_f64 %0, %1, %2, %0" : "+v"(acc) : "v"(x), "v"(y));
}

__device__ inline void lstar_tile_body(const LstarArgs &a, int tile, int k, double2 *ring)
{
    __shared__ double xtab[kExpTab];
    if (threadIdx.x < kExpTab) xtab[threadIdx.x] = a.xtab[threadIdx.x];
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const long plane = long(nx) * ny, V = plane * nz;
    const int ntx = (nx + a.tx - 1) / a.tx, by = tile / ntx, bx = tile - by * ntx;
    const int ex = a.tx + 2, E = ex * (a.ty + 2);
    const int q = min(int(threadIdx.x), E - 1);
    const int ly = q / ex, lx = q - ly * ex;
    const int x0 = bx * a.tx + lx - 1, y0 = by * a.ty + ly - 1;      // in [-1, 2 n)
    auto wrap = [](int x, int n) {
        x += x < 0 ? n : 0;
        return x - (x >= n ? n : 0);
    };
    const bool inner = int(threadIdx.x) < E && unsigned(lx - 1) < unsigned(a.tx) && unsigned(ly - 1) < unsigned(a.ty) &&
                       x0 < nx && y0 < ny;
    const long p = long(wrap(y0, ny)) * nx + wrap(x0, nx);
    const double chiv = a.chi[k * plane + p], chiu = a.chi[(k + 1 < nz ? k + 1 : k) * plane + p];
    // (threads without an output read their neighbours' cells as an inner thread does)
    const int c = min(max(ly, 1), a.ty) * ex + min(max(lx, 1), a.tx);
    auto scalar_int = [](const int *x) { return *(const __attribute__((address_space(4))) int *)(uintptr_t)x; };
    auto scalar_len = [](const double *x) { return *(const __attribute__((address_space(4))) double *)(uintptr_t)x; };
    double mid[2][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}};     // [layer above][upstream column -1, 0, 1], the voxel's own row
#pragma unroll 1
    for (int cls = 0; cls < 2; ++cls) {
        // lines that drift to larger y (their upstream row is j - 1), then to smaller
        const int dy = cls == 0 ? -ex : ex;
        double s000 = 0.0, s010 = 0.0, s001 = 0.0, s011 = 0.0;                         // [x y z crossed]
        double p100 = 0.0, p110 = 0.0, p101 = 0.0, p111 = 0.0, m100 = 0.0, m110 = 0.0, m101 = 0.0, m111 = 0.0;
        auto add = [&](int bits, double gP, double cP, double gM, double cM) {
            switch (bits) {
            case 1: fma_to(p100, gP, cP); fma_to(m100, gM, cM); break;
            case 2: fma_to(s010, gP, cP); fma_to(s010, gM, cM); break;
            case 3: fma_to(p110, gP, cP); fma_to(m110, gM, cM); break;
            case 4: fma_to(s001, gP, cP); fma_to(s001, gM, cM); break;
            case 5: fma_to(p101, gP, cP); fma_to(m101, gM, cM); break;
            case 6: fma_to(s011, gP, cP); fma_to(s011, gM, cM); break;
            default: fma_to(p111, gP, cP); fma_to(m111, gM, cM); break;
            }
        };
        for (int r = 0; r < a.n_pair; ++r) {
            const rt3d::PairInfo *pi = a.pairs + r;
            if (!scalar_int(&pi->down) || (scalar_int(&pi->ysgn) < 0) != (cls == 1)) continue;
            const int dk = scalar_int(&pi->dA) * nz + k;
            const double wmu = scalar_len(&pi->wmu);
            const int n = scalar_int(a.seg_n + dk), m = k + 1 < nz ? min(scalar_int(a.seg_n + dk + 1), 3) : 0;
            // the pair's list in sweep order, from the last m segments of the layer above on
            const int before = scalar_int(&pi->n_seg) - n - (scalar_int(a.seg_off + dk) - scalar_int(a.seg_off + dk - k));
            const rt3d::ColumnSeg *sp = a.cseg + (scalar_int(&pi->c_off) + before - m);
            // axes crossed on coming into each of the last three segments: the flags of the one before each
            int b1 = 0, b2 = 0, b3 = 0, flags = 0;
            auto advance = [&](double &len) {
                typedef int v4i __attribute__((ext_vector_type(4)));
                const v4i w = *(const __attribute__((address_space(4))) v4i *)(uintptr_t)sp;
                ++sp;
                b3 = b2;
                b2 = b1;
                b1 = flags;
                flags = w.z;
                len = __hiloint2double(w.y, w.x);
            };
            double len;
            __syncthreads();
#pragma unroll 1
            for (int t = 0; t < m; ++t) {
                advance(len);
                double e, em1;
                exp_pair_tab(-chiu * len, xtab, e, em1);
                ring[t * E + q] = make_double2(e, em1);
            }
            // the sums of segment t of the layer, whose optical depth and e^-x - 1 are x and em1
            auto sums = [&](int t, double x, double em1) {
                fma_to(s000, 2.0 * wmu, self_term(x, em1));
                const double g = wmu * em1;
                if (t < 1) return;
                const int d1 = ((b1 & 2) ? dy : 0) + c, x1 = b1 & 1;
                const double2 *row = ring + ((t - 1) & 3) * E;
                const double2 P1 = row[d1 - x1], M1 = row[d1 + x1];
                add(b1, g, P1.y, g, M1.y);
                if (t < 2 || (b1 & b2)) return;
                const int b12 = b1 | b2, d2 = ((b12 & 2) ? dy : 0) + c, x2 = b12 & 1;
                const double2 *row2 = ring + ((t - 2) & 3) * E;
                const double2 P2 = row2[d2 - x2], M2 = row2[d2 + x2];
                const double gP = g * P1.x, gM = g * M1.x;
                add(b12, gP, P2.y, gM, M2.y);
                if (t < 3 || (b12 & b3)) return;
                const int b123 = b12 | b3, d3 = ((b123 & 2) ? dy : 0) + c, x3 = b123 & 1;
                const double2 *row3 = ring + ((t - 3) & 3) * E;
                add(b123, gP * P2.x, row3[d3 - x3].y, gM * M2.x, row3[d3 + x3].y);
            };
#pragma unroll 1
            for (int t = m; t < m + n; ++t) {
                advance(len);
                const double x = chiv * len;
                double e, em1;
                exp_pair_tab(-x, xtab, e, em1);
                // after the barrier no thread reads segment t - 4 any more, whose place this one takes
                __syncthreads();
                ring[(t & 3) * E + q] = make_double2(e, em1);
                sums(t, x, em1);
            }
        }
        if (inner) {
            // rows j - 1 (lines to larger y) and j + 1 are complete; the voxel's own row has terms of both
            double *T = a.T + k * plane + p;
            const int row = cls == 0 ? 0 : 6;
            T[(row + 0) * V] = p110;
            T[(row + 1) * V] = s010;
            T[(row + 2) * V] = m110;
            T[(9 + row + 0) * V] = p111;
            T[(9 + row + 1) * V] = s011;
            T[(9 + row + 2) * V] = m111;
        }
        mid[0][0] += p100; mid[0][1] += s000; mid[0][2] += m100;
        mid[1][0] += p101; mid[1][1] += s001; mid[1][2] += m101;
    }
    if (inner) {
        double *T = a.T + k * plane + p;
#pragma unroll
        for (int z = 0; z < 2; ++z)
#pragma unroll
            for (int x = 0; x < 3; ++x) T[(9 * z + 3 + x) * V] = mid[z][x];
    }
}

__global__ __launch_bounds__(kLstarTileThreads) __attribute__((amdgpu_waves_per_eu(6))) void lstar_tile_kernel(LstarArgs a)
{
    extern __shared__ double2 lstar_ring[];
    lstar_tile_body(a, blockIdx.x, blockIdx.y, lstar_ring);
}

// Lambda* from the downward pairs' sums: T[0, 9) of the voxel's layer, T[9, 18) of the layer above
__global__ __launch_bounds__(kPlaneThreads) void lstar_fold_kernel(LstarArgs a)
{
    const int nx = a.nx, ny = a.ny, k = blockIdx.y, p = int(blockIdx.x) * kPlaneThreads + int(threadIdx.x);
    if (p >= nx * ny) return;
    const int j = p / nx, i = p - j * nx;
    const long plane = long(nx) * ny, V = plane * a.nz, v = k * plane + p;
    const int cols[3] = {i == 0 ? nx - 1 : i - 1, i, i == nx - 1 ? 0 : i + 1};
    const int rows[3] = {j == 0 ? ny - 1 : j - 1, j, j == ny - 1 ? 0 : j + 1};
    const double inv = 1.0 / a.chi[v];
#pragma unroll
    for (int o = 0; o < 9; ++o) {
        const long u = long(rows[o / 3]) * nx + cols[o % 3];
        // the voxel's own entry: upward lines add what the downward ones do
        a.L[(9 + o) * V + v] = inv * (a.T[o * V + v] + a.T[(8 - o) * V + k * plane + u]);
        a.L[(18 + o) * V + v] = inv * a.T[(9 + o) * V + v];
        a.L[o * V + v] = k > 0 ? inv * a.T[(17 - o) * V + (k - 1) * plane + u] : 0.0;
    }
}

// The tile of the tiled form: the fewest wavefronts that cover a layer with workgroups of at most
// kLstarTileThreads threads.
inline void lstar_tile(int nx, int ny, int &tx, int &ty)
{
    long best = 0;
    for (int cx = 1; cx <= nx; ++cx) {
        const int w = (nx + cx - 1) / cx;
        if (w + 2 > kLstarTileThreads / 3) continue;
        for (int h = 1; h <= ny && (w + 2) * (h + 2) <= kLstarTileThreads; ++h) {
            const long waves = long((nx + w - 1) / w) * ((ny + h - 1) / h) * (((w + 2) * (h + 2) + 63) / 64);
            if (best == 0 || waves < best) {
                best = waves;
                tx = w;
                ty = h;
            }
        }
    }
}
inline int lstar_tile_threads(const LstarArgs &a) { return ((a.tx + 2) * (a.ty + 2) + 63) / 64 * 64; }
inline int lstar_tile_blocks(const LstarArgs &a) { return ((a.nx + a.tx - 1) / a.tx) * ((a.ny + a.ty - 1) / a.ty); }
inline size_t lstar_tile_lds(const LstarArgs &a) { return size_t(4) * (a.tx + 2) * (a.ty + 2) * sizeof(double2); }

// Whether the downward pairs' sums, folded by symmetry, give Lambda*.  A function of the problem alone: the two forms round
// differently, and a batch's member builds what a single context does, whatever the sweep's shape and splits.
// The sums' 18 planes lie in the partial planes' buffer, which only a sweep and its reduction use and which is made that large
// (lstar_scratch): 12 pairs have 16 to 23 V elements of their own, 8 at most 17.3, and would need half as much memory again
// (65^3, new medium and Lambda*, both forms: 2 x 12 angles 232 and 141 us; 4 x 4, in the full form, 140).
// Symmetry holds between tables of opposite directions that mirror each other, and the tile's walks cross a face at every
// step: with slivers neither is so (8 x 20 angles, 3000 layers of chi = 30: corner entries off by 2% in tiles; 4 x 12, 1200
// layers: entries of 5e-9 of their row off by 8e-6 by symmetry), and all pairs are walked voxel by voxel.
inline bool lstar_by_symmetry(const rt3d::SweepPlan &plan) { return plan.n_pair >= 12 && !plan.slivers; }
inline int64_t lstar_scratch(const rt3d::SweepPlan &plan)
{
    return lstar_by_symmetry(plan) ? 18 * int64_t(plan.nx) * plan.ny * plan.nz : 0;
}

template <typename Ctx>
inline void lstar_args(Ctx *c, LstarArgs &a)
{
    a = LstarArgs{};
    a.nx = c->g.nx; a.ny = c->g.ny; a.nz = c->g.nz; a.n_pair = c->plan.n_pair;
    a.early_exit = c->lstar_early_exit;
    a.pairs = c->pairs; a.seg_off = c->seg_off; a.seg_n = c->seg_n; a.seg_ai = c->seg_ai;
    a.seg_bi = c->seg_bi; a.seg_len = c->seg_len64; a.cseg = c->cseg; a.chi = c->chi; a.L = c->L;
    a.xtab = c->xtab;
    if (lstar_by_symmetry(c->plan)) {
        a.T = static_cast<double *>(c->P);
        if (a.early_exit) lstar_tile(a.nx, a.ny, a.tx, a.ty);
    }
}

// Launches the fold of the downward pairs' sums into Lambda*
inline void launch_lstar_fold(const LstarArgs &a, hipStream_t stream)
{
    hipLaunchKernelGGL(lstar_fold_kernel, dim3((a.nx * a.ny + kPlaneThreads - 1) / kPlaneThreads, a.nz), dim3(kPlaneThreads), 0,
                       stream, a);
}

__global__ __launch_bounds__(kLstarThreads) void lstar_kernel(LstarArgs a)
{
    lstar_body(a, blockIdx.x * kLstarThreads + threadIdx.x, blockIdx.y);
}

// Jacobi coefficients.  K_vu = chi_v Lambda*_vu is symmetric (reciprocity: lines for Omega and -Omega
// coincide and the weights are symmetric), so only the 13 upper neighbours o = 14..26 are stored:
// Kc[o - 14][v] = chi_v Lambda*_o(v).  The entry for a lower neighbour u = v + d(o), o < 13, is
// Kc[12 - o][u] (u's upper neighbour 26 - o is v).  Per voxel: invD = 1 / (chi_v (1 - Lambda*_vv (1-eps_v)))
// and E = (1 - eps_v) invD.
template <typename coef>
__global__ __launch_bounds__(kPlaneThreads) void coef_kernel(int nx, int ny, int nz,
                                                             const double *__restrict__ L,
                                                             const double *__restrict__ chi,
                                                             const double *__restrict__ eps,
                                                             coef *__restrict__ Kc, double *__restrict__ invD,
                                                             double *__restrict__ E)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    const int k = blockIdx.y;
    if (p >= nx * ny) return;
    const long plane = long(nx) * ny, V = plane * nz, v = k * plane + p;
    const double c = chi[v];
    for (int o = 14; o < 27; ++o) {
        const int kk = k + o / 9 - 1;
        Kc[(o - 14) * V + v] = coef((kk < nz) ? c * L[o * V + v] : 0.0);
    }
    const double inv = 1.0 / (c * (1.0 - L[13 * V + v] * (1.0 - eps[v])));
    invD[v] = inv;
    E[v] = (1.0 - eps[v]) * inv;
}

// ------------------------------------------------------------------------------------------------
// Jacobi sweep of the OS equations, optionally fused with the J update and max |dJ|/|J|
// ------------------------------------------------------------------------------------------------

// The sweep dJ_v <- (r_v + sum_{u != v} Lambda*_vu (1-eps_u) dJ_u) / (1 - Lambda*_vv (1-eps_v)) is
// evaluated as (chi_v r_v + sum_u K_vu w_u) invD_v with w = (1 - eps) dJ carried between sweeps.
struct JacobiArgs {
    int nx, ny, nz;
    const double *b;             // chi (J_fs - J_old): the right-hand side of the chi-scaled system
    const void *Kc;              // [13][V] upper coefficients (double, or float in the FP32 form)
    const double *invD, *E;
    const double *w_in;          // (1 - eps) dJ of the previous sweep; null: dJ^0 = 0 (first sweep)
    double *w_out;               // (1 - eps) dJ of this sweep (intermediate sweeps)
    double *J;                   // last sweep: J += dJ (null otherwise)
    unsigned long long *maxrel;  // bits of max |dJ|/|J| (non-negative doubles order like integers)
    const double *Ja;            // anchor iterate of the FP32 form (may be null)
    unsigned long long *maxdist; // bits of max |J - Ja|/|J| when Ja is given, of max |J| when abs_measure
    int *nonfinite;
    int abs_measure;             // 1: maxrel receives max |dJ| and maxdist max |J| (iterates that may vanish)
};

// Block max of q and of the anchor distance into maxrel / maxdist (as integer bits: non-negative
// doubles order like integers); NaN/Inf raise the flag.  The whole block must call this.
__device__ inline void jacobi_block_max(const JacobiArgs &a, double q, double dist, bool bad)
{
    if (bad) { atomicOr(a.nonfinite, 1); q = 0.0; dist = 0.0; }
    for (int offs = 32; offs > 0; offs >>= 1) {
        q = fmax(q, __shfl_xor(q, offs));
        dist = fmax(dist, __shfl_xor(dist, offs));
    }
    __shared__ double wmax[2][16];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) { wmax[0][wid] = q; wmax[1][wid] = dist; }
    __syncthreads();
    if (threadIdx.x == 0) {
        double m = wmax[0][0], md = wmax[1][0];
        for (int w = 1; w < int(blockDim.x) / 64; ++w) { m = fmax(m, wmax[0][w]); md = fmax(md, wmax[1][w]); }
        atomicMax(a.maxrel, static_cast<unsigned long long>(__double_as_longlong(m)));
        if (a.Ja || a.abs_measure) atomicMax(a.maxdist, static_cast<unsigned long long>(__double_as_longlong(md)));
    }
}

// The last sweep of a step: J += dJ, and the convergence measures of voxel v folded into q / dist.
__device__ inline void jacobi_update(const JacobiArgs &a, long v, double acc, double &q, double &dist, bool &bad)
{
    const double dJ = acc * a.invD[v];
    const double Jn = a.J[v] + dJ;
    a.J[v] = Jn;
    double qv, dv = 0.0;
    if (a.abs_measure) {
        qv = fabs(dJ);
        dv = fabs(Jn);
    } else {
        qv = fabs(dJ) / fabs(Jn);
        if (a.Ja) dv = fabs(Jn - a.Ja[v]) / fabs(Jn);
    }
    if (!isfinite(Jn) || !isfinite(qv)) {
        bad = true;
    } else {
        q = fmax(q, qv);
        dist = fmax(dist, dv);
    }
}

// Arithmetic is float64 for either coefficient type.
// The whole block must call this (it ends with a block reduction when J is updated).
template <typename coef>
__device__ inline void jacobi_core(const JacobiArgs &a, int i, int j, int k, bool valid)
{
    const coef *Kc = static_cast<const coef *>(a.Kc);
    double q = 0.0, dist = 0.0;
    bool bad = false;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    if (valid) {
        const long plane = long(nx) * ny, V = plane * nz, v = k * plane + long(j) * nx + i;
        double acc = a.b[v];
        if (a.w_in) {
            const int im = (i == 0) ? nx - 1 : i - 1, ip = (i == nx - 1) ? 0 : i + 1;
            const int jm = (j == 0) ? ny - 1 : j - 1, jp = (j == ny - 1) ? 0 : j + 1;
            const int cols[3] = {im, i, ip};
            const int rows[3] = {jm, j, jp};
            // Branch-free over the planes so that all loads can be in flight together: the plane
            // below is clamped at the bottom and its sum masked; the plane above needs no mask, its
            // coefficients are stored as zero in the top layer.
            const int planes[3] = {k > 0 ? k - 1 : 0, k, k < nz - 1 ? k + 1 : k};
            double part[3] = {0.0, 0.0, 0.0};
#pragma unroll
            for (int o = 0; o < 27; ++o) {
                if (o == 13) continue;
                const long u = planes[o / 9] * plane + long(rows[(o / 3) % 3]) * nx + cols[o % 3];
                const double K = (o > 13) ? double(Kc[(o - 14) * V + v]) : double(Kc[(12 - o) * V + u]);
                part[o / 9] += K * a.w_in[u];
            }
            acc += (k > 0 ? part[0] : 0.0) + part[1] + part[2];
        }
        if (a.w_out) a.w_out[v] = acc * a.E[v];
        if (a.J) jacobi_update(a, v, acc, q, dist, bad);
    }
    if (a.J) jacobi_block_max(a, q, dist, bad);
}

template <typename coef>
__device__ inline void jacobi_body(const JacobiArgs &a, int p, int k)
{
    const bool valid = p < a.nx * a.ny;
    const int j = valid ? p / a.nx : 0;
    jacobi_core<coef>(a, valid ? p - j * a.nx : 0, j, k, valid);
}

template <typename coef>
__global__ __launch_bounds__(kPlaneThreads) void jacobi_kernel(JacobiArgs a)
{
    jacobi_body<coef>(a, blockIdx.x * kPlaneThreads + threadIdx.x, blockIdx.y);
}

// The same sweep on a 1D grid whose blocks are dealt to the 8 XCDs (each with its own L2) in
// contiguous ranges: workgroups go round-robin over the XCDs in launch order, so block b runs on XCD
// b % 8; here that XCD takes the chunks [xcd * G, (xcd + 1) * G) of every plane, G = padded chunks / 8.
// A voxel's mirrored coefficients and iterates sit in the row above (mostly the same or the previous
// chunk) and in the plane below (the same chunk, G * 8 blocks earlier), so they are in that XCD's L2.
// Chunks beyond the plane are padding (no voxels).
template <typename coef>
__global__ __launch_bounds__(kPlaneThreads) void jacobi_kernel_grouped(JacobiArgs a, int group)
{
    const int b = blockIdx.x;
    const int xcd = b & 7, slot = b >> 3;
    const int k = slot / group;
    const int chunk = xcd * group + (slot - k * group);
    jacobi_body<coef>(a, chunk * kPlaneThreads + threadIdx.x, k);
}

// 2D tiles of kTileX x kTileY columns (a wavefront spans two rows of 32), dealt to the XCDs in
// contiguous ranges of tiles per plane as above: the row above a voxel is mostly in its own tile, so
// its iterates and mirrored coefficients come from this workgroup's recent reads.
constexpr int kTileX = 32, kTileY = kPlaneThreads / kTileX;
template <typename coef>
__global__ __launch_bounds__(kPlaneThreads) void jacobi_kernel_tiled(JacobiArgs a, int tiles_x, int group)
{
    const int b = blockIdx.x;
    const int xcd = b & 7, slot = b >> 3;
    const int k = slot / group;
    const int tile = xcd * group + (slot - k * group);
    const int ty = tile / tiles_x, tx = tile - ty * tiles_x;
    const int i = tx * kTileX + (threadIdx.x % kTileX);
    const int j = ty * kTileY + (threadIdx.x / kTileX);
    const bool valid = i < a.nx && j < a.ny;
    jacobi_core<coef>(a, valid ? i : 0, valid ? j : 0, k, valid);
}

// Column form: a thread takes H voxels (i, j, k0 .. k0 + H - 1) and marches up them, keeping the
// previous iterates of three planes in registers, so each voxel loads one new plane of nine iterates
// instead of 26 neighbours (the coefficient streams and the per-voxel sums are those of jacobi_core,
// in the same order).  Every column layer's columns are dealt to the XCDs in contiguous ranges of equal
// length (xcd_column).  H = 4 on grids that fill the chip; smaller grids take shorter columns
// (more threads), see jacobi_column_height.
constexpr int kJacCol = 4;
// Column layer kc of the columns p (p = j nx + i; p >= nx ny: no voxels).  The whole block must call
// this (it ends with a block reduction when J is updated).
template <typename coef, int H = kJacCol, bool Down = false>
__device__ inline void jacobi_column_body(const JacobiArgs &a, int p, int kc)
{
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const bool valid = p < nx * ny;
    const coef *Kc = static_cast<const coef *>(a.Kc);
    double q = 0.0, dist = 0.0;
    bool bad = false;
    if (valid) {
        const int j = p / nx, i = p - j * nx, k0 = kc * H;
        const int kfirst = Down ? (k0 + H - 1 < nz - 1 ? k0 + H - 1 : nz - 1) : k0;
        const long plane = long(nx) * ny, V = plane * nz;
        const int im = (i == 0) ? nx - 1 : i - 1, ip = (i == nx - 1) ? 0 : i + 1;
        const int jm = (j == 0) ? ny - 1 : j - 1, jp = (j == ny - 1) ? 0 : j + 1;
        long off[9];              // the 3 x 3 columns around (i, j), in the stencil's order
#pragma unroll
        for (int m = 0; m < 9; ++m)
            off[m] = long(m < 3 ? jm : (m < 6 ? j : jp)) * nx + (m % 3 == 0 ? im : (m % 3 == 1 ? i : ip));
        double Wm[9], W0[9], Wp[9];   // iterates of the planes k - 1 (clamped), k, k + 1 (clamped)
        if (a.w_in) {
            // the first voxel's plane and the one behind it in the walk (clamped at the grid's faces)
            const long kb = Down ? (kfirst < nz - 1 ? kfirst + 1 : kfirst) : (kfirst > 0 ? kfirst - 1 : 0);
#pragma unroll
            for (int m = 0; m < 9; ++m) {
                if constexpr (Down) Wp[m] = a.w_in[kb * plane + off[m]];
                else Wm[m] = a.w_in[kb * plane + off[m]];
                W0[m] = a.w_in[long(kfirst) * plane + off[m]];
            }
        }
#pragma unroll
        for (int t = 0; t < H; ++t) {
            const int k = Down ? kfirst - t : k0 + t;
            if (Down ? k < k0 : k >= nz) break;
            const long km = k > 0 ? k - 1 : 0, kp = k < nz - 1 ? k + 1 : k;
            const long v = k * plane + off[4];
            double acc = a.b[v];
            if (a.w_in) {
                // the plane ahead in the walk
#pragma unroll
                for (int m = 0; m < 9; ++m) {
                    if constexpr (Down) Wm[m] = a.w_in[km * plane + off[m]];
                    else Wp[m] = a.w_in[kp * plane + off[m]];
                }
                const long pls[3] = {km * plane, long(k) * plane, kp * plane};
                double part[3] = {0.0, 0.0, 0.0};
#pragma unroll
                for (int o = 0; o < 27; ++o) {
                    if (o == 13) continue;
                    const long u = pls[o / 9] + off[o % 9];
                    const double K = (o > 13) ? double(Kc[(o - 14) * V + v]) : double(Kc[(12 - o) * V + u]);
                    const double w = o < 9 ? Wm[o % 9] : (o < 18 ? W0[o % 9] : Wp[o % 9]);
                    part[o / 9] += K * w;
                }
                acc += (k > 0 ? part[0] : 0.0) + part[1] + part[2];
#pragma unroll
                for (int m = 0; m < 9; ++m) {
                    if constexpr (Down) { Wp[m] = W0[m]; W0[m] = Wm[m]; }
                    else { Wm[m] = W0[m]; W0[m] = Wp[m]; }
                }
            }
            if (a.w_out) a.w_out[v] = acc * a.E[v];
            if (a.J) jacobi_update(a, v, acc, q, dist, bad);
        }
    }
    if (a.J) jacobi_block_max(a, q, dist, bad);
}

// The column layers' columns are dealt to the XCDs in contiguous ranges of equal length: column q of XCD xcd's
// range among n (n: none).  Ranges of whole blocks left XCDs idle (65^2 columns: two of eight, 129^2: one for two
// thirds of the time).  us per sweep with those and with these: float64 coefficients 17^3 4.0 and 3.3, 33^3 5.3 and
// 5.1, 65^3 13.1 and 10.8, 97^3 27.4 and 26.5, 113^3 44.6 and 43.4, 129^3 65.3 and 65.3; float32 ones 65^3 9.2 and
// 7.9, 129^3 35.0 and 33.6.
__device__ inline int xcd_column(int n, int xcd, int q)
{
    const int cols = (n + 7) / 8;
    return q < cols ? min(xcd * cols + q, n) : n;
}
// Threads of a block of the column layout: those that leave the fewest lanes of an XCD's range idle, the
// more the better.
inline int jacobi_column_threads(int n)
{
    const int cols = (n + 7) / 8;
    int best = 256;
    for (int t : {192, 128})
        if ((cols + t - 1) / t * t < (cols + best - 1) / best * best) best = t;
    return best;
}

// reverse: the column layers in descending order (top first).  Consecutive sweeps alternate, so each
// starts where the previous one ended and finds its most recent planes still in the caches; the order
// of the blocks does not change any voxel's sum.
// alt_walk: odd column layers walk their voxels top down (the plane two neighbouring layers share is
// then read by both near their start or both near their end); each voxel's sum is unchanged.
template <typename coef, int H = kJacCol>
__global__ __launch_bounds__(kPlaneThreads) void jacobi_kernel_column(JacobiArgs a, int group, int reverse,
                                                                      int alt_walk)
{
    const int blk = blockIdx.x;
    const int xcd = blk & 7, slot = blk >> 3;
    const int kc = slot / group;
    const int kcol = reverse ? int(gridDim.x) / (8 * group) - 1 - kc : kc;
    const int p = xcd_column(a.nx * a.ny, xcd, (slot - kc * group) * int(blockDim.x) + int(threadIdx.x));
    if (alt_walk && (kcol & 1)) jacobi_column_body<coef, H, true>(a, p, kcol);
    else jacobi_column_body<coef, H, false>(a, p, kcol);
}

// Column height of the column form, from the number of workgroups that columns of 4 give: 4 for
// grids that fill the chip with them, 2 for mid-size grids, 1 for small ones.  Measured per float64
// sweep (H = 4 / 2 / 1): 129^3 (2178 workgroups of 4) 67.8 / 67.3 / 70.5 us, 65^3 (289) 13.8 / 13.3 /
// 14.1 us, 17^3 (10) 8.0 / 5.2 / 3.9 us.  Every height gives the same per-voxel sums.
inline int jacobi_column_height(int nx, int ny, int nz)
{
    const long blocks4 = (long(nx) * ny + kPlaneThreads - 1) / kPlaneThreads * ((nz + 3) / 4);
    return blocks4 >= 1024 ? 4 : (blocks4 >= 128 ? 2 : 1);
}

// Walk direction of the column layout (walk: 1 odd layers top down, 0 all bottom up, -1 by coefficient
// type): top-down odd layers pay with float coefficients in columns of 4 and not with float64 ones.
// Measured per sweep (bitwise the same iterates): float coefficients 129^3 38.0 -> 35.8 us,
// 129^2 x 193 55.2 -> 52.9 us, 65^3 (columns of 2) 9.24 against 9.30 us; float64 coefficients 129^3
// 67.4 -> 73.3 us (L2 fetches 389 against 384 MB), 65^3 13.5 -> 13.0 us.
inline bool jacobi_alt_walk(int walk, bool f32, int H) { return walk >= 0 ? walk != 0 : (f32 && H == 4); }

__device__ __forceinline__ double buffer_load(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff, double)
{
    typedef int int2v __attribute__((ext_vector_type(2)));
    const int2v x = __builtin_amdgcn_raw_buffer_load_b64(r, int(voff), int(soff), 0);
    return __hiloint2double(x.y, x.x);
}
__device__ __forceinline__ float buffer_load(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff, float)
{
    return __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, int(voff), int(soff), 0));
}

// Two sweeps in one launch: a workgroup puts out tx x ty x z voxels; a thread takes one voxel of these and
// the layer of voxels around them, computes its first sweep from the previous iterates, which the workgroup has
// brought to LDS, and, if it is one of those put out, its second from the first sweep's values in LDS, with
// the coefficients that it still holds.  Bitwise two sweeps of jacobi_core.
// What bounds a single sweep: on small grids the launch and one wait for memory (3.3 us), on larger ones its whole
// footprint, since an XCD's L2 keeps nothing from one launch to the next; two sweeps have both once.  Against that stand
// 1.5 to 3 times the loads of coefficients within an XCD (the tiles' borders).  us per sweep, single and so:
// 17^3 3.1 and 2.3, 33^3 4.9 and 3.3, 50^3 7.1 and 5.1, 65^3 10.6 and 9.8, 97^3 26.6 and 24.3, 113^3 43.4 and 37.4; but 129^3
// 65.3 and 65.9, and with float coefficients (half the footprint, the same loads) 33^3 4.3 and 3.2, 50^3 5.5 and 4.6, 56^3
// 6.4 and 6.1, 65^3 7.9 and 9.0.  (Walking a tile's planes with three of them in LDS: 11.5 us at 65^3, 72 at 129^3; the
// waits of its steps follow each other.)
template <typename coef>
__device__ inline void jacobi_pair_body(const JacobiArgs &a, const rt3d::JacobiTile &T, int block, double *lds)
{
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const unsigned plane = unsigned(nx) * unsigned(ny), V = plane * unsigned(nz);
    const int bz = block / (T.ntx * T.nty), bxy = block - bz * (T.ntx * T.nty), by = bxy / T.ntx, bx = bxy - by * T.ntx;
    const int x0 = bx * T.tx, y0 = by * T.ty, k0 = bz * T.z;
    const int cx = T.tx + 2, cy = T.ty + 2, cells = T.cells(), wx = T.tx + 4, wy = T.ty + 4, wcells = T.cells0();
    double *w0 = lds, *w1 = lds + wcells;
    const int tid = int(threadIdx.x), q = min(tid, cells - 1);
    const int lz = q / (cx * cy), r = q - lz * (cx * cy), ly = r / cx, lx = r - ly * cx;
    auto wrap = [](int x, int n) {          // x in [-n, 2n)
        x += x < 0 ? n : 0;
        return x - (x >= n ? n : 0);
    };
    const int gx = x0 + lx - 1, gy = y0 + ly - 1, k = k0 + lz - 1;
    const bool live = tid < cells && k >= 0 && k < nz;
    const bool inner = live && unsigned(lx - 1) < unsigned(T.tx) && unsigned(ly - 1) < unsigned(T.ty) &&
                       unsigned(lz - 1) < unsigned(T.z) && gx < nx && gy < ny;
    const int kc = min(max(k, 0), nz - 1);
    unsigned at[9];               // the nine columns around it, in its plane
#pragma unroll
    for (int m = 0; m < 9; ++m)
        at[m] = unsigned(kc) * plane + unsigned(wrap(wrap(gy, ny) + m / 3 - 1, ny) * nx + wrap(wrap(gx, nx) + m % 3 - 1, nx));
    const auto rsrc = [](const void *p, unsigned bytes) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, int(bytes), 0x00027000);
    };
    const __amdgpu_buffer_rsrc_t rK = rsrc(a.Kc, 13u * V * unsigned(sizeof(coef))), rb = rsrc(a.b, V * 8u), rE = rsrc(a.E, V * 8u);
    constexpr int U = rt3d::kPairLoads;
    double wr[U];
    if (a.w_in) {
        const __amdgpu_buffer_rsrc_t rw = rsrc(a.w_in, V * 8u);
#pragma unroll
        for (int t = 0; t < U; ++t) {
            const int e = min(tid + t * int(blockDim.x), wcells - 1);
            if (t * int(blockDim.x) >= wcells) break;
            const int sz = e / (wx * wy), s = e - sz * (wx * wy), sy = s / wx, sx = s - sy * wx;
            const int kk = min(max(k0 + sz - 2, 0), nz - 1);
            wr[t] = buffer_load(rw, (unsigned(kk) * plane + unsigned(wrap(y0 + sy - 2, ny) * nx + wrap(x0 + sx - 2, nx))) * 8u, 0, 0.0);
        }
    }
    coef K[26];
    const unsigned cs = unsigned(sizeof(coef)), down = k > 0 ? plane : 0u;
#pragma unroll
    for (int o = 0; o < 9; ++o) K[o] = buffer_load(rK, (at[o] - down) * cs, unsigned(12 - o) * V * cs, coef(0));
#pragma unroll
    for (int o = 9; o < 13; ++o) K[o] = buffer_load(rK, at[o - 9] * cs, unsigned(12 - o) * V * cs, coef(0));
#pragma unroll
    for (int o = 14; o < 27; ++o) K[o - 1] = buffer_load(rK, at[4] * cs, unsigned(o - 14) * V * cs, coef(0));
    const double b = buffer_load(rb, at[4] * 8u, 0, 0.0), e = buffer_load(rE, at[4] * 8u, 0, 0.0);
    // sum over the neighbours in jacobi_core's order, the planes beyond the grid's faces clamped as there
    auto stencil = [&](const double *w, int sx, int sxy) {
        double part[3] = {0.0, 0.0, 0.0};
        const int dz[3] = {k > 0 ? -sxy : 0, 0, k < nz - 1 ? sxy : 0};
#pragma unroll
        for (int z = 0; z < 3; ++z)
#pragma unroll
            for (int m = 0; m < 9; ++m) {
                const int o = 9 * z + m;
                if (o == 13) continue;
                part[z] = fma(double(K[o < 13 ? o : o - 1]), w[dz[z] + (m / 3 - 1) * sx + m % 3 - 1], part[z]);
            }
        return b + ((k > 0 ? part[0] : 0.0) + part[1] + part[2]);
    };
    double acc = b;
    if (a.w_in) {
#pragma unroll
        for (int t = 0; t < U; ++t)
            if (tid + t * int(blockDim.x) < wcells) w0[tid + t * int(blockDim.x)] = wr[t];
        __syncthreads();
        if (live) acc = stencil(w0 + ((lz + 1) * wy + ly + 1) * wx + lx + 1, wx, wx * wy);
    }
    if (live) w1[q] = acc * e;
    __syncthreads();
    double qmax = 0.0, dist = 0.0;
    bool bad = false;
    if (inner) {
        acc = stencil(w1 + q, cx, cx * cy);
        if (a.w_out) a.w_out[at[4]] = acc * e;
        if (a.J) jacobi_update(a, at[4], acc, qmax, dist, bad);
    }
    if (a.J) jacobi_block_max(a, qmax, dist, bad);
}

template <typename coef>
__global__ __launch_bounds__(rt3d::kPairThreads) void jacobi_kernel_pair(JacobiArgs a, rt3d::JacobiTile T)
{
    extern __shared__ double pair_lds[];
    // blocks go round-robin over the 8 XCDs: neighbouring tiles to one of them
    const int n = int(gridDim.x), per = n / 8, rest = n % 8, x = int(blockIdx.x) & 7, i = int(blockIdx.x) >> 3;
    jacobi_pair_body<coef>(a, T, x * per + min(x, rest) + i, pair_lds);
}

// Grids up to these numbers of voxels take two sweeps per launch: between the sizes above where it pays and where it
// does not.  On 30 grids that are no cubes (flat, tall, long, thin) the number of voxels decides as well: with float64 coefficients pairs
// won on all of them, 200 x 200 x 8 13.5 and 11.0 us per sweep, 8 x 8 x 500 11.9 and 3.9, 193 x 193 x 42 47.0 and 37.8, 512 x 300 x 10 42.1
// and 40.4, 1000 x 50 x 31 47.5 and 44.5, 60 x 60 x 400 44.4 and 35.3; with float ones they are even around the limit (40 x 200 x 24 9.1 and
// 9.6, 24 x 40 x 200 9.3 and 8.2, 129 x 129 x 20 10.9 and 10.9) and lose above (129 x 129 x 90 27.1 and 33.9, 1000 x 50 x 31 29.4 and 37.2) but
// for narrow towers (24 x 24 x 1500 25.8 and 21.6).
// (Its buffer offsets need 13 coefficients of all voxels to stay below 4 GB.)
inline bool jacobi_pair_pays(long V, bool f32) { return V <= (f32 ? 3L << 16 : 3L << 19); }

inline void launch_jacobi_pair(const JacobiArgs &a, const rt3d::JacobiTile &t, bool f32, hipStream_t stream)
{
    const dim3 grid(t.blocks()), blk(t.threads());
    const size_t smem = t.lds();
    if (f32) hipLaunchKernelGGL(jacobi_kernel_pair<float>, grid, blk, smem, stream, a, t);
    else hipLaunchKernelGGL(jacobi_kernel_pair<double>, grid, blk, smem, stream, a, t);
}

// Gauss-Seidel colour pass.  The voxels are coloured per axis so that no two 27-point neighbours share
// a colour: index i has colour i mod 2, except on a periodic axis of odd length, where the last index
// has colour 2 (its neighbours n-2 and 0 are odd and even); z (not periodic) always has two.  A pass
// updates the voxels of one colour (cx, cy, cz) in place: none of them reads another's value, and
// each reads the newest value of every neighbour.  Member q of colour c on an axis is 2q + c, or
// n - 1 for colour 2; cnt holds the members per axis.
__device__ inline int colour_member(int c, int q, int n) { return c == 2 ? n - 1 : 2 * q + c; }

template <typename coef>
__global__ __launch_bounds__(kPlaneThreads) void jacobi_kernel_colour(JacobiArgs a, int3 col, int3 cnt)
{
    const long t = long(blockIdx.x) * kPlaneThreads + threadIdx.x;
    const bool valid = t < long(cnt.x) * cnt.y * cnt.z;
    int i = 0, j = 0, k = 0;
    if (valid) {
        const long rest = t / cnt.x;
        i = colour_member(col.x, int(t - rest * cnt.x), a.nx);
        j = colour_member(col.y, int(rest % cnt.y), a.ny);
        k = colour_member(col.z, int(rest / cnt.y), a.nz);
    }
    jacobi_core<coef>(a, i, j, k, valid);
}

// Colours on an axis of length n (periodic or not) and the members of colour c.
inline int axis_colours(int n, bool periodic) { return periodic && (n % 2) ? 3 : 2; }
inline int colour_count(int c, int n, bool periodic)
{
    if (periodic && (n % 2)) return c == 2 ? 1 : (n - 1) / 2;
    return c == 0 ? (n + 1) / 2 : n / 2;
}

// One Jacobi sweep in the given grid layout: 0 one block per chunk of a plane, 1 the same padded to
// a multiple of 8 chunks per plane, 2 contiguous chunk ranges per XCD, 3 2D tiles, 4 columns.
// reverse: the column layout walks its column layers top first (see jacobi_kernel_column).
// height: column height of layout 4 (1, 2 or 4; 0: jacobi_column_height); walk: see jacobi_alt_walk.
inline void launch_jacobi_sweep(const JacobiArgs &a, int layout, bool f32, hipStream_t stream, bool reverse = false,
                                int height = 0, int walk = -1)
{
    const int chunks = (a.nx * a.ny + kPlaneThreads - 1) / kPlaneThreads;
    const int group = (chunks + 7) / 8;
    const dim3 blk(kPlaneThreads);
    if (layout == 4) {
        const int H = height > 0 ? height : jacobi_column_height(a.nx, a.ny, a.nz);
        const int nt = jacobi_column_threads(a.nx * a.ny), per_xcd = ((a.nx * a.ny + 7) / 8 + nt - 1) / nt;
        const dim3 grid(unsigned(8 * per_xcd) * unsigned((a.nz + H - 1) / H)), cblk(nt);
        const int rev = reverse ? 1 : 0, md = jacobi_alt_walk(walk, f32, H) ? 1 : 0;
        if (H == 1) {
            if (f32) hipLaunchKernelGGL((jacobi_kernel_column<float, 1>), grid, cblk, 0, stream, a, per_xcd, rev, md);
            else hipLaunchKernelGGL((jacobi_kernel_column<double, 1>), grid, cblk, 0, stream, a, per_xcd, rev, md);
        } else if (H == 2) {
            if (f32) hipLaunchKernelGGL((jacobi_kernel_column<float, 2>), grid, cblk, 0, stream, a, per_xcd, rev, md);
            else hipLaunchKernelGGL((jacobi_kernel_column<double, 2>), grid, cblk, 0, stream, a, per_xcd, rev, md);
        } else {
            if (f32) hipLaunchKernelGGL((jacobi_kernel_column<float, 4>), grid, cblk, 0, stream, a, per_xcd, rev, md);
            else hipLaunchKernelGGL((jacobi_kernel_column<double, 4>), grid, cblk, 0, stream, a, per_xcd, rev, md);
        }
    } else if (layout == 3) {
        const int tiles_x = (a.nx + kTileX - 1) / kTileX, tiles_y = (a.ny + kTileY - 1) / kTileY;
        const int tgroup = (tiles_x * tiles_y + 7) / 8;
        const dim3 grid(unsigned(8 * tgroup) * unsigned(a.nz));
        if (f32) hipLaunchKernelGGL(jacobi_kernel_tiled<float>, grid, blk, 0, stream, a, tiles_x, tgroup);
        else hipLaunchKernelGGL(jacobi_kernel_tiled<double>, grid, blk, 0, stream, a, tiles_x, tgroup);
    } else if (layout == 2) {
        const dim3 grid(unsigned(8 * group) * unsigned(a.nz));
        if (f32) hipLaunchKernelGGL(jacobi_kernel_grouped<float>, grid, blk, 0, stream, a, group);
        else hipLaunchKernelGGL(jacobi_kernel_grouped<double>, grid, blk, 0, stream, a, group);
    } else {
        const dim3 grid(layout == 1 ? unsigned(group * 8) : unsigned(chunks), a.nz);
        if (f32) hipLaunchKernelGGL(jacobi_kernel<float>, grid, blk, 0, stream, a);
        else hipLaunchKernelGGL(jacobi_kernel<double>, grid, blk, 0, stream, a);
    }
}

// ------------------------------------------------------------------------------------------------
// Ng acceleration: weighted dot products (fixed-order two-level reduction), the small normal
// equations solved on the device, and the combination.  The iterates live in a ring of R = order + 2
// vectors; with the newest at ring index m, iterate x_i (i = 0 newest) is entry (m - i) mod R.
// ------------------------------------------------------------------------------------------------

constexpr int kNgSums = 9;          // A00 A01 A02 A11 A12 A22 b0 b1 b2
constexpr int kNgBlocks = 512;      // blocks of the dot-product pass of one problem (fixes the order)
constexpr int kNgThreads = 256;
// layout of the Ng work buffer of one problem
constexpr int kNgSumOff = kNgBlocks * kNgSums;   // the 9 sums
constexpr int kNgCoefOff = kNgSumOff + kNgSums;  // c0..c3 (x_new = sum_i c_i x_i) and a valid flag
constexpr int kNgWork = kNgCoefOff + 5;

struct NgArgs {
    long V;
    int order;
    const double *hist;             // [order + 2][V]
    double *work;                   // [kNgWork]
    double *J;                      // receives the extrapolated iterate
    int unit_weights;               // 1: weights 1 instead of 1/x_0^2 (iterates that may vanish)
};

__device__ inline const double *ng_x(const NgArgs &a, int m, int i)
{
    const int R = a.order + 2;
    return a.hist + long((m - i + 4 * R) % R) * a.V;
}

// One block's share of the weighted dot products (weights 1/x_0^2, or 1).  Whole block.
__device__ inline void ng_dots_body(const NgArgs &a, int m, int blk)
{
    const double *x0 = ng_x(a, m, 0), *x1 = ng_x(a, m, 1);
    double acc[kNgSums];
#pragma unroll
    for (int q = 0; q < kNgSums; ++q) acc[q] = 0.0;
    for (long v = long(blk) * kNgThreads + threadIdx.x; v < a.V; v += long(kNgBlocks) * kNgThreads) {
        const double y0 = x0[v];
        const double w = a.unit_weights ? 1.0 : 1.0 / (y0 * y0);
        const double d0 = y0 - x1[v];
        double Q[3] = {0.0, 0.0, 0.0};
        for (int i = 1; i <= a.order; ++i) Q[i - 1] = d0 - (ng_x(a, m, i)[v] - ng_x(a, m, i + 1)[v]);
        acc[0] += w * Q[0] * Q[0];
        acc[1] += w * Q[0] * Q[1];
        acc[2] += w * Q[0] * Q[2];
        acc[3] += w * Q[1] * Q[1];
        acc[4] += w * Q[1] * Q[2];
        acc[5] += w * Q[2] * Q[2];
        acc[6] += w * d0 * Q[0];
        acc[7] += w * d0 * Q[1];
        acc[8] += w * d0 * Q[2];
    }
    __shared__ double red[kNgSums][kNgThreads];
#pragma unroll
    for (int q = 0; q < kNgSums; ++q) red[q][threadIdx.x] = acc[q];
    __syncthreads();
    for (int h = kNgThreads / 2; h > 0; h >>= 1) {
        if (threadIdx.x < h)
            for (int q = 0; q < kNgSums; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x < kNgSums) a.work[blk * kNgSums + threadIdx.x] = red[threadIdx.x][0];
}

// Sums the block partials in a fixed order (one block), then thread 0 solves the order x order
// normal equations by Gaussian elimination with partial pivoting.  A singular system or a
// non-finite solution clears the valid flag (the plain iterate is kept).
__device__ inline void ng_solve_body(const NgArgs &a)
{
    __shared__ double red[kNgSums][kNgThreads];
    for (int q = 0; q < kNgSums; ++q) {
        double s = 0.0;
        for (int b = threadIdx.x; b < kNgBlocks; b += kNgThreads) s += a.work[b * kNgSums + q];
        red[q][threadIdx.x] = s;
    }
    __syncthreads();
    for (int h = kNgThreads / 2; h > 0; h >>= 1) {
        if (threadIdx.x < h)
            for (int q = 0; q < kNgSums; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    double sums[kNgSums];
    for (int q = 0; q < kNgSums; ++q) {
        sums[q] = red[q][0];
        a.work[kNgSumOff + q] = sums[q];
    }
    const int n = a.order;
    double A[3][3] = {{sums[0], sums[1], sums[2]}, {sums[1], sums[3], sums[4]}, {sums[2], sums[4], sums[5]}};
    double b[3] = {sums[6], sums[7], sums[8]}, c[3] = {0.0, 0.0, 0.0};
    bool ok = true;
    for (int col = 0; col < n && ok; ++col) {
        int p = col;
        for (int r = col + 1; r < n; ++r) if (fabs(A[r][col]) > fabs(A[p][col])) p = r;
        if (!(fabs(A[p][col]) > 0.0)) { ok = false; break; }
        if (p != col) {
            for (int q = 0; q < n; ++q) { const double t = A[col][q]; A[col][q] = A[p][q]; A[p][q] = t; }
            const double t = b[col]; b[col] = b[p]; b[p] = t;
        }
        for (int r = col + 1; r < n; ++r) {
            const double f = A[r][col] / A[col][col];
            for (int q = col; q < n; ++q) A[r][q] -= f * A[col][q];
            b[r] -= f * b[col];
        }
    }
    for (int r = n - 1; r >= 0 && ok; --r) {
        double t = b[r];
        for (int q = r + 1; q < n; ++q) t -= A[r][q] * c[q];
        c[r] = t / A[r][r];
        if (!isfinite(c[r])) ok = false;
    }
    double sa = 0.0;
    for (int i = 0; i < n; ++i) sa += c[i];
    a.work[kNgCoefOff + 0] = 1.0 - sa;
    for (int i = 0; i < 3; ++i) a.work[kNgCoefOff + 1 + i] = c[i];
    a.work[kNgCoefOff + 4] = ok ? 1.0 : 0.0;
}

// J_v = c0 x_0 + sum_i c_i x_i (only when the solve succeeded)
__device__ inline void ng_combine_body(const NgArgs &a, int m, long v)
{
    const double *cf = a.work + kNgCoefOff;
    if (cf[4] == 0.0) return;
    double r = cf[0] * ng_x(a, m, 0)[v];
    for (int i = 1; i <= a.order; ++i) r += cf[i] * ng_x(a, m, i)[v];
    a.J[v] = r;
}

__global__ __launch_bounds__(kNgThreads) void ng_dots_kernel(NgArgs a, int m)
{
    ng_dots_body(a, m, blockIdx.x);
}

__global__ __launch_bounds__(kNgThreads) void ng_solve_kernel(NgArgs a)
{
    ng_solve_body(a);
}

__global__ __launch_bounds__(256) void ng_combine_kernel(NgArgs a, int m)
{
    const long v = long(blockIdx.x) * blockDim.x + threadIdx.x;
    if (v < a.V) ng_combine_body(a, m, v);
}

// ------------------------------------------------------------------------------------------------
// Anderson mixing of the outer iteration: windows of (input, output) pairs of the OS step in two rings
// of V-vectors, the input x of a pair replaced by the step's change f = g - x once its output g is there
// (the dot products read ten vectors then instead of eighteen); slot[0..k] are the ring entries of the window, oldest first.  The weighted dot products
// use the fixed two-level partition of the Ng kernels (bitwise reproducible).
// ------------------------------------------------------------------------------------------------

constexpr int kAaMaxDepth = 8;
constexpr int kAaSums = kAaMaxDepth * (kAaMaxDepth + 1) / 2 + kAaMaxDepth;   // A (upper) and b
constexpr int kAaBlocks = 512;
constexpr int kAaThreads = 256;
constexpr int kAaSumOff = kAaBlocks * kAaSums;
constexpr int kAaCoefOff = kAaSumOff + kAaSums;     // gamma_1..gamma_8 and a valid flag
constexpr int kAaWork = kAaCoefOff + kAaMaxDepth + 1;

struct AaArgs {
    long V;
    int k;                          // differences in the window (1..kAaMaxDepth)
    int slot[kAaMaxDepth + 1];      // ring entries of the window, oldest first
    const double *F, *G;            // rings [depth + 1][V] of changes (the newest: inputs) and outputs
    double *work;                   // [kAaWork]
    double *J;                      // receives the mixed input of the next step
};

// Index of the sum A_ij (i <= j < k) and of b_i in a block's partial sums.
__host__ __device__ constexpr int aa_a_index(int i, int j) { return j * (j + 1) / 2 + i; }
__host__ __device__ constexpr int aa_b_index(int i) { return kAaMaxDepth * (kAaMaxDepth + 1) / 2 + i; }

// The step's output J of voxel v joins the pair whose input is in the given slot
__device__ inline void aa_output_body(const AaArgs &a, int slot, long v)
{
    const long o = long(slot) * a.V + v;
    const double g = a.J[v];
    const_cast<double *>(a.F)[o] = g - a.F[o];
    const_cast<double *>(a.G)[o] = g;
}

__global__ __launch_bounds__(256) void aa_output_kernel(AaArgs a, int slot)
{
    const long v = long(blockIdx.x) * blockDim.x + threadIdx.x;
    if (v < a.V) aa_output_body(a, slot, v);
}

// The sums of x[0 .. N) over a wavefront, in the order of an xor tree from offs = 32 down: at each level a lane hands
// half of its sums to its partner and takes over the other half, so N sums cost about N exchanges, not 6 N.
// (Six exchanges for each of the 44 sums were most of the dot products' time: 65^3 17.8 and 7.3 us, a batch of 12 grids up
// to 97^3 189 and 105 us, with the changes f stored instead of the inputs.)
// On return x[0] is sum q where true is returned (six levels leave one sum per lane at most).
template <int N>
__device__ __forceinline__ bool wave_sums(double *x, int lane, int offs, int &q)
{
    if constexpr (N == 1) {
        for (; offs > 0; offs >>= 1) x[0] += __shfl_xor(x[0], offs);
        q = 0;
        return true;
    } else {
        constexpr int M = (N + 1) / 2;
        const bool hi = (lane & offs) != 0;
#pragma unroll
        for (int u = 0; u < M; ++u) {
            const double a = x[u], b = u + M < N ? x[u + M] : 0.0;
            x[u] = (hi ? b : a) + __shfl_xor(hi ? a : b, offs);
        }
        const bool held = wave_sums<M>(x, lane, offs >> 1, q);
        q += hi ? M : 0;
        return held && q < N;
    }
}

// One block's share of A_ij = sum_v w df_i df_j and b_i = sum_v w df_i f_k, w = 1/g_k^2, f = g - x,
// df_j = f_k - f_{k-j}; the sums of a thread, then of a wavefront (xor tree), then of the block's
// wavefronts in order.  Whole block; blk is the block's index among the kAaBlocks of the pass.
__device__ inline void aa_dots_body(const AaArgs &a, int blk)
{
    const int k = a.k;
    double acc[kAaSums];
#pragma unroll
    for (int q = 0; q < kAaSums; ++q) acc[q] = 0.0;
    const double *gk = a.G + long(a.slot[k]) * a.V, *fkp = a.F + long(a.slot[k]) * a.V;
    for (long v = long(blk) * kAaThreads + threadIdx.x; v < a.V; v += long(kAaBlocks) * kAaThreads) {
        const double g = gk[v];
        const double w = 1.0 / (g * g);
        const double fk = fkp[v];
        double df[kAaMaxDepth];
#pragma unroll
        for (int j = 1; j <= kAaMaxDepth; ++j) {
            if (j > k) break;
            const long o = long(a.slot[k - j]) * a.V + v;
            df[j - 1] = fk - a.F[o];
        }
#pragma unroll
        for (int j = 0; j < kAaMaxDepth; ++j) {
            if (j >= k) break;
#pragma unroll
            for (int i = 0; i <= j; ++i) acc[aa_a_index(i, j)] += w * df[i] * df[j];
            acc[aa_b_index(j)] += w * df[j] * fk;
        }
    }
    __shared__ double part[kAaThreads / 64][kAaSums];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    int q;
    const bool held = wave_sums<kAaSums>(acc, lane, 32, q);
    if (held) part[wid][q] = acc[0];
    __syncthreads();
    if (threadIdx.x < kAaSums) {
        double s = part[0][threadIdx.x];
        for (int w2 = 1; w2 < kAaThreads / 64; ++w2) s += part[w2][threadIdx.x];
        a.work[blk * kAaSums + threadIdx.x] = s;
    }
}

__global__ __launch_bounds__(kAaThreads) void aa_dots_kernel(AaArgs a) { aa_dots_body(a, blockIdx.x); }

// Sums the block partials in a fixed order (five runs of blocks, each in order, then the runs), then solves
// the k x k normal equations A gamma = b by Gaussian elimination with partial pivoting, a thread per entry; a
// singular system or a non-finite solution clears the valid flag (the output g_k is then kept as the next
// input).  Whole block.  us with one thread per sum over all blocks and one for the elimination, and so:
// 20 and 8 on average over the windows of a solve, 59 and 12 for a batch of 12 grids.
__device__ inline void aa_solve_body(const AaArgs &a)
{
    constexpr int R = kAaThreads / kAaSums, per = (kAaBlocks + R - 1) / R, U = 16;
    constexpr int N = kAaMaxDepth, W = N + 1;
    __shared__ double run[R][kAaSums];
    __shared__ double tot[kAaSums];
    __shared__ double A[N][W];          // column N: b
    const int tid = int(threadIdx.x);
    if (tid < R * kAaSums) {
        const int r = tid / kAaSums, q = tid - r * kAaSums, b1 = min(kAaBlocks, (r + 1) * per);
        double s = 0.0;
        for (int b = r * per; b < b1; b += U) {
            double x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = a.work[min(b + u, b1 - 1) * kAaSums + q];
#pragma unroll
            for (int u = 0; u < U; ++u) s += b + u < b1 ? x[u] : 0.0;
        }
        run[r][q] = s;
    }
    __syncthreads();
    if (tid < kAaSums) {
        double s = run[0][tid];
        for (int r = 1; r < R; ++r) s += run[r][tid];
        tot[tid] = s;
        a.work[kAaSumOff + tid] = s;
    }
    __syncthreads();
    const int n = a.k, i = tid / W, j = tid - i * W;      // this thread's entry
    const bool mine = i < n && (j < n || j == N);
    if (mine) A[i][j] = j == N ? tot[aa_b_index(i)] : i <= j ? tot[aa_a_index(i, j)] : tot[aa_a_index(j, i)];
    __syncthreads();
    bool ok = true;
    for (int c = 0; c < n; ++c) {
        int p = c;
        for (int r = c + 1; r < n; ++r)
            if (fabs(A[r][c]) > fabs(A[p][c])) p = r;
        if (!(fabs(A[p][c]) > 0.0)) {
            ok = false;
            break;
        }
        // rows c and p change places, then every row below loses its multiple of row c
        const int src = i == c ? p : i == p ? c : i;
        double x = 0.0;
        if (mine) {
            x = A[src][j];
            if (i > c && j >= c) x -= A[src][c] / A[p][c] * A[p][j];
        }
        __syncthreads();
        if (mine) A[i][j] = x;
        __syncthreads();
    }
    if (tid != 0) return;
    double g[N];
    for (int r = 0; r < N; ++r) g[r] = 0.0;
#pragma unroll
    for (int r = N - 1; r >= 0; --r) {
        if (r >= n || !ok) continue;
        double t = A[r][N];
#pragma unroll
        for (int q = r + 1; q < N; ++q)
            if (q < n) t -= A[r][q] * g[q];
        g[r] = t / A[r][r];
        if (!isfinite(g[r])) ok = false;
    }
#pragma unroll
    for (int q = 0; q < N; ++q) a.work[kAaCoefOff + q] = q < n ? g[q] : 0.0;
    a.work[kAaCoefOff + N] = ok ? 1.0 : 0.0;
}

__global__ __launch_bounds__(kAaThreads) void aa_solve_kernel(AaArgs a) { aa_solve_body(a); }

// J = g_k - sum_j gamma_j (g_k - g_{k-j}) when the solve succeeded, else g_k (voxel v).
__device__ inline void aa_combine_body(const AaArgs &a, long v)
{
    const double *cf = a.work + kAaCoefOff;
    const double gk = a.G[long(a.slot[a.k]) * a.V + v];
    double x = gk;
    if (cf[kAaMaxDepth] != 0.0) {
        // all loads before the sums
        double g[kAaMaxDepth];
#pragma unroll
        for (int j = 1; j <= kAaMaxDepth; ++j) g[j - 1] = a.G[long(a.slot[max(a.k - j, 0)]) * a.V + v];
#pragma unroll
        for (int j = 1; j <= kAaMaxDepth; ++j)
            if (j <= a.k) x -= cf[j - 1] * (gk - g[j - 1]);
    }
    a.J[v] = x;
}

__global__ __launch_bounds__(256) void aa_combine_kernel(AaArgs a)
{
    const long v = long(blockIdx.x) * blockDim.x + threadIdx.x;
    if (v < a.V) aa_combine_body(a, v);
}

// finiteness / range check of a device medium
__global__ void check_medium_kernel(long V, const double *chi, const double *eps, const double *B,
                                    int *flag)
{
    long v = long(blockIdx.x) * blockDim.x + threadIdx.x;
    if (v >= V) return;
    const double c = chi[v], e = eps[v], b = B[v];
    const bool ok = isfinite(c) && c > 0.0 && isfinite(e) && e > 0.0 && e <= 1.0 && isfinite(b);
    if (!ok) atomicOr(flag, 1);
}

// LTE-diffusion inner condition: dB/dtau per bottom column, (B_0 - B_1) / ((chi_0 + chi_1) / 2) from
// the bottom voxel and the one above it (the optical distance between their centres)
__global__ void diffusion_slope_kernel(int nxy, const double *chi, const double *B, double *slope)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < nxy) slope[c] = (B[c] - B[nxy + c]) / (0.5 * (chi[c] + chi[nxy + c]));
}

__global__ void check_finite_kernel(long V, const double *x, int *flag)
{
    long v = long(blockIdx.x) * blockDim.x + threadIdx.x;
    if (v >= V) return;
    if (!isfinite(x[v])) atomicOr(flag, 1);
}

}  // namespace
