// sweep_columns.h -- the formal solution's sweep for rows of up to kColumnMaxNx columns (kernels.h holds
// the sweep of wider rows).  Included by kernels.h.
//
// A thread stays in one column and lets the lines of an x-mirrored direction pair come through it.  It
// holds R neighbouring rows that move along y with the lines, so a row's {chi, 2S}, its deposits and both
// lines' intensities (P drifts to larger x, M to smaller) are registers.  Per segment:
//   an x-face ends it: P and M of all R rows go to the neighbour threads through a double-buffered LDS
//                      cell, one barrier;
//   a y-face:          the rows move down by one slot, the row of slot 0 leaves for the partial plane,
//                      the row ahead (loaded one face earlier) comes in;
//   the layer's end:   the R rows left are stored and those of the next layer loaded.
// The segment list is the same for all lines, so these are scalar branches, and a layer's partials are
// the rows that the band has touched, each stored once.
//
// What bounds it: on large grids the VALU (float64: about 31 instructions per row and segment, of which
// the exponential takes 19), on small ones the chain of segments of the
// shallowest directions, 450 + 165 R cycles each, hence R = 1 for those (make_column_plan).  The form
// that it replaces moved the lines through an LDS window of voxels instead, a gather, two LDS exchanges
// and a read-modify-write of the window per segment: the sweep took 2170 us at 129^3 x 256, 621 at 65^3 x 256, 70 at
// 17^3 x 64 and about 2240 in float32 at 129 x 129 x 193 x 256, against 1810 to 1880 (shortest launch 1750), 290, 30 and
// 1710 (1610) here.  Tried and slower: loading the next layer's rows ahead (more moves than latency saved),
// exchanging by DPP wave shifts instead of LDS, window deposits by LDS atomics.
#pragma once

namespace {

// Register moves written as assembly on tied operands: as plain assignments under a branch the compiler
// copies the whole state to merge the paths (30 moves per segment with 4 rows).
__device__ __forceinline__ void set_reg(double &d, double s) { asm volatile("v_mov_b64 %0, %1" : "+v"(d) : "v"(s)); }
__device__ __forceinline__ void set_reg(float &d, float s) { asm volatile("v_mov_b32 %0, %1" : "+v"(d) : "v"(s)); }
// x[r] = x[r + 1]
__device__ __forceinline__ void shift_rows(double (&)[1]) {}
__device__ __forceinline__ void shift_rows(float (&)[1]) {}
__device__ __forceinline__ void shift_rows(double (&x)[4])
{
    asm volatile("v_mov_b64 %0, %1\n\tv_mov_b64 %1, %2\n\tv_mov_b64 %2, %3"
                 : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]));
}
__device__ __forceinline__ void shift_rows(float (&x)[4])
{
    asm volatile("v_mov_b32 %0, %1\n\tv_mov_b32 %1, %2\n\tv_mov_b32 %2, %3"
                 : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]));
}
// The rows move on from slot r + 1 to slot r: before[r] = before[r + 1] + now[r + 1] (slot 3 is the first
// a row meets), now[r] = 0.
__device__ __forceinline__ void shift_sums(double (&)[1], double (&now)[1]) { asm volatile("v_mov_b64 %0, 0" : "+v"(now[0])); }
__device__ __forceinline__ void shift_sums(float (&)[1], float (&now)[1]) { asm volatile("v_mov_b32 %0, 0" : "+v"(now[0])); }
__device__ __forceinline__ void shift_sums(double (&before)[4], double (&now)[4])
{
    asm volatile("v_add_f64 %0, %1, %5\n\tv_add_f64 %1, %2, %6\n\tv_mov_b64 %2, %7\n\t"
                 "v_mov_b64 %4, 0\n\tv_mov_b64 %5, 0\n\tv_mov_b64 %6, 0\n\tv_mov_b64 %7, 0"
                 : "+v"(before[0]), "+v"(before[1]), "+v"(before[2]), "+v"(before[3]), "+v"(now[0]), "+v"(now[1]),
                   "+v"(now[2]), "+v"(now[3]));
}
__device__ __forceinline__ void shift_sums(float (&before)[4], float (&now)[4])
{
    asm volatile("v_add_f32 %0, %1, %5\n\tv_add_f32 %1, %2, %6\n\tv_mov_b32 %2, %7\n\t"
                 "v_mov_b32 %4, 0\n\tv_mov_b32 %5, 0\n\tv_mov_b32 %6, 0\n\tv_mov_b32 %7, 0"
                 : "+v"(before[0]), "+v"(before[1]), "+v"(before[2]), "+v"(before[3]), "+v"(now[0]), "+v"(now[1]),
                   "+v"(now[2]), "+v"(now[3]));
}

__device__ __forceinline__ void buffer_store(double v, __amdgpu_buffer_rsrc_t r, unsigned off)
{
    typedef int int2v __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(int2v{__double2loint(v), __double2hiint(v)}, r, int(off), 0, 0);
}
__device__ __forceinline__ void buffer_store(float v, __amdgpu_buffer_rsrc_t r, unsigned off)
{
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(v), r, int(off), 0, 0);
}

// A copy whose words are known to be the same in every lane
template <typename T> __device__ __forceinline__ T uniform_copy(const T &v)
{
    static_assert(sizeof(T) % 4 == 0);
    int w[sizeof(T) / 4];
    __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
    for (unsigned i = 0; i < sizeof(T) / 4; ++i) w[i] = __builtin_amdgcn_readfirstlane(w[i]);
    T r;
    __builtin_memcpy(&r, w, sizeof(T));
    return r;
}

// A part of a sweep: n layers from k_first on in sweep order, of pairs q0 .. whose lines have left their intensities in state
// ([pair - q0][P, M][line row][column], where the next segment starts) unless first, and leave them there.  The layers'
// blocks hold only these layers.
struct LayerRange {
    int k_first, n, q0, n_pair, first;
    const rt3d::LayerBlock *blocks;
    const int2 *start;            // per (layer, pair), as blocks: the layer's first segment in the list, its row offset modulo ny
    double *state;
};

template <typename real, int R, bool PARTIAL, bool LAYERS>
__device__ __forceinline__ void column_sweep_run(const SweepArgs &a, const WorkItem &it, const rt3d::PairInfo &pi,
                                                 real *edge, const double *xtab, const LayerRange &lr)
{
    using real2 = typename Vec2<real>::type;
    const unsigned nx = a.nx, ny = a.ny, plane = nx * ny;
    const int lane = threadIdx.x & 63;
    const int nq = it.rows * int(nx);
    const bool active = int(threadIdx.x) < nq;
    const int q = active ? int(threadIdx.x) : nq - 1;
    const int g = q / int(nx), c = q - g * int(nx);
    const int j0 = (it.band + g) * R;
    const int rows = PARTIAL ? min(R, int(ny) - j0) : R;
    const int q_lo = c == 0 ? q + int(nx) - 1 : q - 1, q_hi = c == int(nx) - 1 ? q - (int(nx) - 1) : q + 1;
    // own cell (lanes beyond the lines have one of their own), and the neighbour columns'
    real *own = edge + int(threadIdx.x) * column_edge<real>(R);
    const real *from_lo = edge + q_lo * column_edge<real>(R), *from_hi = edge + q_hi * column_edge<real>(R) + R;
    const bool yup = pi.ysgn > 0;
    const unsigned step = yup ? nx : 0u - nx, corr = yup ? 0u - plane : plane;    // next row, and its wrap
    auto fwd = [&](unsigned x) { return min(x + step, x + step + corr); };
    auto back = [&](unsigned x) { return min(x - step, x - step - corr); };
    // slot r carries the lines of row j0 + r (lines drifting up) or j0 + rows - 1 - r (down), so that the
    // rows move from slot r + 1 to slot r; rown: element offset in a plane of the row ahead of slot R - 1
    unsigned rown = unsigned((yup ? j0 + R + pi.row0 : j0 + rows - 1 - R + pi.row0 + R * int(ny)) % int(ny)) * nx;
    const unsigned cb = unsigned(c) * unsigned(sizeof(real2));
    const int dk = pi.down ? -1 : 1;
    const char *csk = reinterpret_cast<const char *>(static_cast<const real2 *>(a.cs) +
                                                     long(LAYERS ? lr.k_first : pi.down ? a.nz - 1 : 0) * plane);
    const long pstep = long(dk) * plane * long(sizeof(real2));
    real chi[R], S2[R], Pi[R], Mi[R];
    // deposits of the row that a slot is in: its own line's, and those of the slots that were there before
    real now[R], before[R];
    real2 vn;                       // the next row's voxel, in flight
    auto load_one = [&](unsigned row) {
        return *reinterpret_cast<const real2 *>(csk + (row * unsigned(sizeof(real2)) + cb));
    };
    auto load_layer = [&]() {
        real2 vl[R];
        unsigned x = rown;
#pragma unroll
        for (int r = R - 1; r >= 0; --r) {
            x = back(x);
            vl[r] = load_one(x);
        }
        vn = load_one(rown);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            chi[r] = vl[r].x;
            S2[r] = vl[r].y + vl[r].y;
        }
    };
    // the lines' place in the state; slots beyond the band's last row have none
    auto line_state = [&](int r) {
        const int row = yup ? j0 + r : j0 + rows - 1 - r;
        return lr.state + long(it.pair - lr.q0) * 2 * plane + long(min(max(row, 0), int(ny) - 1)) * nx + c;
    };
    if (LAYERS && !lr.first) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            Pi[r] = real(line_state(r)[0]);
            Mi[r] = real(line_state(r)[plane]);
        }
    } else {
        unsigned x = rown;
#pragma unroll
        for (int r = R - 1; r >= 0; --r) {
            x = back(x);
            double I = a.I_top;
            if (!pi.down) I = a.Ibot ? a.Ibot[x + c] + (a.Islope ? pi.mu * a.Islope[x + c] : 0.0) : 0.0;
            Pi[r] = Mi[r] = real(I);
            asm volatile("" : "+v"(Pi[r]), "+v"(Mi[r]));
        }
    }
    // descriptors: lane l of a wave holds segment 64 b + l of the block b in use
    const int4 *sg = reinterpret_cast<const int4 *>(a.cseg + pi.c_off);
    const int nseg = pi.n_seg;
    auto fetch = [&](int blk) { return sg[min(blk * 64 + lane, nseg - 1)]; };
    int4 dcur = fetch(0);
    auto settle = [](int4 &d) { asm volatile("" : "+v"(d.x), "+v"(d.y), "+v"(d.z), "+v"(d.w)); };
    settle(dcur);

    // partial planes: the pair's layers follow each other in sweep order, each with the rows it touches,
    // the band's rows walked in the direction the lines drift
    real *P = static_cast<real *>(a.P) + pi.p_off + it.band * pi.band_stride;
    const unsigned pstep_row = step * unsigned(sizeof(real));
    int cover = pi.cover0, cover_next = 0;
    unsigned pbase = (unsigned(g) * unsigned(pi.band_stride) + unsigned(c)) * unsigned(sizeof(real));   // this layer's block
    unsigned pw = pbase + (yup ? 0u : unsigned(cover - 1 - (R - rows)) * nx * unsigned(sizeof(real)));
    // stores outside the band's lines are dropped by the buffer's bounds check (no branch on the lane)
    const unsigned dead = active ? 0u : ~7u;
    const __amdgpu_buffer_rsrc_t prsrc = __builtin_amdgcn_make_buffer_rsrc(
        P, 0, int(unsigned(it.rows) * unsigned(pi.band_stride) * unsigned(sizeof(real))), 0x00027000);
    auto store_row = [&](real v, unsigned drop) { buffer_store(v, prsrc, pw | drop); pw += pstep_row; };
    bool moved = false;
    int buf = 0, s = 0;
    for (int layer = 0; layer < (LAYERS ? lr.n : a.nz); ++layer) {
        load_layer();
#pragma unroll
        for (int r = 0; r < R; ++r) now[r] = before[r] = real(0);
        int flags;
        while (true) {
            const int iw = s & 63;
            const real len = real(__hiloint2double(__builtin_amdgcn_readlane(dcur.y, iw), __builtin_amdgcn_readlane(dcur.x, iw)));
            flags = __builtin_amdgcn_readlane(dcur.z, iw);
            real em1[R], dt[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                dt[r] = chi[r] * len;
                em1[r] = expm1_sweep(-dt[r], xtab);
            }
            if (moved) {
                __syncthreads();
#pragma unroll
                for (int r = 0; r < R; ++r) Pi[r] = from_lo[buf + r];
#pragma unroll
                for (int r = 0; r < R; ++r) Mi[r] = from_hi[buf + r];
                buf = 2 * R - buf;
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                // S2 = 2 S; the two lines' deposits are D = S2 dtau - (uP + uM)(e^-dtau - 1), u = I - S
                const real uP = fma(S2[r], real(-0.5), Pi[r]), uM = fma(S2[r], real(-0.5), Mi[r]);
                Pi[r] = fma(uP, em1[r], Pi[r]);
                Mi[r] = fma(uM, em1[r], Mi[r]);
                now[r] = fma(-(uP + uM), em1[r], fma(S2[r], dt[r], now[r]));
            }
            moved = (flags & rt3d::kNextColumn) != 0;
            if (moved) {
#pragma unroll
                for (int r = 0; r < R; ++r) own[buf + r] = Pi[r];
#pragma unroll
                for (int r = 0; r < R; ++r) own[buf + R + r] = Mi[r];
            }
            const int cover_seg = __builtin_amdgcn_readlane(dcur.w, iw);
            ++s;
            if (iw == 63) {
                dcur = fetch(s >> 6);
                settle(dcur);
            }
            if (flags & rt3d::kLayerEnd) {
                cover_next = cover_seg;
                break;
            }
            if (flags & rt3d::kNextRow) {
                // a y-face: the row of slot 0 is complete, every slot moves on by a row
                store_row(before[0] + now[0], dead);
                shift_sums(before, now);
                shift_rows(chi);
                shift_rows(S2);
                if constexpr (PARTIAL) {
                    // a row entering the band from slots beyond its last row starts from zero
#pragma unroll
                    for (int r = 0; r + 1 < R; ++r) before[r] = r + 1 == rows ? real(0) : before[r];
                }
                set_reg(chi[R - 1], vn.x);
                set_reg(S2[R - 1], vn.y + vn.y);
                rown = fwd(rown);
                vn = load_one(rown);
            }
        }
        // the layer's remaining rows, then the next layer
#pragma unroll
        for (int r = 0; r < R; ++r) store_row(before[r] + now[r], PARTIAL && r >= rows ? ~7u : dead);
        if (flags & rt3d::kNextRow) rown = fwd(rown);
        pbase += unsigned(cover) * nx * unsigned(sizeof(real));
        cover = cover_next;
        pw = pbase + (yup ? 0u : unsigned(cover - 1 - (R - rows)) * nx * unsigned(sizeof(real)));
        csk += pstep;
    }
    if constexpr (LAYERS) {
        if (moved) {
            __syncthreads();
#pragma unroll
            for (int r = 0; r < R; ++r) Pi[r] = from_lo[buf + r];
#pragma unroll
            for (int r = 0; r < R; ++r) Mi[r] = from_hi[buf + r];
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (!active || (PARTIAL && r >= rows)) continue;
            line_state(r)[0] = double(Pi[r]);
            line_state(r)[plane] = double(Mi[r]);
        }
        return;
    }
    if (!pi.down && a.Iem && active) {
        const int sa = pi.sa_last;
        // the last segment's column is c: the lines of A entered the top at column c - sa, of B at c + sa
        const int cA = c - sa < 0 ? c - sa + int(nx) : c - sa, cB = c + sa >= int(nx) ? c + sa - int(nx) : c + sa;
        const long eA = long(pi.dA - a.n_down) * plane + cA, eB = long(pi.dB - a.n_down) * plane + cB;
        const long eP = pi.xsgn > 0 ? eA : eB, eM = pi.xsgn > 0 ? eB : eA;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (PARTIAL && r >= rows) continue;
            const long row = long(yup ? j0 + r : j0 + rows - 1 - r) * nx;
            a.Iem[eP + row] = (a.Iem_base ? a.Iem_base[eP + row] : 0.0) + double(Pi[r]);
            a.Iem[eM + row] = (a.Iem_base ? a.Iem_base[eM + row] : 0.0) + double(Mi[r]);
        }
    }
}

template <typename real, int R, bool LAYERS>
__device__ __forceinline__ void column_sweep_rows(const SweepArgs &a, const WorkItem &it, const rt3d::PairInfo &pi,
                                                  real *edge, const double *xtab, const LayerRange &lr)
{
    const int w0 = __builtin_amdgcn_readfirstlane(int(threadIdx.x) & ~63);
    if (w0 >= it.rows * a.nx) return;      // a wave without lines
    // bands of this wave that reach beyond the grid's last row
    const int last = min(w0 + 63, it.rows * a.nx - 1) / a.nx;
    if ((it.band + last + 1) * R > a.ny) column_sweep_run<real, R, true, LAYERS>(a, it, pi, edge, xtab, lr);
    else column_sweep_run<real, R, false, LAYERS>(a, it, pi, edge, xtab, lr);
}

template <typename real, bool LAYERS = false>
__device__ __forceinline__ void column_sweep_body(const SweepArgs &a, const WorkItem &it, unsigned char *smem_raw,
                                                  const LayerRange &lr = LayerRange{})
{
    rt3d::PairInfo pi = uniform_copy(a.pairs[it.pair]);
    if constexpr (LAYERS) {
        // the pair as if the range's layers were all
        const long at = long(lr.k_first) * lr.n_pair + it.pair;
        const rt3d::LayerBlock lb = uniform_copy(lr.blocks[at]);
        const int2 start = uniform_copy(lr.start[at]);
        pi.n_seg -= start.x - pi.c_off;
        pi.c_off = start.x;
        pi.row0 = start.y;
        pi.cover0 = lb.span + (pi.split ? 1 : rt3d::kColumnRows);
        pi.p_off = lb.off;
        pi.band_stride = long(lb.stride) * a.nx;
    }
    __shared__ double xtab[kExpTab];
    if (std::is_same<real, double>::value && threadIdx.x < kExpTab) xtab[threadIdx.x] = a.xtab[threadIdx.x];
    __syncthreads();
    real *edge = reinterpret_cast<real *>(smem_raw);
    if (pi.split) column_sweep_rows<real, 1, LAYERS>(a, it, pi, edge, xtab, lr);
    else column_sweep_rows<real, rt3d::kColumnRows, LAYERS>(a, it, pi, edge, xtab, lr);
}

template <typename real>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4))) void column_sweep_kernel(SweepArgs a)
{
    extern __shared__ unsigned char smem_raw[];
    column_sweep_body<real>(a, uniform_copy(a.items[blockIdx.x]), smem_raw);
}

template <typename real>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4))) void column_sweep_layers_kernel(SweepArgs a, LayerRange lr)
{
    extern __shared__ unsigned char smem_raw[];
    column_sweep_body<real, true>(a, uniform_copy(a.items[blockIdx.x]), smem_raw, lr);
}

}  // namespace
