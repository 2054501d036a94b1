// noalloc.hip -- the formal solution for callers that cannot allocate device memory (code under HIP
// graph capture, tight serving loops, harnesses that forbid hipMalloc).
//
// rt3d_formal_solution_noalloc computes what rt3d_formal_solution computes (same plan, kernels and
// summation order, so bitwise the same J_fs for the same grid and sweep shape), with no context: the
// caller passes chi, S, the bottom-plane light and the output on the device, and everything else the
// kernels need -- the packed {chi, S} field, the exponential's table, the plan's tables and the partial
// planes of the direction pairs -- lives in one file-scope device array of kScratchBytes.  When the
// partial planes of all pairs do not fit beside the rest, the sweep goes in parts and the angle sum is carried
// from part to part in J_fs in the order of a single pass.  A part is some layers of all downward (then all upward)
// pairs, whose lines leave their intensities in the array from part to part: as many lines are under way as in a
// single pass, and a layer's planes are small.  In the window form (rows of more than 512 columns) a part is some pairs.
// us per call, in parts of pairs and so: 65^3 x 256 3353 and 1765, 129^3 x 64 6600 and 1349, 129^3 x 256 31055 and 7015 (of which
// the plan, made on the host in every call, was about 3000, 700 and 6000 and is half of that now).
//
// The array is a host-side stand-in in host code: the kernels get its device address, taken once per
// device with hipGetSymbolAddress while that device is current, never the array's name.  Every call on
// a device shares that device's array, so calls that overlap on one device (other streams or host
// threads) race; each call returns only after its work on the stream has finished.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/rt3d.h"
#include "context.h"
#include "geometry.h"
#include "kernels.h"

using namespace rt3d_host;

namespace {

constexpr size_t kScratchBytes = size_t(128) << 20;   // 128 MiB per device
constexpr int kMaxDevices = 64;

__device__ __align__(256) unsigned char scratch[kScratchBytes];

std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices] = {};

// failures are reported like a failed context creation: rt3d_last_error(NULL) of the calling thread
int noalloc_fail(int code, const std::string &msg)
{
    set_thread_error(msg);
    return code;
}

// The device address of this device's scratch array (looked up once per device, with it current).
int scratch_address(void **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return noalloc_fail(RT3D_ERR_HIP, std::string("hipGetDevice: ") + hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return noalloc_fail(RT3D_ERR_ARG, "device index out of range");
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return noalloc_fail(RT3D_ERR_HIP, std::string("hipGetSymbolAddress: ") + hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return RT3D_OK;
}

size_t align256(size_t x) { return (x + 255) / 256 * 256; }

// Packs {chi, S} per voxel as the context's source kernel does for a given S.
__global__ __launch_bounds__(kPlaneThreads) void pack_kernel(long V, const double *chi, const double *S, double2 *cs)
{
    const long v = long(blockIdx.x) * kPlaneThreads + threadIdx.x;
    if (v < V) cs[v] = make_double2(chi[v], S[v]);
}

template <typename T>
int upload(unsigned char *dst, const std::vector<T> &h, hipStream_t st)
{
    if (h.empty()) return RT3D_OK;
    hipError_t e = hipMemcpyAsync(dst, h.data(), h.size() * sizeof(T), hipMemcpyHostToDevice, st);
    if (e != hipSuccess) return noalloc_fail(RT3D_ERR_HIP, std::string("hipMemcpyAsync: ") + hipGetErrorString(e));
    return RT3D_OK;
}

}  // namespace

extern "C" {

int rt3d_formal_solution_noalloc(const rt3d_grid_desc *g, const double *chi, const double *S, const double *I_bot,
                                 double *J_fs, void *hip_stream)
{
    set_thread_error(std::string());
    std::string msg;
    if (validate_desc(g, msg) != RT3D_OK) return noalloc_fail(RT3D_ERR_ARG, msg);
    if (g->bottom_bc == 2) return noalloc_fail(RT3D_ERR_ARG, "the LTE-diffusion inner condition needs a context");
    if (!chi || !S || !J_fs) return noalloc_fail(RT3D_ERR_ARG, "chi, S and J_fs must be device pointers");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    rt3d::AngleSet A;
    if (!rt3d::make_angle_set(g->n_theta, g->n_phi, A)) return noalloc_fail(RT3D_ERR_ARG, "bad angle set");
    rt3d::SweepPlan plan;
    if (!build_plan(*g, A, 0, plan, msg)) return noalloc_fail(RT3D_ERR_ARG, msg);
    const int nx = g->nx, ny = g->ny, nz = g->nz;
    const long V = long(nx) * ny * nz;

    // workspace layout: exponential table, {chi, S}, pair tables, segments, layer blocks and starts, work items, the
    // carried sums and intensities, then the partial planes of one part
    std::vector<double> tab(kExpTabSize);
    exp_table(tab.data());
    // the reduction's sum of a chunk of pairs that a part leaves unfinished
    const int chunk = reduce_chunk_pairs(V, plan.n_pair);
    const size_t carry_bytes = chunk < plan.n_pair ? align256(size_t(V) * sizeof(double)) : 0;
    const size_t start_bytes = align256(plan.blocks.size() * sizeof(int2));
    size_t fixed = 0;
    auto measure = [&]() {
        if (!plan.columns) plan.cseg.clear();          // (not read by the window form)
        fixed = align256(tab.size() * sizeof(double)) + align256(size_t(V) * sizeof(double2)) +
                align256(plan.pairs.size() * sizeof(rt3d::PairInfo)) +
                align256(plan.player.size() * sizeof(rt3d::PairLayer)) +
                align256(plan.pseg.size() * sizeof(rt3d::PairSeg)) +
                align256(plan.cseg.size() * sizeof(rt3d::ColumnSeg)) +
                align256(plan.blocks.size() * sizeof(rt3d::LayerBlock)) + (plan.columns ? start_bytes : 0) +
                align256(plan.items.size() * sizeof(rt3d::WorkItem)) + carry_bytes;
        return fixed < kScratchBytes ? (kScratchBytes - fixed) / sizeof(double) : 0;
    };
    std::vector<rt3d::SweepPart> parts;
    size_t room = measure();
    if (int64_t(room) >= plan.p_elems) {
        parts.push_back(rt3d::SweepPart{0, plan.n_pair, 0, nz});
    } else if (plan.columns) {
        // the launches hold half of the pairs; where a pair's planes of one layer do not fit, no pair is split
        for (int t = 0; t < 2 && parts.empty(); ++t) {
            rt3d::make_column_plan(A, kSweepShapes[0].threads, kSweepShapes[0].lines,
                                   t == 0 ? 0.5 * rt3d::column_load(nx, ny, nz, A) : 1e30, plan);
            room = measure();
            parts = rt3d::layer_parts(plan, int64_t(room));
        }
        if (parts.empty() && room > 0) {
            // few layers of very many rows, near the limit: only the window form's planes fit
            if (!build_plan(*g, A, 0, plan, msg, 0.0, 2)) return noalloc_fail(RT3D_ERR_ARG, msg);
            room = measure();
        }
    }
    if (parts.empty() && room > 0) parts = rt3d::pair_parts(plan, int64_t(room));
    if (room == 0)
        return noalloc_fail(RT3D_ERR_ARG, "grid too large for the allocation-free formal solution: its tables need " +
                                              std::to_string(fixed) + " of " + std::to_string(kScratchBytes) +
                                              " workspace bytes");
    if (parts.empty())
        return noalloc_fail(RT3D_ERR_ARG, "grid too large for the allocation-free formal solution: the partial "
                                          "planes of one direction pair exceed its workspace");
    std::vector<int2> start;
    if (plan.columns)
        for (const rt3d::LayerStart &ls : rt3d::layer_starts(plan)) start.push_back(make_int2(ls.seg, ls.row));
    // the partial planes of every part from the start of the buffer, and the work items of its pairs in the plan's dispatch
    // order (parts of the same pairs share them)
    std::vector<rt3d::WorkItem> items;
    for (size_t r = 0; r < parts.size(); ++r) {
        rt3d::SweepPart &part = parts[r];
        const bool same = r > 0 && parts[r - 1].q0 == part.q0;
        part.item0 = same ? parts[r - 1].item0 : int(items.size());
        if (!same)
            for (const rt3d::WorkItem &it : plan.items)
                if (it.pair >= part.q0 && it.pair < part.q1) items.push_back(it);
        part.n_items = same ? parts[r - 1].n_items : int(items.size()) - part.item0;
        if (rt3d::lay_out(plan, part) + rt3d::line_elems(plan, part) > int64_t(room))
            return noalloc_fail(RT3D_ERR_ARG, "grid too large for the allocation-free formal solution");
    }

    void *base = nullptr;
    int rc = scratch_address(&base);
    if (rc) return rc;
    unsigned char *p = static_cast<unsigned char *>(base);
    unsigned char *d_tab = p;        p += align256(tab.size() * sizeof(double));
    unsigned char *d_cs = p;         p += align256(size_t(V) * sizeof(double2));
    unsigned char *d_pairs = p;      p += align256(plan.pairs.size() * sizeof(rt3d::PairInfo));
    unsigned char *d_player = p;     p += align256(plan.player.size() * sizeof(rt3d::PairLayer));
    unsigned char *d_pseg = p;       p += align256(plan.pseg.size() * sizeof(rt3d::PairSeg));
    unsigned char *d_cseg = p;       p += align256(plan.cseg.size() * sizeof(rt3d::ColumnSeg));
    unsigned char *d_blocks = p;     p += align256(plan.blocks.size() * sizeof(rt3d::LayerBlock));
    unsigned char *d_start = p;      p += plan.columns ? start_bytes : 0;
    unsigned char *d_items = p;      p += align256(plan.items.size() * sizeof(rt3d::WorkItem));
    double *d_carry = reinterpret_cast<double *>(p);   p += carry_bytes;
    double *d_P = reinterpret_cast<double *>(p);       // room elements; a part's line intensities at their end
    // from here on an early return first drains the stream: the copies read this call's host tables
    auto drain_fail = [&](int code, const std::string &m) {
        hipStreamSynchronize(st);
        return noalloc_fail(code, m);
    };
    if ((rc = upload(d_tab, tab, st)) || (rc = upload(d_pairs, plan.pairs, st)) ||
        (rc = upload(d_player, plan.player, st)) || (rc = upload(d_pseg, plan.pseg, st)) ||
        (rc = upload(d_cseg, plan.cseg, st)) || (rc = upload(d_blocks, plan.blocks, st)) ||
        (rc = upload(d_start, start, st)) || (rc = upload(d_items, items, st)))
        return drain_fail(rc, thread_error());
    hipLaunchKernelGGL(pack_kernel, dim3(unsigned((V + kPlaneThreads - 1) / kPlaneThreads)), dim3(kPlaneThreads), 0,
                       st, V, chi, S, reinterpret_cast<double2 *>(d_cs));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return drain_fail(RT3D_ERR_HIP, std::string("pack_kernel: ") + hipGetErrorString(e));

    SweepArgs sa{};
    sa.nx = nx; sa.ny = ny; sa.nz = nz;
    sa.n_down = A.n_dir / 2;
    sa.pseg = reinterpret_cast<const rt3d::PairSeg *>(d_pseg);
    sa.player = reinterpret_cast<const rt3d::PairLayer *>(d_player);
    sa.cseg = reinterpret_cast<const rt3d::ColumnSeg *>(d_cseg);
    sa.pairs = reinterpret_cast<const rt3d::PairInfo *>(d_pairs);
    sa.cs = d_cs;
    sa.Ibot = g->bottom_bc == 1 ? nullptr : I_bot;
    sa.Islope = nullptr;
    sa.I_top = g->I_top;
    sa.P = d_P;
    sa.Iem = nullptr;
    sa.Iem_base = nullptr;
    sa.xtab = reinterpret_cast<const double *>(d_tab);

    ReduceArgs ra{};
    ra.nx = nx; ra.ny = ny; ra.nz = nz; ra.n_pair = plan.n_pair;
    ra.blocks = reinterpret_cast<const rt3d::LayerBlock *>(d_blocks);
    ra.P = d_P;
    ra.chi = chi;
    ra.Jfs = J_fs;
    ra.chunk = chunk;
    ra.waves = 1;
    for (const rt3d::SweepPart &part : parts) {
        sa.items = reinterpret_cast<const rt3d::WorkItem *>(d_items) + part.item0;
        if (part.layers < nz) {
            const LayerRange lr{part.down ? nz - 1 - part.step0 : part.step0, part.layers, part.q0, plan.n_pair, part.step0 == 0,
                                ra.blocks, reinterpret_cast<const int2 *>(d_start), d_P + room - rt3d::line_elems(plan, part)};
            hipLaunchKernelGGL(column_sweep_layers_kernel<double>, dim3(unsigned(part.n_items)), dim3(plan.block_threads),
                               sweep_smem_bytes(plan, false), st, sa, lr);
        } else {
            launch_sweep_kernel(sa, plan, 0, part.n_items, false, st);
        }
        e = hipGetLastError();
        if (e != hipSuccess) return drain_fail(RT3D_ERR_HIP, std::string("sweep_kernel: ") + hipGetErrorString(e));
        const dim3 red_grid(unsigned(((nx + 1) / 2 * ny + kPlaneThreads - 1) / kPlaneThreads), unsigned(part.layers));
        const int k0 = part.down ? nz - part.step0 - part.layers : part.step0;
        hipLaunchKernelGGL(plan.columns ? reduce_kernel_pair_range<true> : reduce_kernel_pair_range<false>, red_grid,
                           dim3(kPlaneThreads), 0, st, ra, part.q0, part.q1, k0, part.q0 == 0 ? 1 : 0,
                           part.q1 == plan.n_pair ? 1 : 0, d_carry);
        e = hipGetLastError();
        if (e != hipSuccess) return drain_fail(RT3D_ERR_HIP, std::string("reduce_kernel: ") + hipGetErrorString(e));
    }
    e = hipStreamSynchronize(st);
    if (e != hipSuccess) return noalloc_fail(RT3D_ERR_HIP, std::string("hipStreamSynchronize: ") + hipGetErrorString(e));
    return RT3D_OK;
}

}  // extern "C"
