// Fused evaluation of a sparse polynomial system and its Jacobian on gfx950.
//
// One workgroup handles one polynomial (or a contiguous share of its
// monomials, when G > 1) at one point at a time.  The three stages of the
// paper (Section 2) run inside one kernel:
//
//  1. The point is read once, coalesced, and the power table x_i^r,
//     r = 1..R, of all variables is built in LDS by the lanes in parallel
//     (Section 3.1, first stage; R = d-1 for a maximal exponent d).  An
//     extra column holds the value 1 for padding entries.
//  2. Each monomial is handled by a group of L lanes, CC variables per lane:
//     common factor from the power table, Speelpenning partials with forward
//     and backward products in registers, coefficient and exponent scaling
//     (Sections 3.1 and 3.2; see monomial.hpp).  Supports, exponents and
//     coefficients are read coalesced: lane q of a group reads variables
//     q*CC .. q*CC+CC-1 of its monomial from a monomial-major table.
//  3. Summation (Section 3.3) without the zero-padded dense term array: the
//     outputs of a chunk are ranked by the length of their runs of terms;
//     row i of the LDS staging area holds the i-th term (in monomial
//     order) of every output with more than i terms, the j-th ranked
//     output's at slot rows[i] + j (slots chosen on the host).  The run of
//     rank j is added by 2^log2S lanes (as many as fit one round, up to 16;
//     one lane for large n), each with a cascaded accumulator over every
//     2^log2S-th row, then a butterfly over those lanes, and goes into the
//     output's LDS accumulator: the paper's one thread per output, per
//     chunk.  At each step consecutive lanes read consecutive slots, so the
//     reads are free of bank conflicts.  All orders are fixed, so results
//     are deterministic.
//
// A workgroup may also take a tile of T consecutive points (TILE = true,
// see eval_tile): the chunk inputs then serve all T points, whose power
// tables and accumulators sit side by side in LDS, and with two staging
// buffers one barrier per (chunk, point) item suffices.  Tiles of one point
// with one buffer run the one-point body (eval_group), whose code is free of
// the tile bookkeeping.
//
// With G > 1 the workgroups of one polynomial each write their partial row
// to global memory and a second small kernel (combine_kernel) adds the G
// rows in a fixed order; the kernel boundary makes the rows visible, so no
// device-wide fence is needed inside the evaluation.
//
// A second kernel runs many systems of different shapes in one persistent
// launch over a host-built task list (see batch_kernel).
#include <algorithm>
#include <atomic>
#include <mutex>

#include "eval_body.hpp"

namespace pe {

// Which of the points pt0 + i gridDim.y, i = 0 .. 63, a quotient kernel left
// polynomial p at, among those that are evaluated (bit i; the same answer on
// every thread).  Each wave reads the marks of 64 points at once: one at a time,
// the load was a fifth of the work on a point in FP64.  The caller writes these
// values only after a barrier.
__device__ __forceinline__ uint64_t refused_points(const EvalArgs &a, int p, int64_t pt0)
{
    const int64_t pt = pt0 + (int64_t)(threadIdx.x & 63) * gridDim.y;
    return __ballot(pt < a.n_points && !(a.mask && a.mask[pt] != kMaskLive) &&
                    is_refused(a.f[0][pt * a.n_polys + p]));
}

// One system: workgroup (group, tile block); tiles of T consecutive points,
// strided by gridDim.y.  A group with a single chunk keeps its inputs in
// registers for all its tiles; otherwise the first chunk's inputs are
// fetched again per tile.  The first point's entries are requested first, so
// that their latency overlaps the dependent loads of the group header and the
// chunk inputs.
// REPAIR: only the polynomials at the points that a quotient kernel refused,
// with all shares of a polynomial on one workgroup (not tiled); in a kernel of
// its own, as the tests for it cost the others 3%.
template <class A, int CC, int MAXT, bool TILE, bool REPAIR = false>
__global__ __launch_bounds__(MAXT) __attribute__((amdgpu_waves_per_eu(kWavesPerEu<A>))) void
eval_kernel(const EvalArgs a)
{
    static_assert(!(TILE && REPAIR), "repairs take one point at a time");
    if constexpr (!TILE) {
        using C = typename A::C;
        HIP_DYNAMIC_SHARED(double2, lds_raw)
        const LdsLayout<A> lds = lds_layout<A, false>(lds_raw, a);
        const int group = xcd_order(blockIdx.x, gridDim.x);
        int64_t pt0 = blockIdx.y;
        const int64_t batch = 64 * (int64_t)gridDim.y;  // points asked for at once
        uint64_t todo = 0;
        if constexpr (REPAIR) {
            while (pt0 < a.n_points && !(todo = refused_points(a, group, pt0))) pt0 += batch;
            if (!todo) return;
        }
        const bool has_x = (int)threadIdx.x < a.n_vars;
        // the first point's entry is requested before the tables
        C x0 = A::zero();
        if (!REPAIR && pt0 < a.n_points && has_x) x0 = Io<A>::load(a.x, pt0 * a.n_vars + threadIdx.x);
        const int4 *gi = a.group_info + 2 * (int64_t)group * (REPAIR ? a.merge : 1);
        const int4 g0 = gi[0], g1 = gi[1];
        const int c_begin = g0.x, c_end = REPAIR ? gi[2 * (a.merge - 1)].y : g0.y;
        const bool single = c_end - c_begin == 1;
        ChunkIn<A, CC> in;
        RunIn rin = 0u;
        bool loaded = false, first = true;
        auto point = [&](int64_t pt) {
            if (!first) __syncthreads();  // the previous point is done with LDS
            first = false;
            if ((REPAIR || pt != pt0) && has_x) x0 = Io<A>::load(a.x, pt * a.n_vars + threadIdx.x);
            if (!loaded && c_begin < c_end) {
                // (merged shares: the first one may be empty, without a header)
                in.ci = REPAIR ? a.chunk_info[c_begin] : make_int4(g0.z, g0.w, g1.x, g1.y);
                load_lane_in<A, CC>(a, in);
                rin = load_run_in(a, in.ci);
                loaded = single;
            }
            begin_point<A>(a, pt, lds, x0, gi + 1);
            __syncthreads();
            eval_group<A, CC, (CC <= 4)>(a, group, c_begin, c_end, pt, lds, in, rin);
        };
        if constexpr (REPAIR) {
            for (;;) {
                for (; todo; todo &= todo - 1) point(pt0 + (int64_t)(__ffsll((unsigned long long)todo) - 1) * gridDim.y);
                if ((pt0 += batch) >= a.n_points) break;
                todo = refused_points(a, group, pt0);
            }
        } else {
            for (int64_t pt = pt0; pt < a.n_points; pt += gridDim.y)
                if (!(a.mask && a.mask[pt] != kMaskLive)) point(pt);
        }
    } else {
        using C = typename A::C;
        HIP_DYNAMIC_SHARED(double2, lds_raw)
        const LdsLayout<A> lds = lds_layout<A>(lds_raw, a);
        const int group = xcd_order(blockIdx.x, gridDim.x);
        const int T = a.T;
        const int64_t n_tiles = (a.n_points + T - 1) / T;
        const int64_t tile0 = blockIdx.y;
        const bool has_x = (int)threadIdx.x < a.n_vars;
        // the first point's entry is requested before the tables
        C x0 = A::zero();
        if (tile0 < n_tiles && has_x) x0 = Io<A>::load(a.x, tile0 * T * a.n_vars + threadIdx.x);
        const int4 *gi = a.group_info + 2 * (int64_t)group;
        const int4 g0 = gi[0], g1 = gi[1];
        const int c_begin = g0.x, c_end = g0.y;
        const bool single = c_end - c_begin == 1;
        ChunkIn<A, CC> in;
        RunIn rin = 0u;
        bool loaded = false, first = true;
        for (int64_t tile = tile0; tile < n_tiles; tile += gridDim.y) {
            const int64_t pt0 = tile * T;
            const int npt = (int)min<int64_t>(T, a.n_points - pt0);
            uint32_t live = npt >= 32 ? 0xFFFFFFFFu : ((1u << npt) - 1u);
            if (a.mask)
                for (int t = 0; t < npt; ++t)
                    if (a.mask[pt0 + t] != kMaskLive) live &= ~(1u << t);
            if (!live) continue;
            if (!first) __syncthreads();  // the previous tile is done with LDS
            first = false;
            if (tile != tile0 && has_x) x0 = Io<A>::load(a.x, pt0 * a.n_vars + threadIdx.x);
            if (!loaded && c_begin < c_end) {
                in.ci = make_int4(g0.z, g0.w, g1.x, g1.y);
                load_lane_in<A, CC>(a, in);
                rin = load_run_in(a, in.ci);
                loaded = single;
            }
            begin_tile<A>(a, pt0, live, lds, x0, gi + 1);
            __syncthreads();
            eval_tile<A, CC>(a, group, c_begin, c_end, pt0, npt, live, lds, in, rin);
        }
    }
}

// Many systems in one persistent launch: workgroup b takes the tasks
// b, b + gridDim.x, ... of a host-ordered list (longest first); a task is one
// point of one system and some of its polynomials, which share the power
// table built once for the task.
template <class A, int CC, int MAXT>
__global__ __launch_bounds__(MAXT) void batch_kernel(const BatchArgs b)
{
    using C = typename A::C;
    HIP_DYNAMIC_SHARED(double2, lds_raw)
    ChunkIn<A, CC> in;
    RunIn rin = 0u;
    if (b.repair) {
        // whether a quotient kernel left some polynomial of this workgroup's tasks
        bool any = false;
        for (int64_t t = blockIdx.x + (int64_t)threadIdx.x * gridDim.x; t < b.n_tasks;
             t += (int64_t)blockDim.x * gridDim.x) {
            const BatchTask task = b.tasks[t];
            const BatchDesc &d = b.desc[task.sys];
            const double *f = b.f[0] + d.f_off + task.pt * d.a.n_polys;
            for (int p = task.p0; p < task.p1; p += task.step) any = any || is_refused(f[p]);
        }
        if (!any_of_workgroup(any, reinterpret_cast<int *>(lds_raw))) return;
    }
    for (int64_t t = blockIdx.x; t < b.n_tasks; t += gridDim.x) {
        const BatchTask task = b.tasks[t];
        const BatchDesc &d = b.desc[task.sys];
        EvalArgs a = d.a;
        for (int q = 0; q < 4; ++q) {
            a.x[q] = b.x[q] ? b.x[q] + d.x_off : nullptr;
            a.f[q] = b.f[q] ? b.f[q] + d.f_off : nullptr;
            a.J[q] = b.J[q] ? b.J[q] + d.J_off : nullptr;
        }
        const LdsLayout<A> lds = lds_layout<A, false>(lds_raw, a);
        __syncthreads();  // the previous task is done with LDS
        bool begun = false;
        uint64_t todo = 0;
        for (int i = 0, p = task.p0; p < task.p1; ++i, p += task.step) {
            // the marks of 64 polynomials at once (f of polynomial p is written
            // only by this task, below, after a barrier)
            if ((i & 63) == 0) {
                const int q = p + (int)(threadIdx.x & 63) * task.step;
                todo = __ballot(q < task.p1 && (!b.repair || is_refused(a.f[0][task.pt * a.n_polys + q])));
            }
            if (!((todo >> (i & 63)) & 1)) continue;
            const int4 g0 = a.group_info[2 * p];
            const int4 g1 = a.group_info[2 * p + 1];
            if (g0.x < g0.y) {
                in.ci = make_int4(g0.z, g0.w, g1.x, g1.y);
                load_lane_in<A, CC>(a, in);
                rin = load_run_in(a, in.ci);
            }
            if (!begun) {
                begun = true;
                C x0 = A::zero();
                if ((int)threadIdx.x < a.n_vars)
                    x0 = Io<A>::load(a.x, task.pt * a.n_vars + threadIdx.x);
                begin_point<A>(a, task.pt, lds, x0, a.group_info + 2 * p + 1);
            } else {
                __syncthreads();  // the previous polynomial's outputs have been read
                init_acc<A>(a, lds, 0, a.group_info + 2 * p + 1);
            }
            __syncthreads();
            eval_group<A, CC, false>(a, p, g0.x, g0.y, task.pt, lds, in, rin);
        }
    }
}

// f and J from the G partial rows of each (point, polynomial), added in
// workgroup order.  Thread e of a point takes entry (o, p) with
// e = o * n_polys + p, so consecutive threads write consecutive entries of
// J (and of f, o = n_vars).  The host guarantees (n_vars+1)*n_polys < 2^31.
template <class A>
__global__ __launch_bounds__(256) void combine_kernel(const EvalArgs a)
{
    using C = typename A::C;
    using IO = Io<A>;
    constexpr int W = A::kWords;
    const int n = a.n_vars, np1 = n + 1, P = a.n_polys;
    const int total = np1 * P;
    const int stride = gridDim.x * blockDim.x;
    const int64_t blk = (int64_t)total * W;  // one group's block [o][n_polys]
    for (int64_t pt = blockIdx.y; pt < a.n_points; pt += gridDim.y) {
        if (a.mask && a.mask[pt] != kMaskLive) continue;
        const double *rows = a.partial + pt * a.G * blk;
        for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < total; e += stride) {
            const int o = e / P, p = e - o * P;
            const double *src = rows + (int64_t)e * W;
            C v = IO::get(src);
            for (int g = 1; g < a.G; ++g) v = A::sum(v, IO::get(src + g * blk));
            if (o == n)
                IO::store(a.f, pt * P + p, v);
            else if (a.J[0])
                IO::store(a.J, pt * (int64_t)n * P + e, v);
        }
    }
}

hipError_t launch_combine(int prec, const EvalArgs &args, hipStream_t stream)
{
    const int64_t total = (int64_t)args.n_polys * (args.n_vars + 1);
    if (total <= 0 || args.n_points <= 0) return hipSuccess;
    const unsigned bx = (unsigned)std::min<int64_t>((total + 255) / 256, 4096);
    const unsigned by = (unsigned)std::min<int64_t>(args.n_points, 65535);
    if (prec == 2)
        hipLaunchKernelGGL(combine_kernel<ArithQD>, dim3(bx, by), dim3(256), 0, stream, args);
    else if (prec == 1)
        hipLaunchKernelGGL(combine_kernel<ArithDD>, dim3(bx, by), dim3(256), 0, stream, args);
    else
        hipLaunchKernelGGL(combine_kernel<Arith64>, dim3(bx, by), dim3(256), 0, stream, args);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// dispatch
// ---------------------------------------------------------------------------

using KernelFn = void (*)(const EvalArgs);

template <class A, bool TILE, bool REPAIR>
static KernelFn pick(int cc, int maxt)
{
#define PE_CASE(CCV, MT) \
    if (cc == CCV && maxt == MT) return eval_kernel<A, CCV, MT, TILE, REPAIR>;
    PE_CASE(2, 256) PE_CASE(2, 512) PE_CASE(2, 1024)
    PE_CASE(4, 256) PE_CASE(4, 512) PE_CASE(4, 1024)
    PE_CASE(8, 256) PE_CASE(8, 512) PE_CASE(8, 1024)
#undef PE_CASE
    return nullptr;
}

// quad-double: 256 threads with two or four variables per lane, or 512
// threads with two (two waves per SIMD); one point per workgroup
template <bool REPAIR>
static KernelFn pick_qd(int cc, int maxt)
{
    if (maxt == 512) return cc == 2 ? eval_kernel<ArithQD, 2, 512, false, REPAIR> : nullptr;
    if (maxt != 256) return nullptr;
    if (cc == 2) return eval_kernel<ArithQD, 2, 256, false, REPAIR>;
    if (cc == 4) return eval_kernel<ArithQD, 4, 256, false, REPAIR>;
    return nullptr;
}

// tile and repair: not both (the launch would be refused)
static KernelFn pick_any(int prec, int cc, int maxt, bool tile, bool repair)
{
    if (tile && (repair || prec == 2)) return nullptr;
    if (prec == 2) return repair ? pick_qd<true>(cc, maxt) : pick_qd<false>(cc, maxt);
    if (prec == 1)
        return tile     ? pick<ArithDD, true, false>(cc, maxt)
               : repair ? pick<ArithDD, false, true>(cc, maxt)
                        : pick<ArithDD, false, false>(cc, maxt);
    return tile     ? pick<Arith64, true, false>(cc, maxt)
           : repair ? pick<Arith64, false, true>(cc, maxt)
                    : pick<Arith64, false, false>(cc, maxt);
}

// Tiles of one point with one staging buffer run the one-point kernel body;
// anything else the tiled one.
hipError_t launch_eval(int prec, int cc, int maxt, const EvalArgs &args, dim3 grid, dim3 block,
                       size_t lds_bytes, hipStream_t stream)
{
    KernelFn k = pick_any(prec, cc, maxt, args.T > 1 || args.nbuf > 1, args.repair != 0);
    if (!k) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, grid, block, lds_bytes, stream, args);
    return hipGetLastError();
}

using BatchFn = void (*)(const BatchArgs);

template <class A>
static BatchFn pick_batch(int cc, int maxt)
{
#define PE_CASE(CCV, MT) \
    if (cc == CCV && maxt == MT) return batch_kernel<A, CCV, MT>;
    PE_CASE(2, 256) PE_CASE(2, 512) PE_CASE(2, 1024)
    PE_CASE(4, 256) PE_CASE(4, 512) PE_CASE(4, 1024)
    PE_CASE(8, 256) PE_CASE(8, 512) PE_CASE(8, 1024)
#undef PE_CASE
    return nullptr;
}

hipError_t launch_batch(int prec, int cc, int maxt, const BatchArgs &args, dim3 grid, dim3 block,
                        size_t lds_bytes, hipStream_t stream)
{
    BatchFn k = prec == 1 ? pick_batch<ArithDD>(cc, maxt) : pick_batch<Arith64>(cc, maxt);
    if (!k) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, grid, block, lds_bytes, stream, args);
    return hipGetLastError();
}

int batch_occupancy(int prec, int cc, int maxt, int threads, size_t lds_bytes)
{
    BatchFn k = prec == 1 ? pick_batch<ArithDD>(cc, maxt) : pick_batch<Arith64>(cc, maxt);
    int blocks = 0;
    if (!k || hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, reinterpret_cast<const void *>(k),
                                                           threads, lds_bytes) != hipSuccess) {
        (void)hipGetLastError();
        return 1;
    }
    return blocks > 0 ? blocks : 1;
}

// The static scratch of the allocation-free evaluation.  In host code the
// name `scratch` is only a stand-in for the symbol: its device address, which
// differs per device, comes from hipGetSymbolAddress and is the only handle
// passed to kernels.
static __device__ __align__(256) double scratch[kStaticScratchBytes / sizeof(double)];

constexpr int kMaxScratchDevices = 64;
static std::atomic<void *> g_scratch_ptr[kMaxScratchDevices];
static std::mutex g_scratch_mu;

hipError_t static_scratch_setup()
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxScratchDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_ptr[dev].load()) return hipSuccess;
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev].store(p);
    return hipSuccess;
}

void *static_scratch_ptr(int device)
{
    if (device < 0 || device >= kMaxScratchDevices) return nullptr;
    return g_scratch_ptr[device].load();
}

hipError_t eval_kernels_init()
{
    const int ccs[3] = {2, 4, 8};
    const int mts[3] = {256, 512, 1024};
    for (int prec = 0; prec < 2; ++prec)
        for (int c : ccs)
            for (int m : mts) {
                const void *ks[4] = {reinterpret_cast<const void *>(pick_any(prec, c, m, false, false)),
                                     reinterpret_cast<const void *>(pick_any(prec, c, m, false, true)),
                                     reinterpret_cast<const void *>(pick_any(prec, c, m, true, false)),
                                     reinterpret_cast<const void *>(
                                         prec == 1 ? pick_batch<ArithDD>(c, m)
                                                   : pick_batch<Arith64>(c, m))};
                // best effort: a refusal shows up later as a launch error
                for (const void *k : ks)
                    if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                            kMaxLds) != hipSuccess)
                        (void)hipGetLastError();
            }
    for (int c : {2, 4})
        for (KernelFn k : {pick_qd<false>(c, 256), pick_qd<true>(c, 256)})
            if (hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds) != hipSuccess)
                (void)hipGetLastError();
    return hipSuccess;
}

}  // namespace pe
