// Quotient kernels: f and J with one product per factor of a monomial.
//
//     V_s = c_s prod_j x_{i_j}^{a_j},   f_p = sum_s V_s,
//     df_p/dx_i = (1 / x_i) sum_s a_{s,i} V_s.
//
// One workgroup takes a point (in FP64 two) and a few consecutive
// polynomials.  The power table x_i^r, r = 1..d, and the reciprocals 1 / x_i
// are built in LDS once (Section 3.1's table, one row more).  Then, per chunk
// of monomials:
//   1. each lane (or 2 or 4 lanes) multiplies the factors of one monomial
//      and its coefficient and writes the value V to LDS: k products instead
//      of the about 5k of the forward and backward products (Section 3.2);
//   2. each output's run, a list of (monomial, exponent), is added by 1, 2
//      or 4 lanes reading the V from LDS (Section 3.3's summation, one
//      thread per output); the last chunk's sum times 1 / x_i goes to J.
// Only one value per monomial passes through LDS where the general kernel
// stages k + 1 terms.  All orders are fixed by the system alone (quotient.hpp),
// so results do not depend on the launch shape.
//
// Bound: instruction issue (in double-double 38 FP64 instructions per factor
// and 23 per scaled addition).  Against the general kernel's forward and
// backward products, one MI355X: n = 512, m = 1024, k = 32, d = 5, 256 points
// in double-double 58.2 -> 12.7 ms; n = 100, m = 200, k up to 16, 1000 points
// in FP64 1130 -> 307 us; values only, n = 150, m = 299, k up to 12, 333
// points in double-double 2912 -> 232 us.
//
// Rounding: a term takes k products where the other way takes about 2k, but
// each power is one product longer, and a derivative has the error of 1 / x
// and one product more.  Root mean square of the derivatives' errors in
// double-double, in u^2 of the terms' magnitudes (host, unit-circle points),
// forward and backward products against quotients: k = 16, d = 2 0.73 and
// 0.75, d = 3 1.26 and 1.36; k = 8, d = 3 1.84 and 2.00; k = 6, d = 3 0.76 and
// 0.82; k = 2, d = 3 0.81 and 1.07; in FP64, in u, k = 16, d = 2 0.53 and 0.53,
// k = 2, d = 3 0.74 and 0.94.  (With inv in the place of recip 0.78, 1.42,
// 2.17, 0.88, 1.30; 0.54, 1.11.)  Values' errors are those of the other way
// within the sample's noise.
#include "quotient_body.hpp"

namespace pe {

template <class A>
constexpr int kQuotMaxThreads = 1024;  // 128 registers per lane
template <>
constexpr int kQuotMaxThreads<ArithQD> = 512;  // quad-double values take eight registers per part

// With the Jacobian.  Work item w is a tile of T points and a block, whose
// polynomials lie `blocks` apart: neighbouring polynomials, whose entries of J
// share cache lines (J is polynomial-minor), are then at the same step of
// neighbouring workgroups, and those run on one XCD (workgroup i on XCD i mod
// 8, grid a multiple of 8), whose L2 merges the lines.  With consecutive
// polynomials one after another in a workgroup the lines left the L2 in
// between: at n = 512, 256 points, 11.5 GB written for 2.1 GB of J.
template <class A>
__global__ __launch_bounds__(kQuotMaxThreads<A>) void quot_kernel(const QuotArgs a)
{
    constexpr int T = Pts<A>::T;
    HIP_DYNAMIC_SHARED(double2, lds_raw)
    double2 *end;
    const QuotLds<A> lds = quot_lds<A>(lds_raw, a, end);
    uint32_t *const words = wave_words<A>(a, lds, end);
    const int64_t tiles = (a.n_points + T - 1) / T;
    const int per_xcd = a.by_point ? a.blocks : (a.blocks + 7) / 8;
    const int64_t rounds = a.by_point ? (tiles + 7) / 8 : tiles;
    bool first = true;
    for (int64_t w = blockIdx.x; w < 8 * per_xcd * rounds; w += gridDim.x) {
        const int xcd = (int)(w & 7);
        const int64_t round = (w >> 3) / per_xcd;
        const int slot = (int)((w >> 3) - round * per_xcd);
        const int64_t tile = a.by_point ? round * 8 + xcd : round;
        const int block = a.by_point ? slot : xcd * per_xcd + slot;
        if (tile >= tiles || block >= a.blocks) continue;
        const int64_t pt = tile * T;
        const int npt = (int)min<int64_t>(T, a.n_points - pt);
        uint32_t live = (1u << npt) - 1;
        if (a.mask)
            for (int t = 0; t < npt; ++t)
                if (a.mask[pt + t] != kMaskLive) live &= ~(1u << t);
        if (!live) continue;
        if (!first) __syncthreads();  // the previous points are done with LDS
        first = false;
        quot_table<A, true>(a, lds, pt, npt, block, a.n_polys, a.blocks, true, words);
        __syncthreads();
        const bool bad = bad_point<A>(a, words);
        int vo = 0;
        for (int p = block; p < a.n_polys; p += a.blocks)
            quot_poly<A, false>(a, lds, pt, live, bad, p, vo, true, [] {});
    }
}

// Values only: a wave takes whole polynomials, so that nothing but the power
// table is shared and no wave waits for another.
template <class A>
__global__ __launch_bounds__(kQuotMaxThreads<A>) void quot_values_kernel(const QuotArgs a)
{
    constexpr int T = Pts<A>::T;
    HIP_DYNAMIC_SHARED(double2, lds_raw)
    const int b = xcd_order(blockIdx.x, gridDim.x);
    const int p0 = b * a.PP, p1 = min(a.n_polys, p0 + a.PP);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), nw = (int)blockDim.x >> 6;
    double2 *end;
    QuotLds<A> lds{};
    lds.u = LdsVec<A>::at(lds_raw, a.D * a.n_vars + a.pad, end);
    uint32_t *const words = reinterpret_cast<uint32_t *>(end);
    bool first = true;
    for (int64_t pt = (int64_t)blockIdx.y * T; pt < a.n_points; pt += (int64_t)gridDim.y * T) {
        const int npt = (int)min<int64_t>(T, a.n_points - pt);
        uint32_t live = (1u << npt) - 1;
        if (a.mask)
            for (int t = 0; t < npt; ++t)
                if (a.mask[pt + t] != kMaskLive) live &= ~(1u << t);
        if (!live) continue;
        if (!first) __syncthreads();  // the previous points are done with LDS
        first = false;
        quot_table<A, true>(a, lds, pt, npt, p0, p1, 1, false, words);
        __syncthreads();
        const bool bad = bad_point<A>(a, words);
        for (int p = p0 + wave; p < p1; p += nw) quot_value<A>(a, lds.u, pt, live, bad, p);
    }
}

// Many systems in one persistent launch: workgroup b takes the tasks
// b, b + gridDim.x, ... of the batch's list.  Tasks of systems outside these
// kernels are refused whole.  24 systems of up to 160 variables and 512
// monomials, 24 points each in double-double: 2108 us by the general kernel,
// 1510 us with that kernel's coarse tasks and the descriptors in vector
// registers, 876 us.
template <class A, bool JAC>
__global__ __launch_bounds__(kQuotMaxThreads<A>) void quot_batch_kernel(const QuotBatchArgs b)
{
    HIP_DYNAMIC_SHARED(double2, lds_raw)
    for (int64_t t = blockIdx.x; t < b.n_tasks; t += gridDim.x) {
        const BatchTask task = uniform_struct(b.tasks + t);
        const QuotBatchDesc d = uniform_struct(b.desc + task.sys);
        QuotArgs a = d.a;
        for (int q = 0; q < 4; ++q) {
            a.x[q] = b.x[q] ? b.x[q] + d.x_off : nullptr;
            a.f[q] = b.f[q] ? b.f[q] + d.f_off : nullptr;
            a.J[q] = b.J[q] ? b.J[q] + d.J_off : nullptr;
        }
        if (a.CH == 0) {
            for (int p = task.p0 + (int)threadIdx.x * task.step; p < task.p1; p += (int)blockDim.x * task.step)
                a.f[0][task.pt * a.n_polys + p] = refused();
            continue;
        }
        double2 *end;
        const QuotLds<A> lds = quot_lds<A>(lds_raw, a, end);
        __syncthreads();  // the previous task is done with LDS
        quot_table<A, false>(a, lds, task.pt, 1, task.p0, task.p1, task.step, JAC, nullptr);
        __syncthreads();
        if constexpr (JAC) {
            int vo = 0;
            for (int p = task.p0; p < task.p1; p += task.step)
                quot_poly<A, false>(a, lds, task.pt, 1u, false, p, vo, true, [] {});
        } else {
            const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), nw = (int)blockDim.x >> 6;
            for (int p = task.p0 + wave * task.step; p < task.p1; p += nw * task.step)
                quot_value<A>(a, lds.u, task.pt, 1u, false, p);
        }
    }
}

using QuotFn = void (*)(const QuotArgs);
using QuotBatchFn = void (*)(const QuotBatchArgs);

static QuotFn pick_quot(int prec, int T, bool jac)
{
    if (prec == 2) return jac ? quot_kernel<ArithQD> : quot_values_kernel<ArithQD>;
    if (prec == 1) return jac ? quot_kernel<ArithDD> : quot_values_kernel<ArithDD>;
    if (T == kPointsF64)
        return jac ? quot_kernel<PointsF64<kPointsF64>> : quot_values_kernel<PointsF64<kPointsF64>>;
    return jac ? quot_kernel<Arith64> : quot_values_kernel<Arith64>;
}

static QuotBatchFn pick_quot_batch(int prec, bool jac)
{
    if (prec == 1) return jac ? quot_batch_kernel<ArithDD, true> : quot_batch_kernel<ArithDD, false>;
    return jac ? quot_batch_kernel<Arith64, true> : quot_batch_kernel<Arith64, false>;
}

hipError_t launch_quot(int prec, int T, const QuotArgs &args, dim3 grid, unsigned threads, size_t lds_bytes,
                       hipStream_t stream)
{
    hipLaunchKernelGGL(pick_quot(prec, T, args.J[0] != nullptr), grid, dim3(threads), lds_bytes, stream, args);
    return hipGetLastError();
}

hipError_t launch_quot_batch(int prec, const QuotBatchArgs &args, unsigned grid, unsigned threads,
                             size_t lds_bytes, hipStream_t stream)
{
    hipLaunchKernelGGL(pick_quot_batch(prec, args.J[0] != nullptr), dim3(grid), dim3(threads), lds_bytes,
                       stream, args);
    return hipGetLastError();
}

hipError_t quot_kernels_init()
{
    for (bool jac : {false, true}) {
        const void *ks[] = {reinterpret_cast<const void *>(pick_quot(0, 1, jac)),
                            reinterpret_cast<const void *>(pick_quot(0, kPointsF64, jac)),
                            reinterpret_cast<const void *>(pick_quot(1, 1, jac)),
                            reinterpret_cast<const void *>(pick_quot(2, 1, jac)),
                            reinterpret_cast<const void *>(pick_quot_batch(0, jac)),
                            reinterpret_cast<const void *>(pick_quot_batch(1, jac))};
        // best effort: a refusal shows up later as a launch error
        for (const void *k : ks)
            if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds) != hipSuccess)
                (void)hipGetLastError();
    }
    return hipSuccess;
}

}  // namespace pe
