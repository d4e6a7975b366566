// Single-launch evaluation for calls of few (polynomial, point) pairs, whose
// time is that of their launches: each workgroup tries its polynomial at its
// point by quotients (quotient.hip) and, if they refuse, evaluates it with
// the general stages (eval.hip) itself, where larger calls leave the refused
// ones to a second launch.  Bound: launch, point load and the chain of the
// three stages; general kernel -> here, n = 128, m = 256, k = 16 at one point
// in double-double 16.5 -> 9.9 us per call, in quad-double 117 -> 57 us.  Two
// launches cost about 4 us more.
#include "eval_body.hpp"
#include "quotient_body.hpp"

namespace pe {

// Instantiated like eval_kernel, whose registers and workgroup sizes the
// general stages need.
template <class A, int CC, int MAXT>
__global__ __launch_bounds__(MAXT) __attribute__((amdgpu_waves_per_eu(kWavesPerEu<A>))) void
small_kernel(const EvalArgs a, const QuotArgs qa)
{
    using C = typename A::C;
    HIP_DYNAMIC_SHARED(double2, lds_raw)
    const int p = xcd_order(blockIdx.x, gridDim.x);
    const int64_t pt = blockIdx.y;
    if (a.mask && a.mask[pt] != kMaskLive) return;
    {
        double2 *end;
        const QuotLds<A> lds = quot_lds<A>(lds_raw, qa, end);
        int *const flag = reinterpret_cast<int *>(end);
        if (threadIdx.x == 0) *flag = 0;
        const bool jac = qa.J[0] != nullptr;
        uint32_t *const words = reinterpret_cast<uint32_t *>(end + 1);
        quot_table<A, true>(qa, lds, pt, 1, p, 0, 1, jac, words);
        __syncthreads();
        if (!(bad_point<A>(qa, words) && uniform_int4(qa.poly + p).w)) {
            int vo = 0;
            quot_poly<A, true>(qa, lds, pt, 1u, false, p, vo, jac, [&] { *flag = 1; });
            __syncthreads();
            if (*flag == 0) return;
        }
        __syncthreads();  // the flag and the words have been read
    }
    const LdsLayout<A> lds = lds_layout<A, false>(lds_raw, a);
    const int4 *gi = a.group_info + 2 * (int64_t)p * a.merge;
    const int4 g0 = gi[0];
    const int c_begin = g0.x, c_end = gi[2 * (a.merge - 1)].y;
    C x0 = A::zero();
    if ((int)threadIdx.x < a.n_vars) x0 = Io<A>::load(a.x, pt * a.n_vars + threadIdx.x);
    ChunkIn<A, CC> in;
    RunIn rin = 0u;
    if (c_begin < c_end) {
        in.ci = a.chunk_info[c_begin];
        load_lane_in<A, CC>(a, in);
        rin = load_run_in(a, in.ci);
    }
    begin_point<A>(a, pt, lds, x0, gi + 1);
    __syncthreads();
    eval_group<A, CC, false>(a, p, c_begin, c_end, pt, lds, in, rin);
}

using SmallFn = void (*)(const EvalArgs, const QuotArgs);

template <class A>
static SmallFn pick(int cc, int maxt)
{
#define PE_CASE(CCV, MT) \
    if (cc == CCV && maxt == MT) return small_kernel<A, CCV, MT>;
    PE_CASE(2, 256) PE_CASE(2, 512) PE_CASE(2, 1024)
    PE_CASE(4, 256) PE_CASE(4, 512) PE_CASE(4, 1024)
    PE_CASE(8, 256) PE_CASE(8, 512) PE_CASE(8, 1024)
#undef PE_CASE
    return nullptr;
}

// the instantiations of eval_kernel in quad-double
static SmallFn pick_any(int prec, int cc, int maxt)
{
    if (prec == 1) return pick<ArithDD>(cc, maxt);
    if (prec == 0) return pick<Arith64>(cc, maxt);
    if (cc == 2 && maxt == 512) return small_kernel<ArithQD, 2, 512>;
    if (cc == 2 && maxt == 256) return small_kernel<ArithQD, 2, 256>;
    if (cc == 4 && maxt == 256) return small_kernel<ArithQD, 4, 256>;
    return nullptr;
}

hipError_t launch_small(int prec, int cc, int maxt, const EvalArgs &a, const QuotArgs &q, dim3 grid,
                        unsigned threads, size_t lds_bytes, hipStream_t stream)
{
    SmallFn k = pick_any(prec, cc, maxt);
    if (!k) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k, grid, dim3(threads), lds_bytes, stream, a, q);
    return hipGetLastError();
}

hipError_t small_kernels_init()
{
    for (int prec = 0; prec < 3; ++prec)
        for (int cc : {2, 4, 8})
            for (int maxt : {256, 512, 1024})
                // best effort: a refusal shows up later as a launch error
                if (SmallFn k = pick_any(prec, cc, maxt))
                    if (hipFuncSetAttribute(reinterpret_cast<const void *>(k),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds) != hipSuccess)
                        (void)hipGetLastError();
    return hipSuccess;
}

}  // namespace pe
