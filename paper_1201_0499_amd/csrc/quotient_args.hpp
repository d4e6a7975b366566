// Launch arguments and launch wrappers of the quotient kernels (quotient.hip)
// and of the single-launch kernel (small.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "eval.hpp"
#include "quotient.hpp"

namespace pe {

struct QuotArgs {
    int32_t n_vars, n_polys;
    int32_t D;           // power-table rows x^1 .. x^D
    int32_t pad;         // 1: the power table ends with the entry 1
    int32_t CH;          // monomials per chunk
    int32_t n_blk;       // rank blocks per chunk
    int32_t check;       // quads of factors are checked too (see quot_window)
    int32_t pairs;       // no monomial has more than two variables
    int32_t sparse;      // workgroups of one polynomial each, with few terms for its
                         //   variables: see quot_table
    int32_t skip;        // polynomials in which every variable occurs are left to the
                         //   general kernel at points with a coordinate out of range
                         //   without further work: see bad_point
    int32_t multi;       // some polynomial has more than one chunk
    int32_t log2L;       // lanes per monomial: 1, 2 or 4
    int32_t log2S;       // lanes per run of terms: 1, 2 or 4
    int32_t PP;          // polynomials per workgroup (values only)
    int32_t blocks;      // workgroups that share a point's polynomials: block b takes
                         //   b, b + blocks, ...
    int32_t by_point;    // 1: a point's workgroups run on one XCD; 0: an XCD's
                         //   workgroups take neighbouring polynomials of every point
    int32_t nbuf;        // buffers of chunk values: 1, or 2 (one barrier per chunk)
    uint32_t x_lo, x_span;  // high words of admitted |x| parts: x_lo .. x_lo + x_span - 1
    const uint2 *words;  // see QuotTables
    const double *coef;  // [monomials in table order][4]
    const int2 *slice;
    const int4 *chunk;
    const int4 *poly;
    const int2 *block;
    const uint16_t *runs;
    const uint16_t *out;
    const double *sys_coef;  // [M][4] in the system's order, for folded constants
    int64_t n_points;
    const double *x[8];
    double *f[8];
    double *J[8];            // J[0] == nullptr: values only
    const int32_t *mask;     // as in EvalArgs
};

// One system of a batch (see BatchDesc); CH == 0: outside these kernels.
struct QuotBatchDesc {
    QuotArgs a;
    int64_t x_off, f_off, J_off;
};

struct QuotBatchArgs {
    const QuotBatchDesc *desc;
    const BatchTask *tasks;
    int64_t n_tasks;
    const double *x[4];
    double *f[4];
    double *J[4];
};

// Launches (prec 0 = FP64, 1 = double-double, 2 = quad-double; T points per
// workgroup, 1 or in FP64 kPointsF64).  A polynomial at a point that the
// range rules refuse gets refused() as the leading word of its value; the
// general kernel then evaluates it, and writes all its outputs.
constexpr int kPointsF64 = 2;
hipError_t launch_quot(int prec, int T, const QuotArgs &args, dim3 grid, unsigned threads, size_t lds_bytes,
                       hipStream_t stream);
hipError_t launch_quot_batch(int prec, const QuotBatchArgs &args, unsigned grid, unsigned threads,
                             size_t lds_bytes, hipStream_t stream);

// Both in one launch, the general evaluation on what the quotients refuse:
// workgroups of whole polynomials, one point each (a.merge = all shares,
// a.G = 1; cc and maxt as for launch_eval).
hipError_t launch_small(int prec, int cc, int maxt, const EvalArgs &a, const QuotArgs &q, dim3 grid,
                        unsigned threads, size_t lds_bytes, hipStream_t stream);

// Raise the dynamic LDS limit of the kernels (once per process).
hipError_t quot_kernels_init();
hipError_t small_kernels_init();

}  // namespace pe
