// Path tracker kernels (see track.hpp).  All arithmetic is complex FP64;
// the double-double endgame at t = 1 is the Newton corrector's.
#include <hip/hip_runtime.h>

#include <cmath>

#include "device.hpp"
#include "monomial.hpp"
#include "newton.hpp"
#include "packing.hpp"
#include "track.hpp"

namespace pe {

namespace {

struct Cx {
    double re, im;
};

__device__ __forceinline__ Cx cmul(Cx a, Cx b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
__device__ __forceinline__ Cx cadd(Cx a, Cx b) { return {a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ Cx csub(Cx a, Cx b) { return {a.re - b.re, a.im - b.im}; }
__device__ __forceinline__ Cx cscale(Cx a, double s) { return {a.re * s, a.im * s}; }

// z^e for an integer e >= 0 by repeated squaring
__device__ __forceinline__ Cx cpow(Cx z, int e)
{
    Cx r{1.0, 0.0};
    while (e > 0) {
        if (e & 1) r = cmul(r, z);
        z = cmul(z, z);
        e >>= 1;
    }
    return r;
}

__global__ void start_kernel(int64_t first, int64_t n_paths, int32_t n, const int32_t *deg,
                             double *xrh, double *xrl, double *xih, double *xil)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n_paths) return;
    // mixed-radix digits of the path index, variable 0 fastest; the index
    // is taken modulo the product of the degrees as it goes
    uint64_t q = (uint64_t)(first + p);
    for (int i = 0; i < n; ++i) {
        const uint64_t d = (uint64_t)deg[i];
        const uint64_t k = q % d;
        q /= d;
        double s, c;
        sincospi(2.0 * (double)k / (double)d, &s, &c);
        xrh[p * n + i] = c;
        xrl[p * n + i] = 0.0;
        xih[p * n + i] = s;
        xil[p * n + i] = 0.0;
    }
}

__global__ void init_kernel(TrackArgs a, double h_init, double *xrl, double *xil)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t total = a.n_paths * a.n;
    if (e >= total) return;
    a.xs[0][e] = a.x[0][e];
    a.xs[1][e] = a.x[1][e];
    xrl[e] = 0.0;
    xil[e] = 0.0;
    if (e % a.n == 0) {
        const int64_t p = e / a.n;
        a.t[p] = 0.0;
        a.t1[p] = 0.0;
        a.h[p] = h_init;
        a.phase[p] = 0;
        a.succ[p] = 0;
        a.steps[p] = 0;
        a.status[p] = kRunning;
    }
}

// Entry e of the P x n x n Jacobians (column-major: column c, row i at
// c*n + i): H_x = tau * J_F + (1 - tau) * gamma * diag(d_i x_i^{d_i - 1});
// the threads of column 0 also write the right-hand side of row i.
__global__ void homotopy_kernel(TrackArgs a)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t nn = (int64_t)a.n * a.n;
    if (e >= a.n_paths * nn) return;
    const int64_t p = e / nn;
    if (a.status[p] != kRunning) return;
    const int rem = (int)(e - p * nn);
    const int c = rem / a.n, i = rem - c * a.n;
    const bool predict = a.phase[p] == 0;
    const double tau = predict ? a.t[p] : a.t1[p];
    const Cx gamma{a.gamma_re, a.gamma_im};
    const Cx jf{a.J[0][e], a.J[1][e]};
    Cx hx = cscale(jf, tau);
    const bool diag = c == i, rhs = c == 0;
    if (diag || rhs) {
        const int64_t k = p * a.n + i;
        const Cx x{a.x[0][k], a.x[1][k]};
        const int d = a.deg[i];
        const Cx xd1 = cpow(x, d - 1);
        if (diag) hx = cadd(hx, cscale(cmul(gamma, cscale(xd1, (double)d)), 1.0 - tau));
        if (rhs) {
            const Cx g = csub(cmul(xd1, x), Cx{1.0, 0.0});
            const Cx f{a.f[0][k], a.f[1][k]};
            const Cx gg = cmul(gamma, g);
            // predictor: H_t = F - gamma G; corrector: H = tau F + (1 - tau) gamma G
            const Cx r = predict ? csub(f, gg) : cadd(cscale(f, tau), cscale(gg, 1.0 - tau));
            a.r[0][k] = r.re;
            a.r[1][k] = r.im;
        }
    }
    a.J[0][e] = hx.re;
    a.J[1][e] = hx.im;
}

// Columns K .. n-1 of the Gauss-Jordan elimination of track_small_kernel: lane
// r holds row r (r < n <= NB <= 16) and its right-hand side b.  prow holds
// the pivot row and its right-hand side.  False at a zero or non-finite
// pivot (the same on every lane).  Written by recursion, so that every
// column index is a constant and the rows stay in registers.
template <int NB, int K>
__device__ __forceinline__ bool wave_gauss_jordan(int n, int lane, Cx (&row)[NB], Cx &b, double2 *prow, Cx &inv,
                                                  int &col)
{
    if constexpr (K < NB) {
        if (K >= n) return true;
        double m = lane < n && col < 0 ? fabs(row[K].re) + fabs(row[K].im) : -1.0;
        if (!(m >= 0.0)) m = -1.0;
        double g = m;  // rows are in the first 16 lanes
        g = fmax(g, xor_lane_d<1>(g));
        g = fmax(g, xor_lane_d<2>(g));
        g = fmax(g, xor_lane_d<4>(g));
        g = fmax(g, xor_lane_d<8>(g));
        g = __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(g)),
                             __builtin_amdgcn_readfirstlane(__double2loint(g)));
        if (!(g > 0.0 && isfinite(g))) return false;
        const int pl = __ffsll((unsigned long long)__ballot(m == g)) - 1;
        if (lane == pl) {
#pragma unroll
            for (int c = K; c < NB; ++c)
                if (c < n) prow[c] = make_double2(row[c].re, row[c].im);
            prow[NB] = make_double2(b.re, b.im);
        }
        __syncthreads();
        // 1 / pivot, as the elimination kernels form it
        const double2 pv = prow[K];
        const double sc = fmax(fabs(pv.x), fabs(pv.y));
        const double sr = pv.x / sc, si = pv.y / sc, den = sc * (sr * sr + si * si);
        const Cx iv{sr / den, -si / den};
        Cx l = cmul(row[K], iv);
        if (lane == pl) {
            l = {0.0, 0.0};
            inv = iv;
            col = K;
        }
#pragma unroll
        for (int c = K + 1; c < NB; ++c)
            if (c < n) {
                const double2 q = prow[c];
                row[c].re = fma(-l.re, q.x, fma(l.im, q.y, row[c].re));
                row[c].im = fma(-l.re, q.y, fma(-l.im, q.x, row[c].im));
            }
        const double2 q = prow[NB];
        b.re = fma(-l.re, q.x, fma(l.im, q.y, b.re));
        b.im = fma(-l.re, q.y, fma(-l.im, q.x, b.im));
        __syncthreads();
        return wave_gauss_jordan<NB, K + 1>(n, lane, row, b, prow, inv, col);
    }
    return true;
}

// Sum of the terms get(0 .. len-1) as 2^LV lanes of the general kernel's
// summation add them: lane j takes every 2^LV-th term from j on, even and odd
// ones apart, and a butterfly adds the lanes (absent ones hold zero, which
// changes nothing).
template <int LV, class Get>
__device__ __forceinline__ Cx lanes_sum(const Get &get, int first, int len, int S)
{
    if constexpr (LV == 0) {
        Cx s0 = get(first), s1 = first + S < len ? get(first + S) : Cx{0.0, 0.0};
        int i = first + 2 * S;
        for (; i + S < len; i += 2 * S) {
            s0 = cadd(s0, get(i));
            s1 = cadd(s1, get(i + S));
        }
        if (i < len) s0 = cadd(s0, get(i));
        return cadd(s0, s1);
    } else {
        constexpr int half = 1 << (LV - 1);
        Cx v = lanes_sum<LV - 1>(get, first, len, S);
        if (half < S && first + half < len) v = cadd(v, lanes_sum<LV - 1>(get, first + half, len, S));
        return v;
    }
}

template <int CC>
struct SlotX {
    Arith64::C v[CC];
    __device__ __forceinline__ Arith64::C operator()(int t) const { return v[t]; }
};
template <int CC>
struct SlotExps {
    uint32_t w[CC];
    __device__ __forceinline__ double operator()(int t) const { return (double)((w[t] >> kExpShift) + 1); }
};

// One wave per path, for systems of n <= NB <= 16 variables: the path's
// rounds one after another, nothing but the wave itself waiting for them.  In
// lockstep a round costs six launches and a copy to the host, 50 to 60 us
// whatever the number of paths, and the slowest path decides how many rounds
// there are.  Here a round is
//   1. the power table, then one lane per monomial, then one lane per output
//      (see TrackTerms);
//   2. lane i takes row i of H_x and the right-hand side into registers;
//   3. Gauss-Jordan with partial pivoting across the lanes (largest
//      |re| + |im| of the rows not yet pivoted, the smallest row on ties):
//      the pivot row goes through LDS, read by all lanes at one address;
//   4. the predictor or corrector update, as step_kernel.
// Every operation and its order are those of the lockstep kernels, so paths
// come out the same bit for bit: near a limit (a residual's rounding next to
// the endgame's tolerance) any other rounding ends some path otherwise.
// Latency is the bound, all of it being one dependent chain; hence one wave,
// with no barriers, and one workgroup per path.  Quadrics, n = 10, all 1024
// paths with the endgame: 71.2 ms in lockstep, 11.1 ms here (11 to 16 by card;
// some 1170 rounds of the slowest path at 9 us).
template <int NB, int CC>
__global__ __launch_bounds__(64) void track_small_kernel(TrackArgs a, TrackTerms tt, int rounds)
{
    using C = Arith64::C;
    HIP_DYNAMIC_SHARED(double2, lds_raw)
    const int64_t p = blockIdx.x;
    if (a.status[p] != kRunning) return;
    const int n = a.n, np1 = n + 1, lane = (int)threadIdx.x;
    const int n_terms = tt.n_slots * CC, n_groups = tt.n_slots >> tt.log2VG;
    double2 *const tab = lds_raw;              // [R][n + 1] powers of x, column n = 1
    double2 *const coef = tab + tt.R * np1;    // [n_slots]
    double2 *const term = coef + tt.n_slots;   // [n_terms] derivatives, [n_groups] values
    double2 *const H = term + n_terms + n_groups;  // [n][n + 1] rows of J_F, then F
    double2 *const fold = H + n * np1;         // [n]
    double2 *const prow = fold + n;            // [kTrackSmallVars + 1] pivot row, right-hand side
    double2 *const sol = prow + kTrackSmallVars + 1;  // [kTrackSmallVars] solution
    uint32_t *const word = reinterpret_cast<uint32_t *>(sol + kTrackSmallVars);
    uint16_t *const out = reinterpret_cast<uint16_t *>(word + n_terms);
    uint16_t *const start = out + tt.n_out;
    uint16_t *const run = start + tt.n_out + 1;
    for (int i = lane; i < tt.n_slots; i += 64) coef[i] = make_double2(tt.coef[2 * i], tt.coef[2 * i + 1]);
    for (int i = lane; i < n_terms; i += 64) word[i] = tt.word[i];
    for (int i = lane; i < tt.n_out; i += 64) out[i] = tt.out[i];
    for (int i = lane; i <= tt.n_out; i += 64) start[i] = tt.start[i];
    for (int i = lane; i < tt.n_run; i += 64) run[i] = tt.run[i];
    for (int i = lane; i < n; i += 64) fold[i] = make_double2(tt.fold[2 * i], tt.fold[2 * i + 1]);
    for (int i = lane; i < n * np1; i += 64) H[i] = make_double2(0.0, 0.0);
    for (int i = lane; i < tt.R; i += 64) tab[i * np1 + n] = make_double2(1.0, 0.0);

    const bool mine = lane < n;  // lane i: variable i and row i
    const int64_t k0 = p * n + (mine ? lane : 0);
    Cx x{a.x[0][k0], a.x[1][k0]}, xs{a.xs[0][k0], a.xs[1][k0]};
    const int deg = a.deg[mine ? lane : 0];
    const Cx gamma{a.gamma_re, a.gamma_im};
    double t = a.t[p], t1 = a.t1[p], h = a.h[p];
    int ph = a.phase[p], succ = a.succ[p], steps = a.steps[p];
    int32_t status = kRunning;

    for (int round = 0; round < rounds && status == kRunning; ++round) {
        // 1. F and its Jacobian at x
        if (mine) {
            const C x1{x.re, x.im};
            C xr = x1;
            tab[lane] = make_double2(xr.re, xr.im);
            for (int r = 1; r < tt.R; ++r) {
                xr = Arith64::mul(xr, x1);
                tab[r * np1 + lane] = make_double2(xr.re, xr.im);
            }
        }
        __syncthreads();
        // whole waves: the values are added across lanes
        for (int i0 = 0; i0 < tt.n_slots; i0 += 64) {
            const bool on = i0 + lane < tt.n_slots;
            const int i = on ? i0 + lane : 0;
            SlotX<CC> xv;
            SlotExps<CC> ev;
            C cf, D[CC], V;
#pragma unroll
            for (int u = 0; u < CC; ++u) {
                ev.w[u] = word[i * CC + u];
                const int pos = (int)(ev.w[u] & kPosMask), em1 = (int)(ev.w[u] >> kExpShift);
                const double2 v = tab[pos], w = tab[em1 == 0 ? n : (em1 - 1) * np1 + pos];
                xv.v[u] = {v.x, v.y};
                cf = u == 0 ? C{w.x, w.y} : Arith64::mul(cf, C{w.x, w.y});
            }
            const C c{on ? coef[i].x : 0.0, on ? coef[i].y : 0.0};
            monomial_terms<Arith64, CC>(xv, cf, ev, c, SoloGroup(), D, V);
            for (int d = 1; d < (1 << tt.log2VG); d <<= 1) V = sum_xor_c<Arith64>(V, d);
            if (on) {
#pragma unroll
                for (int u = 0; u < CC; ++u) term[i * CC + u] = make_double2(D[u].re, D[u].im);
                if ((i & ((1 << tt.log2VG) - 1)) == 0)
                    term[n_terms + (i >> tt.log2VG)] = make_double2(V.re, V.im);
            }
        }
        __syncthreads();
        for (int o = lane; o < tt.n_out; o += 64) {
            const int first = start[o], len = start[o + 1] - first, id = out[o];
            const Cx v = lanes_sum<4>(
                [&](int q) {
                    const double2 u = term[run[first + q]];
                    return Cx{u.x, u.y};
                },
                0, len, 1 << tt.log2S);
            // the accumulator starts at zero, a value's at a folded constant
            const int row = id / np1;
            const double2 f0 = id - row * np1 == n ? fold[row] : make_double2(0.0, 0.0);
            H[id] = make_double2(f0.x + v.re, f0.y + v.im);
        }
        __syncthreads();
        // 2. row `lane` of H_x and its right-hand side (see homotopy_kernel)
        const bool predict = ph == 0;
        const double tau = predict ? t : t1;
        Cx row[NB], b{0.0, 0.0};
#pragma unroll
        for (int c = 0; c < NB; ++c) row[c] = {0.0, 0.0};
        if (mine) {
#pragma unroll
            for (int c = 0; c < NB; ++c)
                if (c < n) {
                    const double2 v = H[lane * np1 + c];
                    row[c] = cscale(Cx{v.x, v.y}, tau);
                }
            const double2 fv = H[lane * np1 + n];
            const Cx xd1 = cpow(x, deg - 1);
            const Cx dg = cscale(cmul(gamma, cscale(xd1, (double)deg)), 1.0 - tau);
#pragma unroll
            for (int c = 0; c < NB; ++c)
                if (c == lane) row[c] = cadd(row[c], dg);
            const Cx gg = cmul(gamma, csub(cmul(xd1, x), Cx{1.0, 0.0}));
            const Cx f{fv.x, fv.y};
            b = predict ? csub(f, gg) : cadd(cscale(f, tau), cscale(gg, 1.0 - tau));
        }
        // 3. Gauss-Jordan
        Cx inv{0.0, 0.0};  // 1 / pivot of the lane's row
        int col = -1;      // the column its row was the pivot of
        if (!wave_gauss_jordan<NB, 0>(n, lane, row, b, prow, inv, col)) {
            status = 2;
            break;
        }
        if (col >= 0) {
            const Cx d = cmul(b, inv);
            sol[col] = make_double2(d.re, d.im);
        }
        __syncthreads();
        // 4. the update (see step_kernel)
        const Cx d = mine ? Cx{sol[lane].x, sol[lane].y} : Cx{0.0, 0.0};
        const double hh = fmin(h, 1.0 - t);
        if (mine) x = predict ? csub(x, cscale(d, hh)) : csub(x, d);
        const bool finite = __all(!mine || (isfinite(x.re) && isfinite(x.im)));
        if (predict) {
            t1 = hh >= 1.0 - t ? 1.0 : t + hh;
            ph = 1;
            ++steps;
            if (!finite) status = 3;
        } else {
            double nd = mine ? hypot(d.re, d.im) : 0.0, nx = mine ? hypot(x.re, x.im) : 0.0;
            nd = fmax(nd, xor_lane_d<1>(nd));
            nx = fmax(nx, xor_lane_d<1>(nx));
            nd = fmax(nd, xor_lane_d<2>(nd));
            nx = fmax(nx, xor_lane_d<2>(nx));
            nd = fmax(nd, xor_lane_d<4>(nd));
            nx = fmax(nx, xor_lane_d<4>(nx));
            nd = fmax(nd, xor_lane_d<8>(nd));
            nx = fmax(nx, xor_lane_d<8>(nx));
            // rows are in the first 16 lanes: the first lane's answer
            const bool close = __builtin_amdgcn_readfirstlane((int)(nd <= a.corr_tol * (1.0 + nx))) != 0;
            if (!finite) {
                status = 3;
            } else if (close) {
                xs = x;
                t = t1;
                if (++succ >= 3) {
                    h = fmin(2.0 * h, a.h_max);
                    succ = 0;
                }
                ph = 0;
                if (t >= 1.0) status = 0;
            } else if (ph >= a.corr_iters) {
                x = xs;
                h = 0.5 * h;
                succ = 0;
                ph = 0;
                if (h < a.h_min) status = kTrackStepUnderflow;
            } else {
                ++ph;
            }
        }
        if (status == kRunning && ph == 0 && steps >= a.max_steps) status = kTrackStepLimit;
    }
    if (mine) {
        a.x[0][k0] = x.re;
        a.x[1][k0] = x.im;
        a.xs[0][k0] = xs.re;
        a.xs[1][k0] = xs.im;
    }
    if (lane == 0) {
        a.t[p] = t;
        a.t1[p] = t1;
        a.h[p] = h;
        a.phase[p] = ph;
        a.succ[p] = succ;
        a.steps[p] = steps;
        if (status == kRunning)
            atomicAdd(a.running, 1);
        else
            a.status[p] = status;
    }
}

// One wave per path.
__global__ __launch_bounds__(64) void step_kernel(TrackArgs a)
{
    const int64_t p = blockIdx.x;
    if (a.status[p] != kRunning) return;
    const int lane = threadIdx.x;
    const int n = a.n;
    const int64_t base = p * n;
    const int ph = a.phase[p];
    bool finite = true;
    int32_t status = kRunning;
    if (ph == 0) {
        // Euler predictor: dx/dt = -v with H_x v = H_t
        const double t = a.t[p];
        const double hh = fmin(a.h[p], 1.0 - t);
        for (int i = lane; i < n; i += 64) {
            const int64_t k = base + i;
            const double re = a.x[0][k] - hh * a.d[0][k];
            const double im = a.x[1][k] - hh * a.d[1][k];
            finite = finite && isfinite(re) && isfinite(im);
            a.x[0][k] = re;
            a.x[1][k] = im;
        }
        finite = __all(finite);
        if (lane == 0) {
            a.t1[p] = hh >= 1.0 - t ? 1.0 : t + hh;
            a.phase[p] = 1;
            a.steps[p] += 1;
            if (!finite) status = 3;
        }
    } else {
        // Newton corrector iteration ph at t1
        double nd = 0.0, nx = 0.0;
        for (int i = lane; i < n; i += 64) {
            const int64_t k = base + i;
            const double dre = a.d[0][k], dim = a.d[1][k];
            const double re = a.x[0][k] - dre, im = a.x[1][k] - dim;
            finite = finite && isfinite(re) && isfinite(im);
            a.x[0][k] = re;
            a.x[1][k] = im;
            nd = fmax(nd, hypot(dre, dim));
            nx = fmax(nx, hypot(re, im));
        }
        for (int off = 32; off >= 1; off >>= 1) {
            nd = fmax(nd, __shfl_xor(nd, off, 64));
            nx = fmax(nx, __shfl_xor(nx, off, 64));
        }
        finite = __all(finite);
        int decision;  // 0 continue, 1 accept, 2 reject
        if (!finite)
            decision = 3;
        else if (nd <= a.corr_tol * (1.0 + nx))
            decision = 1;
        else if (ph >= a.corr_iters)
            decision = 2;
        else
            decision = 0;
        if (decision == 1) {
            for (int i = lane; i < n; i += 64) {
                const int64_t k = base + i;
                a.xs[0][k] = a.x[0][k];
                a.xs[1][k] = a.x[1][k];
            }
        } else if (decision == 2) {
            for (int i = lane; i < n; i += 64) {
                const int64_t k = base + i;
                a.x[0][k] = a.xs[0][k];
                a.x[1][k] = a.xs[1][k];
            }
        }
        if (lane == 0) {
            if (decision == 3) {
                status = 3;
            } else if (decision == 1) {
                const double t = a.t1[p];
                a.t[p] = t;
                int s = a.succ[p] + 1;
                if (s >= 3) {
                    a.h[p] = fmin(2.0 * a.h[p], a.h_max);
                    s = 0;
                }
                a.succ[p] = s;
                a.phase[p] = 0;
                if (t >= 1.0) status = 0;
            } else if (decision == 2) {
                const double h = 0.5 * a.h[p];
                a.h[p] = h;
                a.succ[p] = 0;
                a.phase[p] = 0;
                if (h < a.h_min) status = kTrackStepUnderflow;
            } else {
                a.phase[p] = ph + 1;
            }
        }
    }
    if (lane == 0) {
        if (status == kRunning && a.phase[p] == 0 && a.steps[p] >= a.max_steps)
            status = kTrackStepLimit;
        if (status != kRunning)
            a.status[p] = status;
        else
            atomicAdd(a.running, 1);
    }
}

__global__ void endgame_kernel(int64_t n_paths, int32_t *tracked, int32_t *status)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n_paths) return;
    const bool done = status[p] == 0;
    tracked[p] = done ? 1 : 0;
    if (done) status[p] = kRunning;
}

__global__ void end_kernel(int64_t n_paths, const int32_t *tracked, int32_t *status)
{
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n_paths) return;
    if (tracked[p] && status[p] != 0) status[p] = kTrackEndgameFailed;
}

unsigned blocks_for(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

hipError_t launch_track_start(int64_t first, int64_t n_paths, int32_t n, const int32_t *deg,
                              double *const x[4], hipStream_t stream)
{
    if (n_paths <= 0) return hipSuccess;
    hipLaunchKernelGGL(start_kernel, dim3(blocks_for(n_paths, 256)), dim3(256), 0, stream, first,
                       n_paths, n, deg, x[0], x[1], x[2], x[3]);
    return hipGetLastError();
}

hipError_t launch_track_init(const TrackArgs &a, double h_init, double *const xlo[2],
                             hipStream_t stream)
{
    const int64_t total = a.n_paths * a.n;
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(init_kernel, dim3(blocks_for(total, 256)), dim3(256), 0, stream, a, h_init,
                       xlo[0], xlo[1]);
    return hipGetLastError();
}

hipError_t launch_track_homotopy(const TrackArgs &a, hipStream_t stream)
{
    const int64_t total = a.n_paths * (int64_t)a.n * a.n;
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(homotopy_kernel, dim3(blocks_for(total, 256)), dim3(256), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_track_step(const TrackArgs &a, hipStream_t stream)
{
    if (a.n_paths <= 0) return hipSuccess;
    hipLaunchKernelGGL(step_kernel, dim3((unsigned)a.n_paths), dim3(64), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_track_small(const TrackArgs &a, const TrackTerms &tt, int rounds, hipStream_t stream)
{
    if (a.n_paths <= 0) return hipSuccess;
    const size_t lds = track_small_lds(a.n, tt);
    const dim3 grid((unsigned)a.n_paths), block(64);
#define PE_CASE(NBV, CCV)                                                                          \
    if (a.n <= NBV && tt.CC == CCV) {                                                              \
        hipLaunchKernelGGL((track_small_kernel<NBV, CCV>), grid, block, lds, stream, a, tt, rounds); \
        return hipGetLastError();                                                                  \
    }
    PE_CASE(4, 2) PE_CASE(8, 2) PE_CASE(12, 2) PE_CASE(kTrackSmallVars, 2)
    PE_CASE(4, 4) PE_CASE(8, 4) PE_CASE(12, 4) PE_CASE(kTrackSmallVars, 4)
    PE_CASE(4, 8) PE_CASE(8, 8) PE_CASE(12, 8) PE_CASE(kTrackSmallVars, 8)
#undef PE_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_track_endgame(int64_t n_paths, int32_t *tracked, int32_t *status,
                                hipStream_t stream)
{
    if (n_paths <= 0) return hipSuccess;
    hipLaunchKernelGGL(endgame_kernel, dim3(blocks_for(n_paths, 256)), dim3(256), 0, stream,
                       n_paths, tracked, status);
    return hipGetLastError();
}

hipError_t launch_track_end(int64_t n_paths, const int32_t *tracked, int32_t *status,
                            hipStream_t stream)
{
    if (n_paths <= 0) return hipSuccess;
    hipLaunchKernelGGL(end_kernel, dim3(blocks_for(n_paths, 256)), dim3(256), 0, stream, n_paths,
                       tracked, status);
    return hipGetLastError();
}

}  // namespace pe
