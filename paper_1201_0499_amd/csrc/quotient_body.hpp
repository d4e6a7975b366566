// Device code of the quotient evaluation (quotient.hip describes it), shared
// by its kernels and by the single-launch kernel of small.hip.
//
// The arithmetic A is a policy of dd.hpp / qd.hpp for one point, or
// PointsF64<T>: T points side by side in FP64, which share every index,
// address and exponent of the tables.
#pragma once

#include <algorithm>

#include "dd.hpp"
#include "device.hpp"
#include "packing.hpp"
#include "quotient_args.hpp"

namespace pe {

// Entry of a table that no kernel writes, at an address that is the same on
// every lane: read through the scalar cache into scalar registers.  Read as
// ordinary memory, which the kernel's stores might change, it would sit in a
// vector register of every lane.
__device__ __forceinline__ int4 uniform_int4(const int4 *p)
{
    typedef int V __attribute__((ext_vector_type(4)));
    const V v = *(const __attribute__((address_space(4))) V *)p;
    return make_int4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ int2 uniform_int2(const int2 *p)
{
    typedef int V __attribute__((ext_vector_type(2)));
    const V v = *(const __attribute__((address_space(4))) V *)p;
    return make_int2(v.x, v.y);
}

// A whole structure of such memory, of 4-byte words.
template <class S>
__device__ __forceinline__ S uniform_struct(const S *p)
{
    static_assert(sizeof(S) % 4 == 0, "words");
    const auto *src = (const __attribute__((address_space(4))) uint32_t *)p;
    uint32_t w[sizeof(S) / 4];
#pragma unroll
    for (size_t i = 0; i < sizeof(S) / 4; ++i) w[i] = src[i];
    S s;
    __builtin_memcpy(&s, w, sizeof(S));
    return s;
}

// ---------------------------------------------------------------------------
// T points in FP64
// ---------------------------------------------------------------------------

template <int T>
struct PointsF64 {
    struct C {
        Arith64::C v[T];
    };
    template <class F>
    __device__ __forceinline__ static C each(const F &f)
    {
        C r;
#pragma unroll
        for (int t = 0; t < T; ++t) r.v[t] = f(t);
        return r;
    }
    __device__ __forceinline__ static C zero()
    {
        return each([](int) { return Arith64::zero(); });
    }
    __device__ __forceinline__ static C one()
    {
        return each([](int) { return Arith64::one(); });
    }
    __device__ __forceinline__ static C mul(const C &a, const C &b)
    {
        return each([&](int t) { return Arith64::mul(a.v[t], b.v[t]); });
    }
    __device__ __forceinline__ static C sum(const C &a, const C &b)
    {
        return each([&](int t) { return Arith64::sum(a.v[t], b.v[t]); });
    }
};

// T arrays of 16-byte values: the packer spreads the entries that 16 lanes
// read together over the banks (quotient_tables.cpp), for any array of them
template <int T>
struct LdsVec<PointsF64<T>> {
    using C = typename PointsF64<T>::C;
    double2 *p;
    int count;
    __device__ __forceinline__ C get(int i) const
    {
        return PointsF64<T>::each([&](int t) {
            const double2 v = p[t * count + i];
            return Arith64::C{v.x, v.y};
        });
    }
    __device__ __forceinline__ void put(int i, const C &c) const
    {
#pragma unroll
        for (int t = 0; t < T; ++t) p[t * count + i] = make_double2(c.v[t].re, c.v[t].im);
    }
    __device__ __forceinline__ double2 *piece(int i) const { return p + i; }
    __device__ __forceinline__ static LdsVec at(double2 *raw, int count, double2 *&next)
    {
        next = raw + T * (size_t)count;
        return {raw, count};
    }
};

// What differs between one point and several: loads, stores, range checks,
// lane exchanges and sums over the wave.
template <class A>
struct Pts {
    using C = typename A::C;
    using One = A;
    static constexpr int T = 1;
    __device__ __forceinline__ static const typename A::C &at(const C &c, int) { return c; }
    __device__ __forceinline__ static typename A::C &at(C &c, int) { return c; }
    __device__ __forceinline__ static C all(const typename A::C &v) { return v; }
    template <int M>
    __device__ __forceinline__ static C sum_over(const C &v)
    {
        return sum_xor<A, M>(v);
    }
    __device__ __forceinline__ static C other(const C &v, int d) { return shfl_xor_c(v, d); }
};

template <int N>
struct Pts<PointsF64<N>> {
    using A = PointsF64<N>;
    using C = typename A::C;
    using One = Arith64;
    static constexpr int T = N;
    __device__ __forceinline__ static const Arith64::C &at(const C &c, int t) { return c.v[t]; }
    __device__ __forceinline__ static Arith64::C &at(C &c, int t) { return c.v[t]; }
    __device__ __forceinline__ static C all(const Arith64::C &v)
    {
        return A::each([&](int) { return v; });
    }
    template <int M>
    __device__ __forceinline__ static C sum_over(const C &v)
    {
        return A::each([&](int t) { return sum_xor<Arith64, M>(v.v[t]); });
    }
    __device__ __forceinline__ static C other(const C &v, int d)
    {
        return A::each([&](int t) { return shfl_xor_c(v.v[t], d); });
    }
};

// ---------------------------------------------------------------------------
// sums of a * V with a small integer a
// ---------------------------------------------------------------------------

template <class A>
struct RunAcc;

template <>
struct RunAcc<Arith64> {
    Arith64::C s;
    __device__ __forceinline__ void clear() { s = Arith64::zero(); }
    __device__ __forceinline__ void add(const Arith64::C &v, double a)
    {
        s.re = fma(a, v.re, s.re);
        s.im = fma(a, v.im, s.im);
    }
    __device__ __forceinline__ Arith64::C get() const { return s; }
};

template <int T>
struct RunAcc<PointsF64<T>> {
    using C = typename PointsF64<T>::C;
    RunAcc<Arith64> s[T];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int t = 0; t < T; ++t) s[t].clear();
    }
    __device__ __forceinline__ void add(const C &v, double a)
    {
#pragma unroll
        for (int t = 0; t < T; ++t) s[t].add(v.v[t], a);
    }
    __device__ __forceinline__ C get() const
    {
        return PointsF64<T>::each([&](int t) { return s[t].get(); });
    }
};

template <>
struct RunAcc<ArithDD> {
    DWAcc re, im;
    __device__ __forceinline__ void clear()
    {
        re = {0.0, 0.0};
        im = {0.0, 0.0};
    }
    // s + a v: a v.hi exactly as p + e, p into s by TwoSum, everything else
    // (of relative order u) into the FP64 compensation
    __device__ __forceinline__ static void one(DWAcc &s, const dd &v, double a)
    {
        const dd p = two_prod(a, v.hi);
        const dd t = two_sum(s.s, p.hi);
        s.s = t.hi;
        s.c = s.c + (t.lo + fma(a, v.lo, p.lo));
    }
    __device__ __forceinline__ void add(const ArithDD::C &v, double a)
    {
        one(re, v.re, a);
        one(im, v.im, a);
    }
    __device__ __forceinline__ ArithDD::C get() const { return {dw_acc_get(re), dw_acc_get(im)}; }
};

// Sums of the orders u^0 .. u^3, kept apart, and the rest: every term by
// TwoSum, whose errors join the next order.  The sums outgrow the terms, and
// so do their errors; only errors of order u^4 of the sums and u^3 a|v| u of a
// term are rounded.
template <>
struct RunAcc<ArithQD> {
    struct Sums {
        double s0, s1, s2, s3, s4;
    } re, im;
    __device__ __forceinline__ void clear()
    {
        re = {0.0, 0.0, 0.0, 0.0, 0.0};
        im = {0.0, 0.0, 0.0, 0.0, 0.0};
    }
    __device__ __forceinline__ static void one(Sums &s, const qd &v, double a)
    {
        const dd p0 = two_prod(a, v.x0), p1 = two_prod(a, v.x1), p2 = two_prod(a, v.x2);
        const dd t0 = two_sum(s.s0, p0.hi);
        const dd a1 = two_sum(p1.hi, p0.lo), b1 = two_sum(a1.hi, t0.lo), t1 = two_sum(s.s1, b1.hi);
        const dd a2 = two_sum(p2.hi, p1.lo), b2 = two_sum(a1.lo, b1.lo), c2 = two_sum(a2.hi, b2.hi);
        const dd d2 = two_sum(c2.hi, t1.lo), t2 = two_sum(s.s2, d2.hi);
        const dd a3 = two_sum(b2.lo, c2.lo), b3 = two_sum(d2.lo, t2.lo), c3 = two_sum(a3.hi, b3.hi);
        const dd d3 = two_sum(c3.hi, fma(a, v.x3, p2.lo) + a2.lo), t3 = two_sum(s.s3, d3.hi);
        s.s0 = t0.hi;
        s.s1 = t1.hi;
        s.s2 = t2.hi;
        s.s3 = t3.hi;
        s.s4 += ((a3.lo + b3.lo) + c3.lo) + (d3.lo + t3.lo);
    }
    __device__ __forceinline__ void add(const ArithQD::C &v, double a)
    {
        one(re, v.re, a);
        one(im, v.im, a);
    }
    __device__ __forceinline__ static qd sum(const Sums &s)
    {
        double e[5] = {s.s0, s.s1, s.s2, s.s3, s.s4};
        return distill<5>(e);
    }
    __device__ __forceinline__ ArithQD::C get() const { return {sum(re), sum(im)}; }
};

// 1 / x, an error of which every derivative by x would have whole
__device__ __forceinline__ Arith64::C quot_inv(const Arith64::C &x) { return Arith64::recip(x); }
__device__ __forceinline__ ArithDD::C quot_inv(const ArithDD::C &x) { return ArithDD::recip(x); }
// from the double-double reciprocal y, with e = 1 - x y of order 2^-103:
// y + y (e + e^2), the rest e^3
__device__ __forceinline__ ArithQD::C quot_inv(const ArithQD::C &x)
{
    const ArithDD::C d = ArithDD::inv({{x.re.x0, x.re.x1}, {x.im.x0, x.im.x1}});
    const ArithQD::C y{{d.re.hi, d.re.lo, 0.0, 0.0}, {d.im.hi, d.im.lo, 0.0, 0.0}};
    const ArithQD::C e = ArithQD::add(ArithQD::one(), ArithQD::neg(ArithQD::mul(x, y)));
    return ArithQD::add(y, ArithQD::mul(y, ArithQD::add(e, ArithQD::mul(e, e))));
}

__device__ __forceinline__ double lead_re(const Arith64::C &v) { return v.re; }
__device__ __forceinline__ double lead_im(const Arith64::C &v) { return v.im; }
__device__ __forceinline__ double lead_re(const ArithDD::C &v) { return v.re.hi; }
__device__ __forceinline__ double lead_im(const ArithDD::C &v) { return v.im.hi; }
__device__ __forceinline__ double lead_re(const ArithQD::C &v) { return v.re.x0; }
__device__ __forceinline__ double lead_im(const ArithQD::C &v) { return v.im.x0; }

__device__ __forceinline__ void make_nan(Arith64::C &v) { v.re = refused(); }
__device__ __forceinline__ void make_nan(ArithDD::C &v) { v.re.hi = refused(); }
__device__ __forceinline__ void make_nan(ArithQD::C &v) { v.re.x0 = refused(); }

// Distance of a value's exponent field (the larger part's high word without
// sign) above lo; span or more, as unsigned, means out of range.  Zero,
// infinities and NaN are always out.
template <class C>
__device__ __forceinline__ uint32_t range_pos(const C &v, uint32_t lo)
{
    const uint32_t r = (uint32_t)__double2hiint(lead_re(v)) & 0x7FFFFFFFu;
    const uint32_t i = (uint32_t)__double2hiint(lead_im(v)) & 0x7FFFFFFFu;
    return max(r, i) - lo;
}

constexpr uint32_t kProdLo = (uint32_t)(1023 - kProductExp) << 20;
constexpr uint32_t kProdSpan = (uint32_t)(2 * kProductExp) << 20;

// Farthest that a lane's products were from the range, per point.
template <class A>
struct Worst {
    uint32_t w[Pts<A>::T] = {};
    __device__ __forceinline__ void see(const typename A::C &v)
    {
#pragma unroll
        for (int t = 0; t < Pts<A>::T; ++t) w[t] = max(w[t], range_pos(Pts<A>::at(v, t), kProdLo));
    }
    __device__ __forceinline__ void mark(typename A::C &v) const
    {
#pragma unroll
        for (int t = 0; t < Pts<A>::T; ++t)
            if (w[t] >= kProdSpan) make_nan(Pts<A>::at(v, t));
    }
};

// x + 0: turns a negative zero into zero (an output without terms is +0)
__device__ __forceinline__ Arith64::C plus_zero(const Arith64::C &v) { return {v.re + 0.0, v.im + 0.0}; }
__device__ __forceinline__ ArithDD::C plus_zero(const ArithDD::C &v)
{
    return {{v.re.hi + 0.0, v.re.lo + 0.0}, {v.im.hi + 0.0, v.im.lo + 0.0}};
}
__device__ __forceinline__ ArithQD::C plus_zero(const ArithQD::C &v)
{
    return {{v.re.x0 + 0.0, v.re.x1 + 0.0, v.re.x2 + 0.0, v.re.x3 + 0.0},
            {v.im.x0 + 0.0, v.im.x1 + 0.0, v.im.x2 + 0.0, v.im.x3 + 0.0}};
}

// LDS of a workgroup (entries of one value, or of one for each point)
template <class A>
struct QuotLds {
    LdsVec<A> u;    // [D][n]: x^1 .. x^D; then, if the tables need it, the entry 1
    LdsVec<A> y;    // [n]: 1 / x
    LdsVec<A> V;    // [nbuf][CH]: monomial values
    LdsVec<A> acc;  // [n+1] sums over chunks (multi): J entries, then f
};

template <class A>
__device__ __forceinline__ QuotLds<A> quot_lds(double2 *raw, const QuotArgs &a, double2 *&next)
{
    QuotLds<A> l;
    double2 *p = raw;
    l.u = LdsVec<A>::at(p, a.D * a.n_vars + a.pad, p);
    l.y = LdsVec<A>::at(p, a.n_vars, p);
    l.V = LdsVec<A>::at(p, a.nbuf * a.CH, p);
    l.acc = LdsVec<A>::at(p, a.multi ? a.n_vars + 1 : 0, p);
    next = p;
    return l;
}

// The power table and the reciprocals of points pt .. pt+npt-1 (callers add
// the barrier).  A coordinate out of range becomes NaN in the table: the values
// of the polynomials that contain it then are NaN too.  With a.skip (SKIP: it
// may be set) also the wave's word of `words`, and the marks of those of the
// polynomials p, p + step, ... below p1 at such a point in which every variable
// occurs.  With a.sparse only the variables that share a block of ranks with
// one of polynomial p, the workgroup's only one: what no term reads stays
// unset, and what multiplies no terms is 1.
template <class A, bool SKIP>
__device__ __forceinline__ void quot_table(const QuotArgs &a, const QuotLds<A> &lds, int64_t pt, int npt, int p, int p1,
                                           int step, bool jac, uint32_t *words)
{
    using C = typename A::C;
    using P = Pts<A>;
    using One = typename P::One;
    const int n = a.n_vars, NT = (int)blockDim.x;
    int4 pl = make_int4(0, 0, 0, 0), ck = pl;
    int count = n;
    bool bad = false;
    if (a.sparse) {
        pl = uniform_int4(a.poly + p);
        if (pl.x == pl.y) return;
        ck = uniform_int4(a.chunk + pl.x);
        count = a.n_blk * kRankBlock;
    }
    for (int j = (int)threadIdx.x; j < count; j += NT) {
        int i = j;
        if (a.sparse) {
            i = (int)a.out[(int64_t)pl.x * count + j];
            if (i >= n) continue;
            if (a.block[ck.w + j / kRankBlock].y == 0) {
                if (jac) lds.y.put(i, A::one());
                continue;
            }
        }
        C x, y;
#pragma unroll
        for (int t = 0; t < P::T; ++t) {
            typename One::C v = Io<One>::load(a.x, (pt + min(t, npt - 1)) * n + i);
            P::at(y, t) = quot_inv(v);
            if (range_pos(v, a.x_lo) >= a.x_span) {
                make_nan(v);
                P::at(y, t) = One::one();
                bad = true;
            }
            P::at(x, t) = v;
        }
        lds.u.put(i, x);
        C xr = x;
        for (int r = 1; r < a.D; ++r) {
            xr = A::mul(xr, x);
            lds.u.put(r * n + i, xr);
        }
        if (jac) lds.y.put(i, y);
    }
    if (a.pad && threadIdx.x == 0) lds.u.put(a.D * n, A::one());
    if constexpr (SKIP && P::T == 1) {
        if (a.skip) {
            const bool any = __ballot(bad) != 0;
            if ((threadIdx.x & 63) == 0) words[threadIdx.x >> 6] = any;
            if (bad)
                for (int q = p; q < p1; q += step)
                    if (a.poly[q].w) a.f[0][pt * a.n_polys + q] = refused();
        }
    }
}

// Whether a coordinate of the point is out of range, after the table's barrier;
// with a.skip, else never.  Polynomials in which every variable occurs are then
// refused before the work on them (n = 128, m = 256, k = 16, d = 3, one
// coordinate zero at every point, double-double, the general kernel alone, the
// quotients and it, it after a look at the point: one point 16.8, 24.1 and 17.4
// us; 1000 points 5.8, 7.7 and 6.0 ms); the others after it, if they contain it.
// Not for two points in FP64, nor in batches, where the look costs every call 3%.
template <class A>
__device__ __forceinline__ bool bad_point(const QuotArgs &a, const uint32_t *words)
{
    if (Pts<A>::T > 1 || !a.skip) return false;
    const int lane = (int)threadIdx.x & 63;
    return __ballot(lane < (int)(blockDim.x >> 6) && words[lane] != 0) != 0;
}

// Where the words are: in the second buffer of values, if there is one, which
// nothing writes before the barrier after the first polynomial's values.
template <class A>
__device__ __forceinline__ uint32_t *wave_words(const QuotArgs &a, const QuotLds<A> &lds, double2 *end)
{
    return reinterpret_cast<uint32_t *>(a.nbuf > 1 ? lds.V.piece(a.CH) : end);
}

// Factors of one lane's monomial: the quads of words wp[0], wp[cnt], ...
// (Q of them) in the canonical order (quotient.hpp).  Checked after every
// product of quads: a factor there was checked, or is a quad, within the same
// range by the points' or (CHECK) checked itself.
template <class A, bool CHECK>
struct Factors {
    using C = typename A::C;
    const LdsVec<A> &u;
    const uint2 *wp;
    int cnt, Q, qs;  // stride between quads, quads, quads per range
    Worst<A> &worst;

    __device__ __forceinline__ Factors(const LdsVec<A> &table, const uint2 *words, int stride, int quads,
                                       Worst<A> &w)
        : u(table), wp(words), cnt(stride), Q(quads), qs((quads + kParts - 1) / kParts), worst(w)
    {
    }
    __device__ __forceinline__ C quad(const uint2 &w) const
    {
        const C u0 = u.get((int)(w.x & 0xFFFFu)), u1 = u.get((int)(w.x >> 16));
        const C u2 = u.get((int)(w.y & 0xFFFFu)), u3 = u.get((int)(w.y >> 16));
        const C v = A::mul(A::mul(u0, u1), A::mul(u2, u3));
        if (CHECK) worst.see(v);
        return v;
    }
    __device__ __forceinline__ bool has(int r) const { return r * qs < Q; }
    // product of range r (quads r qs .. ), which has at least one quad
    __device__ __forceinline__ C range(int r) const
    {
        const int j0 = r * qs, j1 = min(Q, j0 + qs);
        C p = quad(wp[(int64_t)j0 * cnt]);
        for (int j = j0 + 1; j < j1; ++j) {
            p = A::mul(p, quad(wp[(int64_t)j * cnt]));
            worst.see(p);
        }
        return p;
    }
    // product of all ranges by one lane
    __device__ __forceinline__ C all(bool pairs) const
    {
        // a quad of at most two factors, without its products by 1
        if (pairs) {
            if (Q == 0) return A::one();
            const uint2 w = *wp;
            const C v = A::mul(u.get((int)(w.x & 0xFFFFu)), u.get((int)(w.x >> 16)));
            if (CHECK) worst.see(v);
            return v;
        }
        C prod = A::one();
        for (int h = 0; h < 2 && has(2 * h); ++h) {
            C t = range(2 * h);
            if (has(2 * h + 1)) {
                t = A::mul(t, range(2 * h + 1));
                worst.see(t);
            }
            if (h == 0) {
                prod = t;
            } else {
                prod = A::mul(prod, t);
                worst.see(prod);
            }
        }
        return prod;
    }
};

// Values of the monomials of chunk ck into V at entry vo, one lane per
// monomial (ONE) or as many as the launch says.
template <class A, bool ONE, bool CHECK>
__device__ __forceinline__ void chunk_products(const QuotArgs &a, const int4 &ck, const QuotLds<A> &lds, int vo)
{
    using C = typename A::C;
    using P = Pts<A>;
    using One = typename P::One;
    const int log2L = ONE ? 0 : a.log2L, sub = (int)threadIdx.x & ((1 << log2L) - 1);
    const int items = ck.y << log2L;
    // whole waves take part (lane exchanges), so the trip count is uniform
    for (int w0 = (int)threadIdx.x & ~63; w0 < items; w0 += (int)blockDim.x) {
        const int s = (w0 + ((int)threadIdx.x & 63)) >> log2L;
        const bool on = s < ck.y;
        const int sl = __builtin_amdgcn_readfirstlane(s >> 6);
        const int2 sh = uniform_int2(a.slice + ck.z + sl);
        Worst<A> worst;
        const Factors<A, CHECK> fac(lds.u, a.words + (int64_t)sh.x + (on ? s - 64 * sl : 0), min(64, ck.y - 64 * sl),
                                    sh.y, worst);
        const typename One::C coef = Io<One>::coef(a.coef, (int64_t)ck.x + (on ? s : 0));
        C prod = A::one();
        if (log2L == 0) {
            prod = fac.all(a.pairs);
        } else {
            // ranges 2 sub, 2 sub + 1 of two lanes, or range sub of four; a
            // lower lane's product is the left factor, and only what reaches
            // the group's first lane counts
            const int r0 = log2L == 1 ? 2 * sub : sub;
            if (fac.has(r0)) {
                prod = fac.range(r0);
                if (log2L == 1 && fac.has(r0 + 1)) {
                    prod = A::mul(prod, fac.range(r0 + 1));
                    worst.see(prod);
                }
            }
            for (int d = 1; d < (1 << log2L); d <<= 1) {
                worst.mark(prod);  // so that the other lane learns of it
                prod = A::mul(prod, P::other(prod, d));
                worst.see(prod);
            }
        }
        prod = A::mul(prod, P::all(coef));
        worst.mark(prod);
        if (on && sub == 0) lds.V.put(vo + s, prod);
    }
}

// (a branch for each quad in the place of two loops costs 4% in FP64)
template <class A, bool ONE>
__device__ __forceinline__ void chunk_values(const QuotArgs &a, const int4 &ck, const QuotLds<A> &lds, int vo)
{
    if (a.check)
        chunk_products<A, ONE, true>(a, ck, lds, vo);
    else
        chunk_products<A, ONE, false>(a, ck, lds, vo);
}

// Sum over the wave, by a butterfly.
template <class A>
__device__ __forceinline__ typename A::C wave_sum(typename A::C v)
{
    using P = Pts<A>;
    v = P::template sum_over<1>(v);
    v = P::template sum_over<2>(v);
    v = P::template sum_over<4>(v);
    v = P::template sum_over<8>(v);
    v = P::template sum_over<16>(v);
    return P::template sum_over<32>(v);
}

// f_p (o == n) or df_p/dx_o at the live points from pt on.  on_refused() runs
// on the lane that finds a value refused.
template <class A, class Refused>
__device__ __forceinline__ void quot_store(const QuotArgs &a, int64_t pt, uint32_t live, int p, int o,
                                           const typename A::C &v, const Refused &on_refused)
{
    using P = Pts<A>;
    using One = typename P::One;
    const int n = a.n_vars;
#pragma unroll
    for (int t = 0; t < P::T; ++t) {
        if (P::T > 1 && !((live >> t) & 1u)) continue;
        const typename One::C w = P::at(v, t);
        if (o == n) {
            // a product out of range left a NaN among the values
            if (!isfinite(lead_re(w)) || !isfinite(lead_im(w))) {
                a.f[0][(pt + t) * a.n_polys + p] = refused();
                on_refused();
            } else {
                Io<One>::store(a.f, (pt + t) * a.n_polys + p, w);
            }
        } else {
            Io<One>::store(a.J, ((pt + t) * n + o) * a.n_polys + p, plus_zero(w));
        }
    }
}

// The value of polynomial p by one wave, without the Jacobian: lane l
// multiplies monomials l, l + 64, ... of a chunk and adds their values, then
// the wave adds the lanes; the same operations in the same order as
// chunk_values and chunk_sums.
template <class A, bool CHECK>
__device__ __forceinline__ void quot_value_of(const QuotArgs &a, const LdsVec<A> &u, int64_t pt, uint32_t live, int p)
{
    using C = typename A::C;
    using P = Pts<A>;
    using One = typename P::One;
    const int lane = (int)threadIdx.x & 63;
    const int4 pl = uniform_int4(a.poly + p);
    C f = pl.z > 0 ? P::all(Io<One>::coef(a.sys_coef, pl.z - 1)) : A::zero();
    for (int c = pl.x; c < pl.y; ++c) {
        const int4 ck = uniform_int4(a.chunk + c);
        RunAcc<A> acc;
        acc.clear();
        for (int sl = 0; 64 * sl < ck.y; ++sl) {
            const int2 sh = uniform_int2(a.slice + ck.z + sl);
            const int cnt = min(64, ck.y - 64 * sl);
            if (lane >= cnt) break;  // the chunk's last slice
            Worst<A> worst;
            const Factors<A, CHECK> fac(u, a.words + (int64_t)sh.x + lane, cnt, sh.y, worst);
            const typename One::C coef = Io<One>::coef(a.coef, (int64_t)ck.x + 64 * sl + lane);
            C v = A::mul(fac.all(a.pairs), P::all(coef));
            worst.mark(v);
            acc.add(v, 1.0);
        }
        const C v = wave_sum<A>(acc.get());
        f = c == pl.x && pl.z == 0 ? v : A::sum(f, v);
    }
    if (lane == 0) quot_store<A>(a, pt, live, p, a.n_vars, f, [] {});
}

template <class A>
__device__ __forceinline__ void quot_value(const QuotArgs &a, const LdsVec<A> &u, int64_t pt, uint32_t live,
                                           bool bad, int p)
{
    if (bad && uniform_int4(a.poly + p).w) return;  // marked with the table
    if (a.check)
        quot_value_of<A, true>(a, u, pt, live, p);
    else
        quot_value_of<A, false>(a, u, pt, live, p);
}

// Sum of a run by one lane's NP of its kParts partial sums, combined with
// the other lanes of the run.  e: the lane's entries of the run's first row.
template <class A, int NP>
__device__ __forceinline__ typename A::C run_sum(const LdsVec<A> &V, int vo, const uint16_t *e, int rows)
{
    using C = typename A::C;
    struct alignas(2 * NP) Row {
        uint16_t v[NP];
    };
    constexpr int kStep = kRankBlock * kParts;
    C part[NP];
    Row nx{};
    if (rows > 0) nx = *reinterpret_cast<const Row *>(e);
    for (int i0 = 0; i0 == 0 || i0 < rows; i0 += kRunBlock) {
        RunAcc<A> acc[NP];
#pragma unroll
        for (int q = 0; q < NP; ++q) acc[q].clear();
        const int i1 = min(rows, i0 + kRunBlock);
        for (int i = i0; i < i1; ++i) {
            const Row r = nx;
            e += kStep;
            if (i + 1 < rows) nx = *reinterpret_cast<const Row *>(e);
#pragma unroll
            for (int q = 0; q < NP; ++q)
                acc[q].add(V.get(vo + (int)(r.v[q] & ((1 << kEntryBits) - 1))),
                           (double)(r.v[q] >> kEntryBits));
        }
#pragma unroll
        for (int q = 0; q < NP; ++q) part[q] = i0 == 0 ? acc[q].get() : A::sum(part[q], acc[q].get());
    }
    if constexpr (NP == 4) return A::sum(A::sum(part[0], part[1]), A::sum(part[2], part[3]));
    if constexpr (NP == 2) return Pts<A>::template sum_over<1>(A::sum(part[0], part[1]));
    return Pts<A>::template sum_over<2>(Pts<A>::template sum_over<1>(part[0]));
}

// The sums of chunk ck (number ci): with jac the outputs' runs, and the sum
// of the values.  put(o, v) gets output o's sum on one lane.
template <class A, int NP, class Put>
__device__ __forceinline__ void chunk_sums(const QuotArgs &a, int ci, const int4 &ck, const QuotLds<A> &lds,
                                           int vo, bool jac, const Put &put)
{
    using C = typename A::C;
    constexpr int S = kParts / NP;
    const int lane = (int)threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int nw = (int)blockDim.x >> 6;
    const int n_rank = a.n_blk * kRankBlock;
    const int items = jac ? (n_rank * S + 63) / 64 : 0;  // waves' worth of runs
    for (int k = 0; k * nw <= items; ++k) {
        // waves in turn, backwards in odd rounds: the values' sum, the last
        // item, falls on a wave with short runs
        const int it = k * nw + ((k & 1) ? nw - 1 - wave : wave);
        if (it > items) continue;
        if (it < items) {
            const int rank = (it * 64 + lane) / S, sub = lane & (S - 1);
            const int blk = rank / kRankBlock;
            const bool on = rank < n_rank;
            const int2 bh = on ? a.block[ck.w + blk] : make_int2(0, 0);
            const uint16_t *e = a.runs + ((int64_t)bh.x * kRankBlock + (rank & (kRankBlock - 1))) * kParts +
                                sub * NP;
            const int o = on ? (int)a.out[(int64_t)ci * n_rank + rank] : 0xFFFF;
            const C v = run_sum<A, NP>(lds.V, vo, e, bh.y);
            if (sub == 0 && o != 0xFFFF) put(o, v);
        } else {
            // at most kMaxQuotChunk / 64 <= kRunBlock terms per lane
            RunAcc<A> acc;
            acc.clear();
            for (int i = lane; i < ck.y; i += 64) acc.add(lds.V.get(vo + i), 1.0);
            const C v = wave_sum<A>(acc.get());
            if (lane == 0) put(a.n_vars, v);
        }
    }
}

// Polynomial p at the points from pt on, of which those with their bit set in
// live are written (bad: see bad_point); vo is the buffer in use (it
// alternates).  FEW: lanes per monomial and per run as the launch says (calls
// of few workgroups); else one lane per monomial and two per run.  on_refused:
// see quot_store.
template <class A, bool FEW, class Refused>
__device__ __forceinline__ void quot_poly(const QuotArgs &a, const QuotLds<A> &lds, int64_t pt, uint32_t live,
                                          bool bad, int p, int &vo, bool jac, const Refused &on_refused)
{
    using C = typename A::C;
    using P = Pts<A>;
    using One = typename P::One;
    const int n = a.n_vars;
    const int4 pl = uniform_int4(a.poly + p);
    if (bad && pl.w) return;  // marked with the table
    for (int c = pl.x; c < pl.y; ++c) {
        const int4 ck = uniform_int4(a.chunk + c);
        chunk_values<A, !FEW>(a, ck, lds, vo);
        __syncthreads();
        const bool first = c == pl.x, last = c + 1 == pl.y;
        auto put = [&](int o, C v) {
            if (!first)
                v = A::sum(lds.acc.get(o), v);
            else if (o == n && pl.z > 0)
                v = A::sum(P::all(Io<One>::coef(a.sys_coef, pl.z - 1)), v);
            if (!last) {
                lds.acc.put(o, v);
                return;
            }
            if (o != n) v = A::mul(lds.y.get(o), v);
            quot_store<A>(a, pt, live, p, o, v, on_refused);
        };
        if (!FEW || a.log2S == 1)
            chunk_sums<A, 2>(a, c, ck, lds, vo, jac, put);
        else if (a.log2S == 0)
            chunk_sums<A, 4>(a, c, ck, lds, vo, jac, put);
        else
            chunk_sums<A, 1>(a, c, ck, lds, vo, jac, put);
        // with two buffers the next item writes the other one; it comes back
        // to this one only after a barrier that follows these reads
        if (a.nbuf > 1)
            vo = vo ? 0 : a.CH;
        else
            __syncthreads();
    }
    if (pl.x == pl.y) {
        // no monomials but a folded constant, or none at all
        for (int t = 0; t < P::T; ++t) {
            if (P::T > 1 && !((live >> t) & 1u)) continue;
            if (threadIdx.x == 0)
                Io<One>::store(a.f, (pt + t) * a.n_polys + p,
                               pl.z > 0 ? Io<One>::coef(a.sys_coef, pl.z - 1) : One::zero());
            if (jac)
                for (int o = (int)threadIdx.x; o < n; o += (int)blockDim.x)
                    Io<One>::store(a.J, ((pt + t) * n + o) * a.n_polys + p, One::zero());
        }
    }
}

}  // namespace pe
