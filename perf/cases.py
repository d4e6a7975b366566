"""Timed cases: what a program that uses the library asks of it.

Every case goes through the public binding (System, Batch) with the library's
own choice of schedule, the way a program that has not tuned anything calls
it.  The sizes are those of this repository's workloads and of the ranges
around them: n = 8 to 512 variables, m = 8 to 1024 monomials per polynomial,
k = 1 to 32 variables per monomial, exponents up to 5, one point to about a
thousand, in complex FP64, double-double and quad-double.

A system is regular (every monomial has k variables) or ragged (each monomial
draws its number of variables from 1..k, and the last one of every polynomial
is a constant).  Coefficients and points lie on the unit circle and carry
random low words.  Newton's systems get one constant per polynomial that puts
a root at a generic unit-circle point; starts are 1e-6 away from it.

Left out of what a case returns: the residual norms of the corrector and the
tracker, which at convergence are rounding noise below the tolerance that the
status already reports, and the tracker's step counts, which rounding decides
(the tracker's tests do not compare them either).
"""
import math

import numpy as np
import torch

import paper_1201_0499_amd as pe

DEV = "cuda"


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # one evaluation of a small system: latency of a single call
        dict(name="eval_dd_tiny", kind="eval", prec="dd", n=8, m=8, k=4, d=2, P=1, ragged=False),
        # one point of a system of the paper's scale, as inside one path's predictor-corrector
        dict(name="eval_dd_point", kind="eval", prec="dd", n=128, m=256, k=16, d=3, P=1, ragged=False),
        # the same in quad-double, for paths that need more than 32 digits
        dict(name="eval_qd_point", kind="eval", prec="qd", n=128, m=256, k=16, d=3, P=1, ragged=False),
        # many points of an uneven system in FP64: the Jacobians of a tracker's paths
        dict(name="eval_f64_points", kind="eval", prec="f64", n=100, m=201, k=16, d=4, P=1000, ragged=True),
        # the largest evaluation of one GPU: the benchmark's headline
        dict(name="eval_dd_large", kind="eval", prec="dd", n=512, m=1024, k=32, d=5, P=256, ragged=False),
        # residuals only (no Jacobian) of an uneven system at many points
        dict(name="values_dd", kind="values", prec="dd", n=150, m=300, k=12, d=4, P=333, ragged=True),
        # many uneven systems in one launch
        dict(name="batch_dd", kind="batch", prec="dd", systems=24, n=160, m=512, k=16, d=4, P=24),
        # the corrector from many starts, mixed precision, paper scale
        dict(name="newton_mixed", kind="newton", mode="mixed", n=128, m=256, k=16, d=3, P=1024, tol=1e-28),
        # the corrector entirely in double-double, an odd size
        dict(name="newton_dd", kind="newton", mode="dd", n=100, m=150, k=8, d=3, P=256, tol=1e-28),
        # the corrector to quad-double accuracy
        dict(name="newton_qd", kind="newton", mode="qd", n=64, m=128, k=8, d=3, P=256, tol=1e-56),
        # the corrector on a system whose elimination no longer fits the registers of a workgroup
        dict(name="newton_mixed_large", kind="newton", mode="mixed", n=400, m=600, k=24, d=4, P=128, tol=1e-26),
        # all paths of a system of quadrics, with the double-double endgame
        dict(name="track", kind="track", n=10, P=1024),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges, at most as dear as the largest listed one."""
    kind = rng.choice(["eval", "eval", "eval", "values", "batch", "newton", "newton", "track"])
    d = rng.randint(1, 5)
    if kind == "track":
        n = rng.randint(3, 10)
        return dict(kind="track", n=n, P=rng.randint(2 ** (n - 1), 2 ** n))
    if kind == "batch":
        n = _log(rng, 24, 160)
        return dict(kind="batch", prec=rng.choice(["dd", "f64"]), systems=rng.randint(3, 24), n=n,
                    m=_log(rng, 24, 512), k=rng.randint(3, 16), d=max(d, 2), P=_log(rng, 1, 24))
    if kind == "newton":
        mode = rng.choice(["mixed", "mixed", "dd", "qd"])
        n = _log(rng, 12, 96 if mode == "qd" else 400)
        k = rng.randint(4, min(24, n // 2))
        P = _log(rng, 8, 256 if mode == "mixed" and n <= 128 else 64)
        return dict(kind="newton", mode=mode, n=n, m=_log(rng, max(16, n // 2), 300), k=k, d=min(d + 1, 4),
                    P=P, tol=1e-56 if mode == "qd" else 1e-26)
    prec = rng.choice(["dd", "dd", "f64", "qd"]) if kind == "eval" else rng.choice(["dd", "f64"])
    n = _log(rng, 8, 128 if prec == "qd" else 512)
    m = _log(rng, 8, 1024)
    k = rng.randint(2, min(32 if prec != "qd" else 16, n))
    top = (1 << 27) if prec == "qd" else (1 << 32)
    P = min(_log(rng, 1, 1024), max(1, top // (n * m * k)), max(1, (1 << 26) // (n * n)))
    return dict(kind=kind, prec=prec, n=n, m=m, k=k, d=min(d, 3) if prec == "qd" else d, P=P,
                ragged=bool(rng.getrandbits(1)))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _low(g, hi):
    """Low words, uniform within half an ulp of hi."""
    ulp = torch.ldexp(torch.ones_like(hi), torch.frexp(hi).exponent - 53)
    return (torch.rand(hi.shape, generator=g, device=DEV, dtype=torch.float64) - 0.5) * ulp


def _unit(g, shape, words=2):
    """Unit-circle values: `words` planes of the real part, then of the imaginary part."""
    th = torch.rand(shape, generator=g, device=DEV, dtype=torch.float64) * (2 * math.pi)
    out = []
    for hi in (torch.cos(th), torch.sin(th)):
        out.append(hi)
        for _ in range(words - 1):
            out.append(_low(g, out[-1]))
    return out


def _subsets(g, rows, n, k):
    """Uniform random k-subsets of range(n), sorted."""
    if 2 * k > n:
        return torch.rand((rows, n), generator=g, device=DEV).argsort(dim=1)[:, :k].sort(dim=1).values
    out = torch.randint(0, n, (rows, k), generator=g, device=DEV).sort(dim=1).values
    while True:
        bad = (out[:, 1:] == out[:, :-1]).any(dim=1).nonzero().flatten()
        if bad.numel() == 0:
            return out
        out[bad] = torch.randint(0, n, (bad.numel(), k), generator=g, device=DEV).sort(dim=1).values


class _Sys:
    """A square system: per monomial k padded variables and exponents (exponent 0 = absent)."""

    def __init__(self, g, n, m, k, d, ragged=False, constant=None):
        self.n, self.m, self.k, self.d = n, m + (constant is not None), k, d
        pos = _subsets(g, n * m, n, k).reshape(n, m, k)
        ex = torch.randint(1, d + 1, (n, m, k), generator=g, device=DEV)
        if ragged:
            size = torch.randint(1, k + 1, (n, m, 1), generator=g, device=DEV)
            size[:, -1] = 0
            ex = torch.where(torch.arange(k, device=DEV) < size, ex, 0)
        self.coef = [c.reshape(n, m) for c in _unit(g, (n * m,))]
        if constant is not None:
            c0 = constant(pos, ex, self.coef)
            pos = torch.cat([pos, pos[:, :1]], dim=1)
            ex = torch.cat([ex, torch.zeros_like(ex[:, :1])], dim=1)
            self.coef = [torch.cat([a, b[:, None]], dim=1) for a, b in zip(self.coef, c0)]
        self.pos, self.ex = pos.contiguous(), ex.contiguous()

    def handle(self):
        keep = self.ex.reshape(-1) > 0
        size = (self.ex > 0).sum(dim=2).reshape(-1)
        start = torch.cat([torch.zeros(1, dtype=torch.int64, device=DEV), size.cumsum(0)])
        host = lambda t: t.cpu().numpy()  # noqa: E731
        return pe.System(self.n, self.n, np.arange(0, self.n * self.m + 1, self.m), host(start),
                         host(self.pos.reshape(-1)[keep].to(torch.int32)),
                         host(self.ex.reshape(-1)[keep].to(torch.int32)),
                         [host(c.reshape(-1)) for c in self.coef])


# double-double in plain torch, for the constants of the known-root systems

def _two_sum(a, b):
    s = a + b
    t = s - a
    return s, (a - (s - t)) + (b - t)


def _two_prod(a, b):
    def split(v):
        c = v * 134217729.0
        h = c - (c - v)
        return h, v - h
    p = a * b
    (ah, al), (bh, bl) = split(a), split(b)
    return p, ((ah * bh - p) + ah * bl + al * bh) + al * bl


def _dadd(x, y):
    s, e = _two_sum(x[0], y[0])
    t, f = _two_sum(x[1], y[1])
    s, e = _two_sum(s, e + t)
    return _two_sum(s, e + f)


def _dmul(x, y):
    p, e = _two_prod(x[0], y[0])
    return _two_sum(p, e + (x[0] * y[1] + x[1] * y[0]))


def _cmul(x, y):
    neg = lambda v: (-v[0], -v[1])  # noqa: E731
    re = _dadd(_dmul(x[:2], y[:2]), neg(_dmul(x[2:], y[2:])))
    im = _dadd(_dmul(x[:2], y[2:]), _dmul(x[2:], y[:2]))
    return (*re, *im)


def _root_constant(xs):
    """constant(pos, ex, coef): minus the sum of the terms at xs, in double-double."""
    def constant(pos, ex, coef):
        v = tuple(coef)
        for j in range(pos.shape[2]):
            x = tuple(c[pos[:, :, j]] for c in xs)
            for r in range(int(ex[:, :, j].max())):
                w = _cmul(v, x)
                v = tuple(torch.where(ex[:, :, j] > r, a, b) for a, b in zip(w, v))
        parts = [v[:2], v[2:]]
        out = []
        for part in parts:
            while part[0].shape[1] > 1:
                if part[0].shape[1] % 2:
                    part = tuple(torch.cat([c, torch.zeros_like(c[:, :1])], dim=1) for c in part)
                part = _dadd(tuple(c[:, 0::2] for c in part), tuple(c[:, 1::2] for c in part))
            out += [-part[0][:, 0], -part[1][:, 0]]
        return out
    return constant


def _buffers(shape, planes):
    return [torch.empty(shape, dtype=torch.float64, device=DEV) for _ in range(planes)]


def _quadrics(g, n):
    """x_i^2, three products, two linear terms and a constant per polynomial."""
    rng = np.random.RandomState(int(torch.randint(0, 1 << 30, (1,), generator=g, device=DEV)))
    pos, ex, start, pstart = [], [], [0], [0]
    for i in range(n):
        monos = [[(i, 2)]]
        pairs = set()
        while len(pairs) < min(3, n * (n - 1) // 2):
            pairs.add(tuple(sorted(rng.choice(n, 2, replace=False).tolist())))
        monos += [[(a, 1), (b, 1)] for a, b in sorted(pairs)]
        monos += [[(int(a), 1)] for a in sorted(rng.choice(n, min(2, n), replace=False))]
        for mono in monos + [[]]:
            pos += [v for v, _ in mono]
            ex += [e for _, e in mono]
            start.append(len(pos))
        pstart.append(len(start) - 1)
    th = rng.uniform(0, 2 * math.pi, len(start) - 1)
    zero = np.zeros(th.size)
    return pe.System(n, n, pstart, start, pos, ex, (np.cos(th), zero, np.sin(th), zero))


def _batch_shapes(c):
    """The uneven shapes of a batch: part of the case, not of its inputs."""
    rng = np.random.RandomState(c["systems"] * 1000 + c["n"] + c["m"])
    out = []
    for _ in range(c["systems"]):
        n = int(rng.randint(16, c["n"] + 1))
        out.append((n, int(rng.randint(16, c["m"] + 1)), int(rng.randint(2, min(c["k"], n) + 1))))
    return out


def _newton_system(c, g):
    xs = _unit(g, (c["n"],))
    return _Sys(g, c["n"], c["m"], c["k"], c["d"], constant=_root_constant(xs)), xs


def _eval_inputs(c, seed):
    g = _gen(seed)
    s = _Sys(g, c["n"], c["m"], c["k"], c["d"], c["ragged"])
    return s, _unit(g, (c["P"], c["n"]), 4 if c["prec"] == "qd" else 2)


def _batch_inputs(c, seed):
    g = _gen(seed)
    syss = [_Sys(g, n, m, k, c["d"]) for n, m, k in _batch_shapes(c)]
    return syss, [_unit(g, (c["P"], s.n)) for s in syss]


def prepare(c, seed):
    kind = c["kind"]
    st = dict(case=c)
    if kind in ("eval", "values"):
        s, x = _eval_inputs(c, seed)
        n, P, planes = c["n"], c["P"], 8 if c["prec"] == "qd" else 4
        st.update(S=s.handle(), x=x, f=_buffers((P, n), planes),
                  J=_buffers((P, n, n), planes) if kind == "eval" else None)
        if c["prec"] != "qd":
            st["S"].get_schedule(P)  # the system's tables, which such a program keeps
    elif kind == "batch":
        syss, pts = _batch_inputs(c, seed)
        handles = [s.handle() for s in syss]
        B = pe.Batch(handles)
        pps = np.full(len(syss), c["P"], np.int64)
        _, fo, jo = B.layout(pps)
        st.update(S=handles, B=B, pps=pps, x=[torch.cat([p[q].reshape(-1) for p in pts]) for q in range(4)],
                  f=_buffers((int(fo[-1]),), 4), J=_buffers((int(jo[-1]),), 4))
    elif kind == "newton":
        g = _gen(seed)
        s, xs = _newton_system(c, g)
        n, P = c["n"], c["P"]
        start = []
        for h in (0, 2):
            delta = (torch.rand((P, n), generator=g, device=DEV, dtype=torch.float64) * 2 - 1) * 1e-6
            hi, e = _two_sum(xs[h].expand(P, n).contiguous(), delta)
            hi, lo = _two_sum(hi, e + xs[h + 1])
            start += [hi, lo] + ([torch.zeros_like(hi)] * 2 if c["mode"] == "qd" else [])
        i32 = lambda: torch.empty(P, dtype=torch.int32, device=DEV)  # noqa: E731
        st.update(S=s.handle(), start=start, x=_buffers((P, n), len(start)),
                  res=torch.empty(P, dtype=torch.float64, device=DEV), iters=i32(), status=i32())
    else:
        n, P = c["n"], c["P"]
        i32 = lambda: torch.empty(P, dtype=torch.int32, device=DEV)  # noqa: E731
        st.update(S=_quadrics(_gen(seed), n), x=_buffers((P, n), 4),
                  t=torch.empty(P, dtype=torch.float64, device=DEV),
                  res=torch.empty(P, dtype=torch.float64, device=DEV), steps=i32(), status=i32())
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

_PREC = {"dd": pe.PE_DD, "f64": pe.PE_FP64}


def _written(planes, prec):
    """The planes that a call writes: in FP64 the low ones are not touched."""
    return planes if planes is None or prec != "f64" else [planes[0], planes[2]]


def run(st):
    c = st["case"]
    kind = c["kind"]
    if kind in ("eval", "values"):
        if c["prec"] == "qd":
            st["S"].eval_jac_qd(c["P"], st["x"], st["f"], st["J"])
        else:
            st["S"].eval_jac(c["P"], st["x"], st["f"], st["J"], _PREC[c["prec"]])
        out = dict(f=_written(st["f"], c["prec"]))
        return out if st["J"] is None else dict(out, J=_written(st["J"], c["prec"]))
    if kind == "batch":
        st["B"].eval_jac(st["pps"], st["x"], st["f"], st["J"], _PREC[c["prec"]])
        return dict(f=_written(st["f"], c["prec"]), J=_written(st["J"], c["prec"]))
    if kind == "newton":
        for a, b in zip(st["x"], st["start"]):
            a.copy_(b)
        if c["mode"] == "qd":
            st["S"].newton_qd(c["P"], st["x"], st["res"], st["iters"], st["status"], tol=c["tol"])
        else:
            st["S"].newton(c["P"], st["x"], st["res"], st["iters"], st["status"], tol=c["tol"],
                           mode=pe.PE_NEWTON_DD if c["mode"] == "dd" else pe.PE_NEWTON_MIXED)
        return dict(x=st["x"], iters=st["iters"], status=st["status"])
    st["S"].start_solutions(0, c["P"], st["x"])
    st["S"].track(c["P"], st["x"], st["t"], st["steps"], st["status"], st["res"])
    return dict(x=st["x"], t=st["t"], status=st["status"])


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

# bytes of a complex value; flops of a complex product and of a complex sum
_BYTES = {"f64": 16, "dd": 32, "qd": 64}
_MUL = {"f64": 8, "dd": 88, "qd": 900}
_ADD = {"f64": 2, "dd": 40, "qd": 250}


def _eval_work(n, m, k, P, prec, jac=True):
    """m monomials of k variables in each of n polynomials: their values (k products each), and with
    the Jacobian one more product and sum per variable; tables read once, points in, f and J out."""
    terms = float(n) * m * P
    flops = terms * (k * _MUL[prec] + _ADD[prec] + (k * (_ADD[prec] + _MUL[prec]) if jac else 0))
    tables = float(n) * m * (32 + 4 * k)
    return dict(bytes=tables + _BYTES[prec] * P * (2.0 * n + (n * n if jac else 0)), flops=flops)


def work(c):
    kind = c["kind"]
    if kind in ("eval", "values"):
        k = (c["k"] + 1) / 2 if c["ragged"] else c["k"]
        return _eval_work(c["n"], c["m"], k, c["P"], c["prec"], kind == "eval")
    if kind == "batch":
        parts = [_eval_work(n, m, k, c["P"], c["prec"]) for n, m, k in _batch_shapes(c)]
        return {q: sum(p[q] for p in parts) for q in ("bytes", "flops")}
    if kind == "newton":
        # steps of an evaluation, a residual and a solve (n^3/3 complex multiply-adds)
        n, m, k, P = c["n"], c["m"], c["k"], c["P"]
        jp, rp, steps = dict(mixed=("f64", "dd", 3), dd=("dd", "dd", 3), qd=("f64", "qd", 5))[c["mode"]]
        ev = _eval_work(n, m, k, P, jp)
        rs = _eval_work(n, m, k, P, rp, False)
        lu = P * n ** 3 / 3.0 * (_MUL[jp] + _ADD[jp])
        flops = steps * (ev["flops"] + lu) + (0 if c["mode"] == "dd" else (steps + 1) * rs["flops"])
        return dict(bytes=float(n) * m * (32 + 4 * k) + 2.0 * P * n * _BYTES[rp], flops=flops)
    # tracker: about 55 steps of 2.5 evaluations and solves per path
    n, P = c["n"], c["P"]
    one = _eval_work(n, 7, 1.5, P, "f64")["flops"] + P * n ** 3 / 3.0 * 10
    return dict(bytes=float(P) * n * 32, flops=140.0 * one)


# ---------------------------------------------------------------------------
# what the passes compute, in 64 bits and without the library
# ---------------------------------------------------------------------------

_FRAC = 320  # fraction bits of the fixed-point evaluation


def _fixed(planes):
    """Exact fixed-point integers of a sum of planes (object array)."""
    out = np.zeros(planes[0].shape, dtype=object)
    for p in planes:
        m, e = np.frexp(p.cpu().numpy())
        mi = (m * 2.0 ** 53).astype(np.int64).astype(object)
        sh = e.astype(np.int64) - 53 + _FRAC
        up, down = np.maximum(sh, 0).astype(object), np.maximum(-sh, 0).astype(object)
        out = out + ((mi << up) >> down)
    return out


def _words(v, words):
    """Planes of the nearest sum of `words` doubles of fixed-point integers."""
    planes = np.zeros((words,) + v.shape)
    one = 1 << _FRAC
    flat = planes.reshape(words, -1)
    for i, a in enumerate(v.reshape(-1)):
        a = int(a)
        for w in range(words):
            hi = a / one
            flat[w, i] = hi
            m, e = math.frexp(hi)
            sh = e - 53 + _FRAC
            mi = int(m * 2.0 ** 53)
            a -= mi << sh if sh >= 0 else mi >> -sh
    return [torch.from_numpy(p) for p in planes]


def _exact_fixed(s, x, words, jac):
    """f and J at each point in fixed point: J = (sum of a V) / x with V the terms' values."""
    def mul(a, b):
        return ((a[0] * b[0] - a[1] * b[1]) >> _FRAC, (a[0] * b[1] + a[1] * b[0]) >> _FRAC)
    n, m, k = s.n, s.m, s.k
    h = len(x) // 2
    xr, xi = _fixed(x[:h]), _fixed(x[h:])
    coef = (_fixed(s.coef[:2]).reshape(-1), _fixed(s.coef[2:]).reshape(-1))
    pos, ex = s.pos.cpu().numpy().reshape(-1, k), s.ex.cpu().numpy().reshape(-1, k)
    row = np.repeat(np.arange(n), m)
    P = xr.shape[0]
    fs = [np.zeros((P, n), dtype=object) for _ in range(2)]
    Js = [np.zeros((P, n, n), dtype=object) for _ in range(2)]
    for p in range(P):
        one = np.full(n, 1 << _FRAC, dtype=object)
        pw = [(one, one * 0)]
        for _ in range(int(ex.max())):
            pw.append(mul(pw[-1], (xr[p], xi[p])))
        tab = [np.stack([q[c] for q in pw]) for c in range(2)]
        v = coef
        for j in range(k):
            v = mul(v, (tab[0][ex[:, j], pos[:, j]], tab[1][ex[:, j], pos[:, j]]))
        for c in range(2):
            fs[c][p] = v[c].reshape(n, m).sum(axis=1)
        if not jac:
            continue
        sums = [np.zeros((n, n), dtype=object) for _ in range(2)]
        for c in range(2):
            for j in range(k):
                np.add.at(sums[c], (pos[:, j], row), v[c] * ex[:, j].astype(object))
        den = (xr[p] * xr[p] + xi[p] * xi[p]) >> _FRAC
        inv = ((xr[p] << _FRAC) // den, -((xi[p] << _FRAC) // den))
        Js[0][p], Js[1][p] = mul(sums, (inv[0][:, None], inv[1][:, None]))
    f = _words(fs[0], words) + _words(fs[1], words)
    return f, (_words(Js[0], words) + _words(Js[1], words)) if jac else None


def _exact_f64(s, x, jac):
    """The leading words of f and J in complex FP64, a block of monomials at a time."""
    n, m, k = s.n, s.m, s.k
    h = len(x) // 2
    z = torch.complex(x[0], x[h])
    P = z.shape[0]
    tab = torch.stack([z ** e for e in range(s.d + 1)])          # [d+1][P][n]
    coef = torch.complex(s.coef[0], s.coef[2])
    f = torch.empty((P, n), dtype=torch.complex128, device=DEV)
    J = torch.empty((P, n, n), dtype=torch.complex128, device=DEV) if jac else None
    part = max(1, (1 << 25) // (m * k))
    for p in range(n):
        E = torch.zeros((m, n), dtype=torch.float64, device=DEV).scatter_add_(1, s.pos[p], s.ex[p].double())
        for a in range(0, P, part):
            b = min(P, a + part)
            v = tab[s.ex[p], a:b, s.pos[p]].prod(dim=1) * coef[p][:, None]      # [m][points]
            f[a:b, p] = v.sum(dim=0)
            if jac:
                J[a:b, :, p] = torch.complex(v.real.T.contiguous() @ E, v.imag.T.contiguous() @ E) / z[a:b]
    return f, J


def _exact_eval(s, x, prec, jac):
    """f and J as `run` lays them out: every word for small cases, else the leading words."""
    words = len(x) // 2
    if prec != "f64" and s.n * s.m * s.k * x[0].shape[0] <= 1 << 20:
        return _exact_fixed(s, x, words, jac)
    f, J = _exact_f64(s, x, jac)
    def lay(v):
        if v is None:
            return None
        gap = [None] * (words - 1) if prec != "f64" else []
        return [v.real.contiguous()] + gap + [v.imag.contiguous()] + gap
    return lay(f), lay(J)


def exact(c, seed):
    kind = c["kind"]
    if kind in ("eval", "values"):
        s, x = _eval_inputs(c, seed)
        f, J = _exact_eval(s, x, c["prec"], kind == "eval")
        return dict(f=f) if J is None else dict(f=f, J=J)
    if kind == "batch":
        syss, pts = _batch_inputs(c, seed)
        parts = [_exact_f64(s, x, True) for s, x in zip(syss, pts)]
        out = {}
        for name, i in (("f", 0), ("J", 1)):
            v = torch.cat([p[i].reshape(-1) for p in parts])
            gap = [None] if c["prec"] == "dd" else []
            out[name] = [v.real.contiguous()] + gap + [v.imag.contiguous()] + gap
        return out
    if kind == "newton" and c["mode"] != "qd":
        # the root itself; a quad-double one is only known to the constant's double-double rounding
        _, xs = _newton_system(c, _gen(seed))
        return dict(x=[v.expand(c["P"], c["n"]).contiguous() for v in xs], iters=None, status=None)
    return None
