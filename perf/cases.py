"""What users of this library have it do, as timed cases.

A case is a dict of plain values; `prepare` makes what a program holds before the
call (device tensors, radial handles, a server with its registered atoms), `run` is
one pass through the public entry points and returns everything the pass computes,
`exact` is the same in plain float64 torch from the definitions (normalised
associated Legendre functions, natural cubic spline), and `work` counts each input
read once and each output written once.

Kinds of case:
  eval     sh_eval / sh_eval_unit / sh_eval_angles (and the _f32 twins)
  complex  sh_eval_complex, spinor: sh_eval_spinor (and the _f32 twins)
  jac      sh_eval_jac: values and Cartesian Jacobian
  train    spherical_harmonics under autograd, forward and backward
  proj     sh_projectors(_f32) with a radial handle that the program keeps
  noalloc  sh_projectors_noalloc from knot values on the device
  serve    a burst of requests to the projector server, waited for and read
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2510_05282_amd as sh
from paper_2510_05282_amd.serve import Server

R_MAX = 3.0  # projector spheres, in the units of the grid
BOX = 20.0

DTYPE = {"f64": torch.float64, "f32": torch.float32}
ELEM = {"f64": 8, "f32": 4}


def listed():
    return [
        # one molecule's neighbour list: the call is launch and latency
        {"name": "eval_small", "kind": "eval", "input": "xyz", "dtype": "f64", "lmax": 4, "n": 1000},
        # the 100,064-point parity set of the tests: an ordinary one-off evaluation
        {"name": "eval_plain", "kind": "eval", "input": "xyz", "dtype": "f64", "lmax": 9, "n": 100064},
        # single precision on a point count that is no multiple of anything: every
        # row of the output starts at another alignment
        {"name": "eval_odd_f32", "kind": "eval", "input": "xyz", "dtype": "f32", "lmax": 6, "n": 1000003},
        # the bandwidth sweep of the benchmark, a quarter of its points
        {"name": "eval_sweep", "kind": "eval", "input": "xyz", "dtype": "f64", "lmax": 9, "n": 1 << 24},
        # complex harmonics of one radial shell set, odd count
        {"name": "complex_f64", "kind": "complex", "dtype": "f64", "lmax": 6, "n": 250001},
        # a machine-learned potential's edge features, forward and backward
        {"name": "train_f32", "kind": "train", "dtype": "f32", "lmax": 3, "n": 20000},
        # the differentiated evaluation of the benchmark (lmax 6), a quarter of its points
        {"name": "train_f64", "kind": "train", "dtype": "f64", "lmax": 6, "n": 1 << 22},
        # beyond the explicit formulas: the recurrence, forward and backward
        {"name": "train_rec", "kind": "train", "dtype": "f64", "lmax": 16, "n": 200001},
        # the projector set-up of a 64-atom cell: spheres of radius 3 on a 0.2 grid
        {"name": "proj_64", "kind": "proj", "dtype": "f64", "lmax": 3, "channels": 4, "atoms": 64,
         "points": 14137, "n_r": 2000},
        # a large single-precision build from tables of more channels than it asks for
        {"name": "proj_large", "kind": "proj", "dtype": "f32", "lmax": 3, "channels": 10, "atoms": 64,
         "points": 150000, "n_r": 2000},
        # radial functions that change with every build, inside code that may not allocate
        {"name": "proj_noalloc", "kind": "noalloc", "dtype": "f64", "lmax": 6, "atoms": 24, "points": 4189,
         "n_r": 2000},
        # a burst of uneven requests: lmax 0..9, 1e3..1e6 points, 80% in double precision
        {"name": "serve_burst", "kind": "serve", "requests": 48, "n_lo": 1000, "n_hi": 1000000},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["eval", "eval", "eval", "complex", "spinor", "jac", "train", "train", "proj", "proj",
                       "noalloc", "serve"])
    if kind == "serve":
        hi = _log_int(rng, 20000, 1000000)
        return {"kind": kind, "requests": rng.randint(4, 48), "n_lo": 1000, "n_hi": hi}
    dtype = rng.choice(["f64", "f32"])
    if kind in ("proj", "noalloc"):
        lmax = rng.randint(0, 6 if kind == "noalloc" else 9)
        n_r = rng.choice([300, 1000, 2000])
        atoms = _log_int(rng, 1, 24 if kind == "noalloc" else 256)
        most = min(200000, 4_000_000_000 // (8 * (lmax + 1) ** 2 * atoms))
        case = {"kind": kind, "dtype": dtype, "lmax": lmax, "atoms": atoms, "points": _log_int(rng, 300, most),
                "n_r": n_r}
        if kind == "proj":
            case["channels"] = rng.choice([lmax + 1, 10])
        return case
    case = {"kind": kind, "dtype": "f64" if kind == "jac" else dtype}
    if kind == "eval":
        case["input"] = rng.choice(["xyz", "xyz", "unit", "angles"])
    case["lmax"] = rng.randint(1, 9) if kind != "train" else rng.choice([1, 2, 3, 4, 6, 9, 12, 16])
    rows = (case["lmax"] + 1) ** 2 * {"eval": 1, "complex": 2, "spinor": 8, "jac": 4, "train": 2}[kind]
    n = _log_int(rng, 200, min(6_000_000, 4_000_000_000 // (8 * rows)))
    case["n"] = n if rng.random() < 0.5 else max(256, n // 64 * 64)
    return case


# ---------------------------------------------------------------- inputs


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _rand(g, *shape):
    return torch.rand(shape, generator=g, dtype=torch.float64, device="cuda")


def _randn(g, *shape, dtype=torch.float64):
    return torch.randn(shape, generator=g, dtype=dtype, device="cuda")


def _directions(g, n):
    d = _randn(g, n, 3)
    return d / d.norm(dim=1, keepdim=True)


def _points(case, g):
    """Isotropic points with radius in [0.1, 5] (unit vectors or angles where the case says so)."""
    n, dt = case["n"], DTYPE[case["dtype"]]
    d = _directions(g, n)
    how = case.get("input", "xyz")
    if how == "unit":
        return (d.to(dt).contiguous(),)
    if how == "angles":
        return (torch.acos(d[:, 2].clamp(-1, 1)).to(dt).contiguous(),
                torch.atan2(d[:, 1], d[:, 0]).to(dt).contiguous())
    return ((d * (0.1 + 4.9 * _rand(g, n, 1))).to(dt).contiguous(),)


def _radials(seed, tables, channels, n_r):
    """[tables][channels][n_r]: smooth radial functions that vanish at R_MAX, scaled to max |R| = 1."""
    rng = np.random.default_rng(seed)
    r = np.linspace(0.0, R_MAX, n_r)
    cut = (1.0 - (r / R_MAX) ** 2) ** 2
    c = rng.standard_normal((tables, channels, 3))
    a = rng.uniform(0.5, 2.0, size=(tables, channels, 3))
    v = np.zeros((tables, channels, n_r))
    l = np.arange(channels)[None, :, None]
    for k in range(3):
        v += c[:, :, k, None] * r ** (l + 2 * k) * np.exp(-a[:, :, k, None] * r * r)
    v *= cut
    return v / np.abs(v).max(axis=2, keepdims=True)


def _spheres(case, g, dt):
    """Centres in the box and each atom's grid points in grid order, as (centers, offsets, points) in dt.
    The spacing gives about case["points"] points within R_MAX; an atom holds the 98 to 100% of that
    number (uneven, the same for every seed) that lie nearest to its centre."""
    na = case["atoms"]
    h = R_MAX * (4.0 * math.pi / 3.0 / case["points"]) ** (1.0 / 3.0)
    rng = np.random.default_rng(case["points"])
    counts = np.maximum(1, (case["points"] * rng.uniform(0.98, 1.0, size=na)).astype(np.int64))
    centers = (BOX * _rand(g, na, 3)).to(dt)
    m = int(math.floor(2.0 * R_MAX / h)) + 3
    k = torch.arange(m, dtype=torch.float64, device="cuda")
    pts = []
    for c, n in zip(centers.to(torch.float64), counts):
        lo = torch.floor((c - R_MAX) / h)
        p = torch.cartesian_prod(lo[0] + k, lo[1] + k, lo[2] + k) * h
        near = ((p - c) ** 2).sum(1).topk(int(n), largest=False, sorted=False).indices.sort().values
        pts.append(p[near].to(dt))
    offsets = torch.zeros(na + 1, dtype=torch.int64)
    offsets[1:] = torch.from_numpy(counts).cumsum(0)
    return centers.contiguous(), offsets.cuda(), torch.cat(pts).contiguous()


def _requests(case, seed):
    """(lmax, n, dtype, centre) of each request: the mix belongs to the case, the centres to the seed."""
    rng, place = np.random.default_rng([case["requests"], case["n_hi"]]), np.random.default_rng(seed)
    lo, hi = math.log(case["n_lo"]), math.log(case["n_hi"])
    return [(int(rng.integers(0, 10)), int(round(math.exp(rng.uniform(lo, hi)))),
             "f64" if rng.uniform() < 0.8 else "f32", place.uniform(0.0, BOX, size=3))
            for _ in range(case["requests"])]


def _request_inputs(case, seed):
    """Per request its points in the ball of radius R_MAX about its centre; per lmax the tables of its requests."""
    reqs, g = _requests(case, seed), _gen(seed)
    pts = [(torch.from_numpy(c).cuda() + _directions(g, n) * R_MAX * _rand(g, n, 1) ** (1 / 3)).to(DTYPE[d]).contiguous()
           for _, n, d, c in reqs]
    tables = {l: _radials(seed + l, sum(r[0] == l for r in reqs), l + 1, 2000) for l in {r[0] for r in reqs}}
    return reqs, pts, tables


class _Serving:
    """A program's server with its registered atoms; the results of the last burst are held until the next."""

    def __init__(self, case, seed):
        self.reqs, self.points, tables = _request_inputs(case, seed)
        out = sum((l + 1) ** 2 * n * ELEM[d] + 256 for l, n, d, _ in self.reqs)
        self.server = Server(out + (64 << 20), max_pending=len(self.reqs) + 1, n_slots=3)
        radials = {l: sh.Radial(t, R_MAX) for l, t in tables.items()}
        used = dict.fromkeys(radials, 0)
        self.atoms = []
        for (l, _, _, c), p in zip(self.reqs, self.points):
            self.atoms.append(self.server.add_atom(p, c, radials[l], table=used[l]))
            used[l] += 1
        self.held = []


class _Results(list):
    """Result tensors that alias the server's memory, and so keep the server alive."""


def prepare(case, seed):
    kind = case["kind"]
    if kind == "serve":
        return {"case": case, "serving": _Serving(case, seed)}
    g, dt = _gen(seed), DTYPE[case["dtype"]]
    if kind in ("proj", "noalloc"):
        centers, offsets, points = _spheres(case, g, dt)
        s = {"case": case, "centers": centers, "offsets": offsets, "points": points}
        v = _radials(seed, case["atoms"], case.get("channels", case["lmax"] + 1), case["n_r"])
        if kind == "proj":
            s["radial"] = sh.Radial(v, R_MAX)
        else:
            s["values"] = torch.from_numpy(v).cuda()
            s["out"] = torch.empty((case["lmax"] + 1) ** 2 * points.shape[0], dtype=dt, device="cuda")
        return s
    s = {"case": case, "in": _points(case, g)}
    if kind == "train":
        s["x"] = s.pop("in")[0].requires_grad_(True)
        s["G"] = _randn(g, (case["lmax"] + 1) ** 2, case["n"], dtype=dt)
    return s


# ---------------------------------------------------------------- the timed pass

_EVAL = {"xyz": sh.sh_eval, "unit": sh.sh_eval_unit, "angles": sh.sh_eval_angles}
_EVAL_F32 = {"xyz": sh.sh_eval_f32, "unit": sh.sh_eval_unit_f32, "angles": sh.sh_eval_angles_f32}


def run(s):
    case = s["case"]
    kind, f64 = case["kind"], case.get("dtype") == "f64"
    if kind == "eval":
        return (_EVAL if f64 else _EVAL_F32)[case["input"]](case["lmax"], *s["in"])
    if kind == "complex":
        return (sh.sh_eval_complex if f64 else sh.sh_eval_complex_f32)(case["lmax"], *s["in"])
    if kind == "spinor":
        return (sh.sh_eval_spinor if f64 else sh.sh_eval_spinor_f32)(case["lmax"], *s["in"])
    if kind == "jac":
        return sh.sh_eval_jac(case["lmax"], *s["in"])
    if kind == "train":
        y = sh.spherical_harmonics(s["x"], case["lmax"])
        (grad,) = torch.autograd.grad(y, s["x"], s["G"])
        return y.detach(), grad
    if kind == "proj":
        fn = sh.sh_projectors if f64 else sh.sh_projectors_f32
        return fn(case["lmax"], s["centers"], s["offsets"], s["points"], s["radial"])
    if kind == "noalloc":
        return sh.sh_projectors_noalloc(case["lmax"], s["centers"], s["offsets"], s["points"], s["values"], R_MAX,
                                        out=s["out"])
    v = s["serving"]
    for t in v.held:
        v.server.release(t)
    v.held = [v.server.submit(a, r[0]) for a, r in zip(v.atoms, v.reqs)]
    for t in v.held:
        v.server.wait(t)
    out = _Results(v.server.result(t, l, n, DTYPE[d]) for t, (l, n, d, _) in zip(v.held, v.reqs))
    out.serving = v
    return out


# ---------------------------------------------------------------- work


def work(case):
    kind = case["kind"]
    if kind == "serve":
        reqs = _requests(case, 0)
        return {"bytes": sum(n * ELEM[d] * (3 + (l + 1) ** 2) for l, n, d, _ in reqs),
                "flops": sum(n * 8 * (l + 1) ** 2 for l, n, _, _ in reqs)}
    s, F = ELEM[case["dtype"]], (case["lmax"] + 1) ** 2
    if kind in ("proj", "noalloc"):
        n = case["atoms"] * case["points"]
        b = n * s * (3 + F)
        if kind == "noalloc":
            b += case["atoms"] * (case["lmax"] + 1) * case["n_r"] * 8
        return {"bytes": b, "flops": n * 8 * F}
    n = case["n"]
    values = {"eval": F, "complex": 2 * F, "spinor": 8 * F, "jac": 4 * F, "train": 2 * F + 3}[kind]
    inputs = 2 if case.get("input") == "angles" else 3
    per = {"eval": 6, "complex": 8, "spinor": 16, "jac": 24, "train": 18}[kind]
    return {"bytes": n * s * (inputs + values), "flops": n * per * F}


# ---------------------------------------------------------------- the same in plain float64


def _harmonics(u, lmax):
    """Yields (l, m, P, dP) for m >= 0 at unit vectors u: P the normalised Legendre factor of z
    (sin^m taken out, sqrt 2 for m > 0), dP its z-derivative, from the three-term recurrence."""
    z = u[:, 2]
    d = torch.full_like(z, 1.0 / math.sqrt(4.0 * math.pi))
    zero = torch.zeros_like(z)
    for m in range(lmax + 1):
        if m > 0:
            d = d * math.sqrt((2 * m + 1) / (2 * m)) * (math.sqrt(2.0) if m == 1 else 1.0)
        p2, q2, p1, q1 = zero, zero, d, zero
        yield m, m, p1, q1
        for l in range(m + 1, lmax + 1):
            a = math.sqrt((4 * l * l - 1) / (l * l - m * m))
            b = math.sqrt(((l - 1) ** 2 - m * m) / (4 * (l - 1) ** 2 - 1))
            p, q = a * (z * p1 - b * p2), a * (p1 + z * q1 - b * q2)
            p2, q2, p1, q1 = p1, q1, p, q
            yield l, m, p, q


def _powers(u, lmax):
    """C_m, S_m with C_m + i S_m = (x + i y)^m, m = 0..lmax."""
    x, y = u[:, 0], u[:, 1]
    C, S = [torch.ones_like(x)], [torch.zeros_like(x)]
    for _ in range(lmax):
        C, S = C + [x * C[-1] - y * S[-1]], S + [x * S[-1] + y * C[-1]]
    return C, S


def _unit(case, s_in):
    p = [t.to(torch.float64) for t in s_in]
    if case.get("input") == "angles":
        return torch.stack([torch.sin(p[0]) * torch.cos(p[1]), torch.sin(p[0]) * torch.sin(p[1]), torch.cos(p[0])], 1)
    return p[0] if case.get("input") == "unit" else p[0] / p[0].norm(dim=1, keepdim=True)


def _real(u, lmax, out=None):
    out = torch.empty(((lmax + 1) ** 2, u.shape[0]), dtype=torch.float64, device=u.device) if out is None else out
    C, S = _powers(u, lmax)
    for l, m, P, _ in _harmonics(u, lmax):
        torch.mul(P, C[m], out=out[l * l + l + m])
        if m:
            torch.mul(P, S[m], out=out[l * l + l - m])
    return out


def _complex(u, lmax):
    R = _real(u, lmax)
    Y = torch.empty(R.shape, dtype=torch.complex128, device=u.device)
    for l in range(lmax + 1):
        Y[l * l + l] = R[l * l + l].to(torch.complex128)
        for m in range(1, l + 1):
            w = torch.complex(R[l * l + l + m], R[l * l + l - m]) / math.sqrt(2.0)
            Y[l * l + l + m] = (-1) ** m * w
            Y[l * l + l - m] = w.conj()
    return Y


def _spinor(u, lmax):
    """m_j = m + 1/2: the upper component holds Y_l^m, the lower one Y_l^(m+1)."""
    Y = _complex(u, lmax)
    out = torch.zeros((2 * (lmax + 1) ** 2, 2, u.shape[0]), dtype=torch.complex128, device=u.device)
    for l in range(lmax + 1):
        for m in range(-l - 1, l + 1):
            hi, lo = math.sqrt((l + m + 1) / (2 * l + 1)), math.sqrt((l - m) / (2 * l + 1))
            rows = [(2 * l * l + 3 * l + m + 1, hi, lo)]  # j = l + 1/2
            if -l <= m < l:
                rows.append((2 * l * l + l + m, -lo, hi))  # j = l - 1/2
            for k, up, down in rows:
                if m >= -l:
                    out[k, 0] = up * Y[l * l + l + m]
                if m < l:
                    out[k, 1] = down * Y[l * l + l + m + 1]
    return out


def _gradients(x, lmax):
    """Yields (row, value, gradient [3][n] with respect to x)."""
    r = x.norm(dim=1)
    u = x / r[:, None]
    C, S = _powers(u, lmax)
    zero = torch.zeros_like(r)
    for l, m, P, Q in _harmonics(u, lmax):
        for sign in (1, -1) if m else (1,):
            A, B = (C, S) if sign > 0 else (S, C)
            ax = m * A[m - 1] if m else zero
            ay = -sign * m * B[m - 1] if m else zero
            g = torch.stack([P * ax, P * ay, Q * A[m]])
            ug = (u.T * g).sum(0)
            yield l * l + l + sign * m, P * A[m], (g - u.T * ug) / r


def _spline(v):
    """Second derivatives (times h^2) of the natural cubic splines through v[..., n_r], by the Thomas algorithm."""
    n = v.shape[-1]
    M, c = np.zeros_like(v), np.zeros(n)
    rhs = 6.0 * (v[..., 2:] - 2.0 * v[..., 1:-1] + v[..., :-2])
    for k in range(1, n - 1):
        den = 4.0 - c[k - 1]
        c[k] = 1.0 / den
        M[..., k] = (rhs[..., k - 1] - M[..., k - 1]) / den
    for k in range(n - 3, 0, -1):
        M[..., k] -= c[k] * M[..., k + 1]
    return M


def _projector(p, center, v, M, lmax):
    """[F][n] projectors of points p (float64) about center, from one table v and its M (device, [channels][n_r])."""
    d = p - center
    r = d.norm(dim=1)
    n_r = v.shape[1]
    q = r * ((n_r - 1) / R_MAX)
    i = q.floor().long().clamp(0, n_r - 2)
    b = q - i
    a = 1.0 - b
    out = _real(d / torch.where(r > 0, r, torch.ones_like(r))[:, None], lmax)
    for l in range(lmax + 1):
        R = a * v[l][i] + b * v[l][i + 1] + ((a ** 3 - a) * M[l][i] + (b ** 3 - b) * M[l][i + 1]) / 6.0
        out[l * l:(l + 1) ** 2] *= torch.where(r <= R_MAX, R, torch.zeros_like(R))
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "serve":
        reqs, pts, tables = _request_inputs(case, seed)
        dev = {l: (torch.from_numpy(t).cuda(), torch.from_numpy(_spline(t)).cuda()) for l, t in tables.items()}
        used, out = dict.fromkeys(tables, 0), []
        for (l, _, _, c), p in zip(reqs, pts):
            v, M = (t[used[l]] for t in dev[l])
            used[l] += 1
            out.append(_projector(p.to(torch.float64), torch.from_numpy(c).cuda(), v, M, l))
        return out
    g, dt, lmax = _gen(seed), DTYPE[case["dtype"]], case["lmax"]
    if kind in ("proj", "noalloc"):
        centers, offsets, points = _spheres(case, g, dt)
        t = _radials(seed, case["atoms"], case.get("channels", lmax + 1), case["n_r"])
        v, M = torch.from_numpy(t).cuda(), torch.from_numpy(_spline(t)).cuda()
        o = offsets.tolist()
        return torch.cat([_projector(points[o[k]:o[k + 1]].to(torch.float64), centers[k].to(torch.float64), v[k], M[k],
                                     lmax).reshape(-1) for k in range(case["atoms"])])
    x = _points(case, g)
    if kind in ("eval", "complex", "spinor"):
        u = _unit(case, x)
        return {"eval": _real, "complex": _complex, "spinor": _spinor}[kind](u, lmax)
    xd, F = x[0].to(torch.float64), (lmax + 1) ** 2
    y = torch.empty((F, case["n"]), dtype=torch.float64, device="cuda")
    if kind == "jac":
        jac = torch.empty((3, F, case["n"]), dtype=torch.float64, device="cuda")
        for f, value, grad in _gradients(xd, lmax):
            y[f], jac[:, f] = value, grad
        return y, jac
    G = _randn(g, F, case["n"], dtype=dt)
    total = torch.zeros((3, case["n"]), dtype=torch.float64, device="cuda")
    for f, value, grad in _gradients(xd, lmax):
        y[f] = value
        total += G[f].to(torch.float64) * grad
    return y, total.T.contiguous()
