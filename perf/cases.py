"""Performance cases: what a program that computes fermion propagators has this
library do, at the sizes and options it does it with.

Every case is a dict of plain values; ``kind`` names the entry point:

* ``apply``     ``Lattice.apply`` on canonical fields, FP64 (an application that
                converts at every call);
* ``native``    ``Lattice.apply_native`` on half fields in the library's layout,
                FP64, FP32 or FP16 (the operator inside a caller's own solver);
* ``solve``     ``Lattice.solve``: one propagator component, FP64 or with FP32 /
                FP16 inner iterations;
* ``batch``     ``solve_batch``: the 12 spin-colour point sources on two lattices;
* ``mg``        ``Lattice.solve_mg`` (two-level multigrid with the SAP smoother);
* ``stag``      ``Lattice.stag_solve``;
* ``dwf``       the native domain-wall D or D^dag;
* ``dwf_solve`` ``Lattice.dwf_solve_eo``.

Solves run to a true residual of 1e-12, two decades below the default, as for
propagators that enter differences, so that the solution itself (and not only
its residual) is fixed to well below 1e-9.

Fields are made on the GPU from the seed: links U = exp(i eps H) re-projected
onto SU(3), complex Gaussian sources (point sources in the batch). ``exact``
writes the operators out in plain torch complex128.
"""

import math

import numpy as np
import torch

from paper_2303_05883_amd import lqcd

TOL = 1e-12
PREC = {"f64": lqcd.F64, "f32": lqcd.F32, "f16": lqcd.F16}
C128 = torch.complex128


# ------------------------------------------------------------------ the cases

def _dims(case, pre=""):
    return tuple(case[pre + k] for k in ("lx", "ly", "lz", "lt"))


def _with_dims(case, dims, pre=""):
    case.update(zip((pre + "lx", pre + "ly", pre + "lz", pre + "lt"), (int(d) for d in dims)))
    return case


def listed():
    def c(name, kind, dims, **kw):
        return _with_dims({"name": name, "kind": kind, **kw}, dims)

    return [
        # the smallest call: one clover D on the 8^4 lattice of the unit tests, where launches and latency count
        c("apply_D_f64_8x8x8x8", "apply", (8, 8, 8, 8), op="D", kappa=0.137, csw=1.0),
        # the same call on the production lattice: conversions in and out around the full operator
        c("apply_D_f64_32x32x32x64", "apply", (32, 32, 32, 64), op="D", kappa=0.137, csw=1.0),
        # the benchmark's Dslash, tuned as the benchmark tunes it
        c("hop_f32_32x32x32x64", "native", (32, 32, 32, 64), op="HOP_EO", prec="f32", kappa=0.135, csw=0.0, tuned=True),
        # the operator of an FP16 inner solver on the middle lattice of the batch workload
        c("schur_f16_24x24x24x48", "native", (24, 24, 24, 48), op="DPREC_SCHUR", prec="f16", kappa=0.137, csw=1.0,
          tuned=False),
        # FP64 on a ragged lattice: no extent a multiple of 8, the last 64-site block partly empty
        c("schur_f64_30x22x26x38", "native", (30, 22, 26, 38), op="DPREC_SCHUR", prec="f64", kappa=0.137, csw=1.0,
          tuned=False),
        # mixed-precision Wilson solve on a small lattice (many of these in an ensemble): short kernels
        c("solve_wilson_f32_16x16x16x32", "solve", (16, 16, 16, 32), inner="f32", kappa=0.135, csw=0.0),
        # mixed-precision clover solve with FP16 inner iterations
        c("solve_clover_f16_24x24x24x48", "solve", (24, 24, 24, 48), inner="f16", kappa=0.137, csw=1.0),
        # two lattices of uneven size, 12 point sources each, solved together
        _with_dims(c("batch_f32_16x16x16x32_12x12x12x24", "batch", (16, 16, 16, 32), inner="f32", nrhs=12,
                     kappa=0.137, csw=1.0), (12, 12, 12, 24), "second_"),
        # multigrid: SAP smoother, coarse solves and the FP64 flexible BiCGStab around them
        c("mg_16x16x16x32", "mg", (16, 16, 16, 32), kappa=0.137, csw=1.0, nvec=8),
        # staggered CG in FP64
        c("stag_f64_24x24x24x48", "stag", (24, 24, 24, 48), inner="f64", mass=0.05),
        # D^dag of the Moebius domain-wall operator on the paper's larger local volume
        c("dwf_dag_f64_64x32x16x8_ls8", "dwf", (64, 32, 16, 8), ls=8, prec="f64", dag=True, b5=1.5, c5=0.5),
        # even-odd domain-wall solve with FP32 inner CG
        c("dwf_solve_f32_16x16x16x16_ls8", "dwf_solve", (16, 16, 16, 16), ls=8, inner="f32", b5=1.5, c5=0.5),
    ]


def _draw_dims(rng, lo, hi, step=2):
    """Even extents (multiples of ``step``) whose product is spread over [lo, hi] in its logarithm."""
    while True:
        v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        e = [max(step, step * round(v ** 0.25 * math.exp(rng.uniform(-0.5, 0.5)) / step)) for _ in range(3)]
        e.append(max(step, step * round(v / (e[0] * e[1] * e[2]) / step)))
        if e[3] >= 4 and lo <= e[0] * e[1] * e[2] * e[3] <= hi:
            return tuple(e)


def draw(rng):
    kind = rng.choice(["apply", "native", "native", "solve", "batch", "mg", "stag", "dwf", "dwf_solve"])
    case = {"kind": kind}
    if kind in ("apply", "native", "solve"):
        case.update(rng.choice([{"kappa": 0.135, "csw": 0.0}, {"kappa": 0.137, "csw": 1.0}, {"kappa": 0.13, "csw": 1.2}]))
    if kind == "apply":
        case["op"] = rng.choice(["D", "DPREC_SCHUR", "DEO", "DOO_INV"])
        return _with_dims(case, _draw_dims(rng, 4096, 2097152))
    if kind == "native":
        case.update(op=rng.choice(["HOP_EO", "HOP_OE", "DPREC_SCHUR"]), prec=rng.choice(["f64", "f32", "f16"]),
                    tuned=rng.choice([True, False]))
        return _with_dims(case, _draw_dims(rng, 4096, 2097152))
    if kind == "solve":
        case["inner"] = rng.choice(["f64", "f32", "f16"])
        return _with_dims(case, _draw_dims(rng, 4096, 400000))
    if kind == "batch":
        case.update(inner=rng.choice(["f32", "f16"]), nrhs=rng.choice([3, 7, 12]), kappa=0.137, csw=1.0)
        _with_dims(case, _draw_dims(rng, 8192, 131072))
        return _with_dims(case, _draw_dims(rng, 4096, 41472), "second_")
    if kind == "mg":
        case.update(kappa=rng.choice([0.135, 0.136, 0.137]), csw=1.0, nvec=rng.choice([4, 6, 8]))
        return _with_dims(case, _draw_dims(rng, 8192, 131072, 8))
    if kind == "stag":
        case.update(inner=rng.choice(["f64", "f32"]), mass=rng.choice([0.05, 0.1, 0.2]))
        return _with_dims(case, _draw_dims(rng, 4096, 663552))
    case.update(rng.choice([{"b5": 1.0, "c5": 0.0}, {"b5": 1.5, "c5": 0.5}]), ls=rng.choice([4, 6, 8, 12, 16]))
    if kind == "dwf":
        case.update(prec=rng.choice(["f64", "f32"]), dag=rng.choice([True, False]))
        return _with_dims(case, _draw_dims(rng, 4096, 2097152 // case["ls"]))
    case["inner"] = rng.choice(["f64", "f32"])
    return _with_dims(case, _draw_dims(rng, 1024, 524288 // case["ls"]))


# ------------------------------------------------------------------ inputs

M5, MF = 1.8, 0.05  # domain-wall height and mass
EPS = 0.3           # smoothness of the links


def _gen(seed, what):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + what) % (1 << 62))
    return g


def _mm3(a, b):
    return torch.stack([torch.stack([sum(a[..., i, k] * b[..., k, j] for k in range(3)) for j in range(3)], -1)
                        for i in range(3)], -2)


def _gauge(dims, seed):
    """exp(i EPS H), H traceless Hermitian from a complex Gaussian matrix, rows 0 and 1 re-orthonormalised."""
    lx, ly, lz, lt = dims
    gen = _gen(seed, 1)
    out = torch.empty((lt, lz, ly, lx, 4, 3, 3), dtype=C128, device="cuda")
    for mu in range(4):
        g = torch.view_as_complex(torch.randn((lt, lz, ly, lx, 3, 3, 2), generator=gen, device="cuda", dtype=torch.float64))
        h = 0.5 * (g + g.conj().transpose(-1, -2))
        tr = (h[..., 0, 0] + h[..., 1, 1] + h[..., 2, 2]) / 3
        for k in range(3):
            h[..., k, k] -= tr
        a = (1j * EPS / 4) * h  # the exponential of a quarter of it by its series, squared twice
        u, term = a.clone(), a
        for n in range(2, 11):
            term = _mm3(term, a) / n
            u += term
        for k in range(3):
            u[..., k, k] += 1
        u = _mm3(u, u)
        u = _mm3(u, u)
        r0 = u[..., 0, :] / torch.linalg.vector_norm(u[..., 0, :], dim=-1, keepdim=True)
        r1 = u[..., 1, :] - (r0.conj() * u[..., 1, :]).sum(-1, keepdim=True) * r0
        r1 = r1 / torch.linalg.vector_norm(r1, dim=-1, keepdim=True)
        out[..., mu, 0, :] = r0
        out[..., mu, 1, :] = r1
        for k in range(3):
            i, j = (k + 1) % 3, (k + 2) % 3
            out[..., mu, 2, k] = (r0[..., i] * r1[..., j] - r0[..., j] * r1[..., i]).conj()
    return out


def _gauss(shape, seed, what=2):
    r = torch.randn(tuple(shape) + (2,), generator=_gen(seed, what), device="cuda", dtype=torch.float64)
    return torch.view_as_complex(r) * math.sqrt(0.5)


def _spinor(dims, seed, lead=()):
    lx, ly, lz, lt = dims
    return _gauss(tuple(lead) + (lt, lz, ly, lx, 4, 3), seed)


def _points(dims, n):
    """The first n spin-colour point sources at the origin."""
    lx, ly, lz, lt = dims
    b = torch.zeros((n, lt, lz, ly, lx, 4, 3), dtype=C128, device="cuda")
    for r in range(n):
        b[r, 0, 0, 0, 0, r // 3, r % 3] = 1
    return b


def _lattice(dims, seed, kappa=None, csw=0.0, stream=None):
    lat = lqcd.Lattice(dims, -1, stream=stream)
    lat.set_gauge(_gauge(dims, seed))
    if kappa is not None:
        lat.set_clover(kappa, csw)
    return lat


def _in_parity(op):
    return 1 if op in ("HOP_EO", "DEO", "DOO_INV") else 0


def prepare(case, seed):
    kind, dims = case["kind"], _dims(case)
    s = {"case": case}
    if kind in ("apply", "native", "solve", "mg"):
        s["lat"] = lat = _lattice(dims, seed, case["kappa"], case["csw"])
    if kind in ("stag", "dwf", "dwf_solve"):
        s["lat"] = lat = _lattice(dims, seed)
    if kind == "native":
        prec = PREC[case["prec"]]
        if case["tuned"]:
            lat.autotune(prec)
        nb = lat.field_bytes(prec)
        s["in"] = torch.zeros(nb, dtype=torch.uint8, device="cuda")
        s["out"] = torch.zeros(nb, dtype=torch.uint8, device="cuda")
        lat.import_field(prec, _in_parity(case["op"]), _spinor(dims, seed), s["in"])
    elif kind == "dwf":
        prec, ls = PREC[case["prec"]], case["ls"]
        nb = lat.dwf_field_bytes(prec, ls)
        for k in ("in", "out", "tmp"):
            s[k] = torch.zeros(nb, dtype=torch.uint8, device="cuda")
        lat.dwf_import(prec, ls, _spinor(dims, seed, (ls,)), s["in"])
    elif kind == "batch":
        stream = torch.cuda.Stream()
        both = (dims, _dims(case, "second_"))
        s["lats"] = [_lattice(d, seed + 500 * k, case["kappa"], case["csw"], stream) for k, d in enumerate(both)]
        s["b"] = [_points(d, case["nrhs"]) for d in both]
        s["x"] = [torch.zeros_like(b) for b in s["b"]]
        lqcd.batch_autotune(s["lats"], [case["nrhs"]] * 2, PREC[case["inner"]])
    else:
        lx, ly, lz, lt = dims
        if kind == "stag":
            s["b"] = _gauss((lt, lz, ly, lx, 3), seed)
        else:
            s["b"] = _spinor(dims, seed, (case["ls"],) if kind == "dwf_solve" else ())
        s["x"] = torch.zeros_like(s["b"])
        if kind == "mg":
            start = _gauss((case["nvec"], lt, lz, ly, lx, 4, 3), seed, 3)
            lat.mg_setup(start, agg=(4, 4, 4, 4), nvec=case["nvec"], setup_iters=4,
                         sap_block=(8, 4, 2, 2) if lx % 16 == 0 else (4, 4, 2, 2), ncycles=4, nmr=6)
    return s


# ------------------------------------------------------------------ one pass

def _native_view(buf, prec):
    """A native field's numbers: its reals, or in FP16 its codes and its sites' scales."""
    if prec != "f16":
        return buf.view(torch.float64 if prec == "f64" else torch.float32)
    blocks = buf.view(-1, 64 * 52)
    return {"codes": blocks[:, :64 * 48].view(torch.float16), "scales": blocks[:, 64 * 48:].view(torch.float32)}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "batch":
        lqcd.solve_batch(state["lats"], state["b"], state["x"], tol=TOL, inner_prec=PREC[case["inner"]])
        return state["x"]
    lat = state["lat"]
    if kind == "native":
        lat.apply_native(case["op"], PREC[case["prec"]], state["in"], state["out"])
        return _native_view(state["out"], case["prec"])
    if kind == "dwf":
        lat.dwf_apply_native_repeat(case["ls"], M5, MF, PREC[case["prec"]], [state["in"]], [state["out"]], 1,
                                    dag=case["dag"], b5=case["b5"], c5=case["c5"], tmp=state["tmp"])
        return _native_view(state["out"], case["prec"])
    b, x = state["b"], state["x"]
    if kind == "apply":
        return lat.apply(case["op"], lqcd.F64, b, x)
    if kind == "solve":
        lat.solve(b, x, tol=TOL, inner_prec=PREC[case["inner"]])
    elif kind == "mg":
        lat.solve_mg(b, x, tol=TOL)
    elif kind == "stag":
        lat.stag_solve(case["mass"], b, x, tol=TOL, inner_prec=PREC[case["inner"]])
    else:
        lat.dwf_solve_eo(case["ls"], M5, MF, b, x, tol=TOL, b5=case["b5"], c5=case["c5"], inner_prec=PREC[case["inner"]])
    return x


# ------------------------------------------------------------------ work

def work(case):
    """Each input read once and each output written once; for a solve, of every
    iteration, at a fixed number of iterations that such systems take."""
    kind = case["kind"]

    def hop_io(v, word, clover):  # one even-odd operator: all links, one half field in and out
        return v * (4 * 12 * word) + v / 2 * (48 * word) + (v / 2 * 72 * word if clover else 0)

    v = math.prod(_dims(case))
    clover = case.get("csw", 0.0) != 0.0
    word = {"f64": 8, "f32": 4, "f16": 2}[case.get("prec", case.get("inner", "f64"))]
    if kind == "apply":
        return {"bytes": v * (2 * 192 + 4 * 96 + (576 if clover else 0)), "flops": v * (1320 + (504 if clover else 0))}
    if kind == "native":
        two = case["op"] == "DPREC_SCHUR"
        return {"bytes": hop_io(v, word, False) + (2 if two and clover else 0) * v / 2 * 72 * word,
                "flops": v / 2 * ((2 if two else 1) * 1320 + (1008 if two and clover else 0))}
    if kind in ("solve", "batch", "mg"):
        its = 330 if clover else 80
        one = 4 * (1320 + (504 if clover else 0)) + 600
        if kind == "solve":
            return {"bytes": its * (4 * hop_io(v, word, clover) + v / 2 * 14 * 24 * word), "flops": its * v / 2 * one}
        if kind == "mg":  # 40 iterations of two smoothings (8 half-lattice launches of 6 block steps) each
            return {"bytes": 40 * (2 * 8 * v / 2 * (8 * 48 + 288 + 6 * 96) + 2 * v * (768 + 576) + 20 * v * 192),
                    "flops": 40 * (2 * 8 * 6 * v / 2 * 1920 + 2 * v * 1824)}
        v += math.prod(_dims(case, "second_"))
        n = case["nrhs"]
        return {"bytes": its * (4 * (v * 48 * word + v / 2 * (72 + 48 * n) * word) + n * v / 2 * 14 * 24 * word),
                "flops": its * n * v / 2 * one}
    if kind == "stag":
        its = 30 / case["mass"]
        return {"bytes": its * (2 * (v * 48 * word + v / 2 * 12 * word) + v / 2 * 9 * 6 * word),
                "flops": its * v / 2 * (2 * 570 + 60)}
    n5 = v * case["ls"]
    if kind == "dwf":
        return {"bytes": n5 * 48 * word + v * 48 * word, "flops": n5 * 1512}
    return {"bytes": 160 * (4 * (v * 48 * word) + n5 / 2 * (8 + 6) * 24 * word), "flops": 160 * n5 / 2 * 4 * 1600}


# ------------------------------------------------------------------ the same in plain torch, 64 bits

AXIS = (-3, -4, -5, -6)  # of x, y, z, t in a spinor field [..., t, z, y, x, spin, colour]


def _gammas():
    s = [np.array([[0, 1], [1, 0]], complex), np.array([[0, -1j], [1j, 0]]), np.array([[1, 0], [0, -1]], complex)]
    z = np.zeros((2, 2))
    return [np.block([[z, -1j * m], [1j * m, z]]) for m in s] + [np.diag([1, 1, -1, -1]).astype(complex)]


GAMMA = _gammas()
GAMMA5 = GAMMA[0] @ GAMMA[1] @ GAMMA[2] @ GAMMA[3]
ONE = np.eye(4)


def _spin(m, f):
    """m (4 x 4) on the spin index."""
    rows = []
    for i in range(4):
        row = None
        for j in range(4):
            if m[i, j] != 0:
                t = f[..., j, :] * complex(m[i, j])
                row = t if row is None else row + t
        rows.append(torch.zeros_like(f[..., 0, :]) if row is None else row)
    return torch.stack(rows, -2)


def _colour(u, f, dag=False):
    """u or u^dag [..., 3, 3] on the colour index of a spinor field (u without its spin index)."""
    out = []
    for a in range(3):
        out.append(sum((u[..., b, a].conj() if dag else u[..., a, b]).unsqueeze(-1) * f[..., b] for b in range(3)))
    return torch.stack(out, -1)


def _flip(f, mu, step, axis):
    """The neighbour's value, antiperiodic in t."""
    g = torch.roll(f, -step, axis)
    if mu == 3:
        g.select(axis, g.shape[axis] - 1 if step > 0 else 0).neg_()
    return g


def _hop(u, f, dag=False):
    out = torch.zeros_like(f)
    for mu in range(4):
        um = u[..., mu, :, :]
        s = -1 if dag else 1
        out += _spin(ONE - s * GAMMA[mu], _colour(um, _flip(f, mu, 1, AXIS[mu])))
        out += _spin(ONE + s * GAMMA[mu], _colour(torch.roll(um, 1, 3 - mu), _flip(f, mu, -1, AXIS[mu]), True))
    return out


def _field_strength(u, mu, nu):
    def sh(m, d, k):
        return torch.roll(m, -k, 3 - d)

    def dg(m):
        return m.conj().transpose(-1, -2)

    a, b = u[..., mu, :, :], u[..., nu, :, :]
    am, bm, an, bn = sh(a, mu, -1), sh(b, mu, -1), sh(a, nu, -1), sh(b, nu, -1)
    q = _mm3(_mm3(a, sh(b, mu, 1)), _mm3(dg(sh(a, nu, 1)), dg(b)))
    q = q + _mm3(_mm3(b, dg(sh(am, nu, 1))), _mm3(dg(bm), am))
    q = q + _mm3(_mm3(dg(am), dg(sh(bm, nu, -1))), _mm3(sh(am, nu, -1), bn))
    q = q + _mm3(_mm3(dg(bn), an), _mm3(sh(bn, mu, 1), dg(a)))
    return (q - dg(q)) / 8j


class _Wilson:
    """D, its even-odd pieces and its solve."""

    def __init__(self, u, kappa, csw):
        self.u, self.kappa, self.csw = u, kappa, csw
        self.f = []
        if csw:
            for mu in range(4):
                for nu in range(mu + 1, 4):
                    sg = (GAMMA[mu] @ GAMMA[nu] - GAMMA[nu] @ GAMMA[mu]) / 2j
                    self.f.append((sg * kappa * csw, _field_strength(u, mu, nu)))
        lt, lz, ly, lx = u.shape[:4]
        t, z, y, x = torch.meshgrid(*(torch.arange(n, device="cuda") for n in (lt, lz, ly, lx)), indexing="ij")
        self.par = ((x + y + z + t) & 1)[..., None, None]

    def only(self, f, p):
        return torch.where(self.par == p, f, torch.zeros((), dtype=f.dtype, device="cuda"))

    def a(self, f):
        out = f.clone()
        for sg, fs in self.f:
            out += _spin(sg, _colour(fs, f))
        return out

    def a_inv(self, f):
        """A is 1 + a small Hermitian part: a conjugate-gradient solve per site, to rounding."""
        if not self.f:
            return f.clone()
        x, r = torch.zeros_like(f), f.clone()
        p, rr = r.clone(), (r.abs() ** 2).sum((-1, -2), keepdim=True)
        for _ in range(40):
            q = self.a(p)
            al = rr / (p.conj() * q).real.sum((-1, -2), keepdim=True).clamp_min(1e-300)
            x += al * p
            r -= al * q
            rn = (r.abs() ** 2).sum((-1, -2), keepdim=True)
            if float(rn.max()) < 1e-34:
                break
            p = r + (rn / rr.clamp_min(1e-300)) * p
            rr = rn
        return x

    def d(self, f):
        return self.a(f) - self.kappa * _hop(self.u, f)

    def op(self, name, f):
        e, o = (lambda v: self.only(v, 0)), (lambda v: self.only(v, 1))
        if name == "D":
            return self.d(f)
        if name in ("HOP_EO", "DEO"):
            return e(_hop(self.u, o(f))) * (1 if name == "HOP_EO" else -self.kappa)
        if name == "HOP_OE":
            return o(_hop(self.u, e(f)))
        if name == "DOO_INV":
            return o(self.a_inv(o(f)))
        if name == "DPREC_SCHUR":
            return e(self.a(e(f)) - self.kappa ** 2 * _hop(self.u, o(self.a_inv(o(_hop(self.u, e(f)))))))
        raise ValueError(name)


def _sites(f):
    return tuple(range(f.dim() - 6, f.dim()))


def _bicgstab(apply, b, its=900):
    """apply(x) = b for every leading index of b, restarted from the true residual down to rounding."""
    dims = _sites(b)

    def dot(p, q):
        return (p.conj() * q).sum(dims, keepdim=True)

    x, bn, best = torch.zeros_like(b), dot(b, b).real.sqrt(), None
    for _ in range(3):
        r = b - apply(x)
        rel = float((dot(r, r).real.sqrt() / bn).max())
        if rel < 2e-15 or (best is not None and rel > 0.5 * best):
            break
        best = rel
        rh, p, e = r.clone(), r.clone(), torch.zeros_like(b)
        rho, r0 = dot(rh, r), dot(r, r).real
        for _ in range(its):
            v = apply(p)
            al = rho / dot(rh, v)
            s = r - al * v
            t = apply(s)
            om = dot(t, s) / dot(t, t)
            e += al * p + om * s
            r = s - om * t
            if float((dot(r, r).real / r0).max()) < 1e-26 or float((dot(r, r).real.sqrt() / bn).max()) < 1e-15:
                break
            rn = dot(rh, r)
            p = r + (rn / rho) * (al / om) * (p - om * v)
            rho = rn
        x += e
    return x


def _cg(apply, b, its=4000):
    """apply(x) = b, apply Hermitian and positive, to rounding."""
    x = torch.zeros_like(b)
    bb = float((b.abs() ** 2).sum())
    for _ in range(3):
        r = b - apply(x)
        rr = float((r.abs() ** 2).sum())
        if rr < 1e-30 * bb:
            break
        p, stop = r.clone(), max(1e-26 * rr, 1e-31 * bb)
        for _ in range(its):
            q = apply(p)
            al = rr / float((p.conj() * q).real.sum())
            x += al * p
            r = r - al * q
            rn = float((r.abs() ** 2).sum())
            if rn < stop:
                break
            p = r + (rn / rr) * p
            rr = rn
    return x


def _stag_hop(u, f):
    lt, lz, ly, lx = u.shape[:4]
    t, z, y, x = torch.meshgrid(*(torch.arange(n, device="cuda") for n in (lt, lz, ly, lx)), indexing="ij")
    out = torch.zeros_like(f)
    g = f.unsqueeze(-2)
    for mu, e in enumerate((0 * x, x, x + y, x + y + z)):
        um = u[..., mu, :, :]
        w = _colour(um, _flip(g, mu, 1, AXIS[mu])) - _colour(torch.roll(um, 1, 3 - mu), _flip(g, mu, -1, AXIS[mu]), True)
        out += 0.5 * (1 - 2 * (e & 1)).unsqueeze(-1) * w.squeeze(-2)
    return out


class _DomainWall:
    def __init__(self, u, b5, c5):
        self.u, self.b5, self.c5 = u, b5, c5

    def s(self, f, dag=False):
        up, dn = torch.roll(f, -1, 0), torch.roll(f, 1, 0)
        up[-1] *= -MF
        dn[0] *= -MF
        pp, pm = (ONE + GAMMA5) / 2, (ONE - GAMMA5) / 2
        return _spin(pp if dag else pm, up) + _spin(pm if dag else pp, dn)

    def d(self, f):
        w = self.b5 * f + self.c5 * self.s(f) if self.c5 else self.b5 * f
        return (4 - M5) * w - 0.5 * _hop(self.u, w) + f - self.s(f)

    def ddag(self, f):
        w = (4 - M5) * f - 0.5 * _hop(self.u, f, True)
        return self.b5 * w + self.c5 * self.s(w, True) + f - self.s(f, True)


def _half(f, p):
    """The sites of parity p of f [..., t, z, y, x, 12 or (4, 3)] in checkerboard order: [..., sites, 12]."""
    lead = f.dim() - 6
    lt, lz, ly, lx = f.shape[lead:lead + 4]
    g = f.reshape(f.shape[:lead] + (lt, lz, ly, lx // 2, 2, 12))
    t, z, y = torch.meshgrid(*(torch.arange(n, device="cuda") for n in (lt, lz, ly)), indexing="ij")
    odd = ((t + z + y + p) & 1).bool()[..., None, None]
    return torch.where(odd, g[..., 1, :], g[..., 0, :]).reshape(f.shape[:lead] + (-1, 12))


def _blocked(h, prec):
    """[sites, 12] in 64-site blocks, word-major inside a block, as the reals (FP16: codes and scales)."""
    n = h.shape[0]
    pad = -n % 64
    h = torch.cat([h, torch.zeros((pad, 12), dtype=C128, device="cuda")]).reshape(-1, 64, 12)
    scales = None
    if prec == "f16":
        r = torch.view_as_real(h).reshape(h.shape[0], 64, 24)
        scales = r.abs().amax(-1)
        h = h / scales.clamp_min(1e-300).unsqueeze(-1)
    per = {"f64": 1, "f32": 2, "f16": 4}[prec]
    w = h.reshape(-1, 64, 12 // per, per).transpose(1, 2).contiguous()
    w = torch.view_as_real(w)
    return w.reshape(-1) if scales is None else {"codes": w.reshape(w.shape[0], -1), "scales": scales}


MOST = 6_500_000  # complex numbers of a vector that a plain solve is done for


def exact(case, seed):
    kind, dims = case["kind"], _dims(case)
    v = math.prod(dims)
    if kind == "batch":
        d2, n = _dims(case, "second_"), case["nrhs"]
        if math.prod(d2) * 12 * n > MOST:
            return None
        w = _Wilson(_gauge(d2, seed + 500), case["kappa"], case["csw"])
        return [None, _bicgstab(w.d, _points(d2, n))]
    if kind in ("solve", "mg", "stag", "dwf_solve") and v * (3 if kind == "stag" else 12 * case.get("ls", 1)) > MOST:
        return None
    u = _gauge(dims, seed)
    if kind == "stag":
        lx, ly, lz, lt = dims
        b, m = _gauss((lt, lz, ly, lx, 3), seed), case["mass"]
        # D^dag D = m^2 - H^2, since H is anti-Hermitian
        return _cg(lambda f: m * m * f - _stag_hop(u, _stag_hop(u, f)), m * b - _stag_hop(u, b))
    if kind in ("dwf", "dwf_solve"):
        w = _DomainWall(u, case["b5"], case["c5"])
        b = _spinor(dims, seed, (case["ls"],))
        if kind == "dwf_solve":
            return _cg(lambda f: w.ddag(w.d(f)), w.ddag(b))
        o = w.ddag(b) if case["dag"] else w.d(b)
        return torch.cat([_blocked(_half(o, p).transpose(0, 1).reshape(-1, 12), case["prec"]) for p in (0, 1)])
    w = _Wilson(u, case["kappa"], case["csw"])
    b = _spinor(dims, seed)
    if kind in ("solve", "mg"):
        return _bicgstab(w.d, b)
    o = w.op(case["op"], b)
    if kind == "apply":
        return o
    return _blocked(_half(o, 1 if case["op"] == "HOP_OE" else 0), case["prec"])
