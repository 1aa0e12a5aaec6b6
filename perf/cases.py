"""Workloads of the two-flavour Wilson HMC library, one call (or one short sequence of calls) each.

A case is a plain dict: `kind` names the work, `t, z, y, x` the lattice extents (time first), `width` the spread of the
synthetic SU(3) links exp(i sum_a theta_a lambda_a / 2), theta_a ~ N(0, width^2), and the rest the options of the calls.
`listed()` are the named ones, `draw(rng)` gives one more of the same ranges, `prepare` makes what a program holds before
the call, `run` is one pass, `work` its unavoidable bytes and operations and `exact` the same outputs from plain torch in
64 bits.  Lattices: 4^4 (the checks), 12^3x24 and 16^3x32 (the ensembles of arXiv:1805.03560), 24^3x48 and 32^3x64 (the
solver and operator benchmarks), and extents that are no powers of two.
"""
import math
from fractions import Fraction

import torch

from paper_1805_03560_amd import whmc

DEV = "cuda:0"
PREC = {"f64": whmc.F64, "f32": whmc.F32, "f16": whmc.F16}


def _case(kind, dims, **kw):
    t, z, y, x = dims
    return dict(kind=kind, t=t, z=z, y=y, x=x, **kw)


def listed():
    return [
        # the smallest call: M^dag M on a 4^4 lattice, as checks and tiny test runs make it; launches and latency
        dict(_case("mdagm", (4, 4, 4, 4), width=1.0, eo=True, nrhs=1), name="mdagm_4x4"),
        # full-lattice M^dag M for two masses on a lattice whose extents are no powers of two
        dict(_case("mdagm", (18, 6, 10, 14), width=0.55, eo=False, nrhs=2), name="mdagm_full_ragged"),
        # the operator benchmark: H_eo then H_oe, FP64 with all link entries
        dict(_case("hop", (64, 32, 32, 32), width=0.3, prec="f64", links=18, dagger=False), name="hop_f64_32x64"),
        # the same in the single precision storage of a mixed solver, adjoint
        dict(_case("hop", (48, 24, 24, 24), width=0.3, prec="f32", links=12, dagger=True), name="hop_f32_24x48"),
        # many sources through one sweep of the links
        dict(_case("hopm", (48, 24, 24, 24), width=0.3, nrhs=12), name="hop_12rhs_24x48"),
        # a solve on the lattice of the paper's main runs, FP64
        dict(_case("cg", (24, 12, 12, 12), width=0.55, prec="f64", links=18, nrhs=1, kappa=0.15), name="cg_f64_12x24"),
        # the production solve of the largest lattice: FP16 bulk with FP64 residuals
        dict(_case("cg", (64, 32, 32, 32), width=0.3, prec="f16", links=12, nrhs=1, kappa=0.12), name="cg_f16_32x64"),
        # four masses at once, FP32 bulk
        dict(_case("cg", (48, 24, 24, 24), width=0.55, prec="f32", links=12, nrhs=4, kappa=0.145), name="cg_f32_4rhs_24x48"),
        # gauge and kappa^4-filtered pseudo-fermion force with FP64 solves: one outer force of the 16^3x32 runs
        dict(_case("force", (32, 16, 16, 16), width=0.55, n_t=15, kappa=0.145), name="force_16x32"),
        # the inner level of the integrator on the largest lattice: gauge force, P step, T step
        dict(_case("gauge", (64, 32, 32, 32), width=0.3), name="gauge_step_32x64"),
        # a configuration and sources from and to the canonical layouts: load, check, pack, unpack, export
        dict(_case("io", (48, 24, 24, 24), width=0.55, nrhs=4), name="import_export_24x48"),
        # a whole call: molecular dynamics of the paper's 12^3x24 runs (kappa^4 filter, Omelyan, mixed solves)
        dict(_case("md", (24, 12, 12, 12), width=0.55, n_t=15, kappa=0.145, m=2, m0=4), name="md_12x24"),
    ]


# sites of a drawn lattice, per kind: from the smallest a program would use to the listed one
_SITES = {"mdagm": (256, 32 ** 3 * 64), "hop": (2048, 32 ** 3 * 64), "hopm": (2048, 24 ** 3 * 48),
          "cg": (2048, 24 ** 3 * 48), "force": (2048, 16 ** 3 * 32), "gauge": (2048, 32 ** 3 * 64),
          "io": (2048, 24 ** 3 * 48), "md": (1024, 12 ** 3 * 24)}


def _draw_dims(rng, lo, hi):
    """even extents, time the longest or near it, with a volume spread over its logarithm"""
    want = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    for _ in range(10000):
        side = (want / 2) ** 0.25
        d = [max(4, 2 * round(side * f * rng.uniform(0.7, 1.4) / 2)) for f in (2, 1, 1, 1)]
        if 0.7 * want <= math.prod(d) <= min(1.4 * want, hi):
            return d
    return [4, 4, 4, 4]


def draw(rng):
    kind = rng.choice(sorted(_SITES))
    dims = _draw_dims(rng, *_SITES[kind])
    if kind == "mdagm":
        return _case(kind, dims, width=rng.choice([0.3, 0.55, 1.0]), eo=rng.random() < 0.6, nrhs=rng.choice([1, 1, 2, 3]))
    if kind == "hop":
        prec = rng.choice(["f64", "f64", "f32"])
        return _case(kind, dims, width=rng.choice([0.3, 0.55]), prec=prec, links=rng.choice([18, 12, 8]),
                     dagger=rng.random() < 0.5)
    if kind == "hopm":
        return _case(kind, dims, width=0.3, nrhs=rng.choice([2, 3, 4, 6, 8, 12]))
    if kind == "cg":
        return _case(kind, dims, width=0.55, prec=rng.choice(["f64", "f32", "f16"]), links=12,
                     nrhs=rng.choice([1, 1, 2, 4, 5]), kappa=round(rng.uniform(0.13, 0.148), 4))
    if kind == "force":
        return _case(kind, dims, width=0.55, n_t=rng.choice([7, 11, 15]), kappa=round(rng.uniform(0.13, 0.148), 4))
    if kind == "gauge":
        return _case(kind, dims, width=rng.choice([0.3, 0.55]))
    if kind == "io":
        return _case(kind, dims, width=rng.choice([0.3, 0.55]), nrhs=rng.choice([1, 2, 3, 4]))
    return _case(kind, dims, width=0.55, n_t=rng.choice([7, 15]), kappa=round(rng.uniform(0.13, 0.146), 4),
                 m=rng.choice([1, 2]), m0=rng.choice([2, 4]))


# ------------------------------------------------------------------ inputs
def _dims(c):
    return (c["t"], c["z"], c["y"], c["x"])


def _rng(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _mm(a, b):
    """product of 3x3 matrices, elementwise (no batched library product)"""
    return sum(a[..., :, k:k + 1] * b[..., k:k + 1, :] for k in range(3))


def _algebra(c):
    """sum_a c_a T_a, T_a = i lambda_a / 2"""
    s = 1 / math.sqrt(3.0)
    d0, d1, d2 = 0.5 * (c[..., 2] + s * c[..., 7]), 0.5 * (-c[..., 2] + s * c[..., 7]), -s * c[..., 7]
    z = torch.zeros_like(d0)
    re = torch.stack([z, 0.5 * c[..., 1], 0.5 * c[..., 4], -0.5 * c[..., 1], z, 0.5 * c[..., 6], -0.5 * c[..., 4],
                      -0.5 * c[..., 6], z], -1)
    im = torch.stack([d0, 0.5 * c[..., 0], 0.5 * c[..., 3], 0.5 * c[..., 0], d1, 0.5 * c[..., 5], 0.5 * c[..., 3],
                      0.5 * c[..., 5], d2], -1)
    return torch.complex(re, im).reshape(c.shape[:-1] + (3, 3))


def _exp(A):
    """exp of antihermitian 3x3 matrices: Taylor series of A / 2^s and s squarings"""
    n = float(A.abs().max()) * 3
    s = max(0, math.ceil(math.log2(max(n, 1e-3) / 0.25)))
    B, one = A * 2.0 ** -s, torch.eye(3, dtype=A.dtype, device=A.device)
    E = one + B / 14
    for k in range(13, 0, -1):
        E = one + _mm(B, E) / k
    for _ in range(s):
        E = _mm(E, E)
    return E


def _links(c, seed):
    n = math.prod(_dims(c)) * 4
    out = torch.empty((n, 3, 3), dtype=torch.complex128, device=DEV)
    g = _rng(seed * 10 + 1)
    for lo in range(0, n, 1 << 21):
        hi = min(n, lo + (1 << 21))
        out[lo:hi] = _exp(_algebra(c["width"] * torch.randn((hi - lo, 8), generator=g, dtype=torch.float64, device=DEV)))
    return out.reshape(_dims(c) + (4, 3, 3))


def _spinors(shape, seed):
    """complex Gaussian with density exp(-|eta|^2)"""
    r = torch.randn(tuple(shape) + (2,), generator=_rng(seed), dtype=torch.float64, device=DEV)
    return torch.view_as_complex(r) * math.sqrt(0.5)


def _sources(c, seed):
    """canonical source fields of a case"""
    v = math.prod(_dims(c))
    if c["kind"] == "mdagm":
        return _spinors((c["nrhs"], v // 2 if c["eo"] else v, 4, 3), seed * 10 + 2)
    if c["kind"] == "io":
        return _spinors((c["nrhs"], v, 4, 3), seed * 10 + 2)
    return _spinors((c.get("nrhs", 1), v // 2, 4, 3), seed * 10 + 2)


def _momenta(c, seed):
    return torch.randn(_dims(c) + (4, 8), generator=_rng(seed * 10 + 3), dtype=torch.float64, device=DEV)


def _kappas(c):
    """target hopping parameter first, then heavier ones, as in mass preconditioning"""
    k = c.get("kappa", 0.156)
    return [k - 0.003 * r for r in range(c["nrhs"])]


_BETA = 5.6


def _md_params(c):
    md = whmc.cg_params(tol=1e-11, prec=whmc.F16, links=whmc.L12, delta=1e-2)
    return whmc.hmc_params(beta=_BETA, kappa=c["kappa"], k=2, n_t=c["n_t"], n_max=29, integrator=whmc.OMELYAN,
                           m=c["m"], m0=c["m0"], tau=0.2 * c["m"], md_solver=md)


def prepare(case, seed):
    c, kind = case, case["kind"]
    ctx = whmc.Context(_dims(c))
    U = _links(c, seed)
    s = {"case": c, "ctx": ctx}
    if kind != "io":
        ctx.load_gauge(U, unitarity_tol=1e-11)
    if kind == "mdagm":
        s["in"] = ctx.pack_spinor(_sources(c, seed), 0 if c["eo"] else -1)
        s["out"] = torch.empty_like(s["in"])
        s["kappas"] = _kappas(c)
    elif kind == "hop":
        p = PREC[c["prec"]]
        ctx.autotune_hop()   # once per lattice, as the benchmark does
        s["in"] = ctx.convert_spinor(ctx.pack_spinor(_sources(c, seed), 1), whmc.F64, p)
        s["out"] = [ctx.half_spinor(p), ctx.half_spinor(p)]
    elif kind == "hopm":
        ctx.autotune(whmc.F64, whmc.L18, c["nrhs"])
        s["in"] = ctx.pack_spinor(_sources(c, seed), 1)
        s["out"] = torch.empty_like(s["in"])
    elif kind == "cg":
        ctx.autotune_hop()
        s["in"] = ctx.pack_spinor(_sources(c, seed), 1)
        s["out"] = torch.empty_like(s["in"])
        s["params"] = (whmc.cg_params(tol=1e-12, links=c["links"]) if c["prec"] == "f64" else
                       whmc.cg_params(tol=1e-11, prec=PREC[c["prec"]], links=c["links"],
                                      delta=1e-4 if c["prec"] == "f32" else 1e-2))
        s["kappas"] = _kappas(c)
    elif kind == "force":
        ctx.autotune_hop()
        s["in"] = ctx.pack_spinor(_sources(c, seed), 1)
        s["out"] = ctx.algebra()
    elif kind == "gauge":
        s["in"] = ctx.pack_algebra(_momenta(c, seed))
        s["pi"], s["F"] = torch.empty_like(s["in"]), ctx.algebra()
    elif kind == "io":
        s["U"], s["in"], s["pi"] = U, _sources(c, seed), _momenta(c, seed)
    elif kind == "md":
        ctx.autotune_hop()
        s["U"], s["in"] = U, ctx.pack_spinor(_sources(c, seed), 1)
        s["pi0"] = ctx.pack_algebra(_momenta(c, seed))
        s["pi"], s["params"] = torch.empty_like(s["pi0"]), _md_params(c)
    else:
        raise ValueError(kind)
    return s


# ------------------------------------------------------------------ one pass
def run(s):
    c, ctx, kind = s["case"], s["ctx"], s["case"]["kind"]
    if kind == "mdagm":
        return ctx.apply_MdagM(s["in"], s["kappas"], out=s["out"], eo=c["eo"])
    if kind == "hop":
        p = PREC[c["prec"]]
        e = ctx.apply_H(s["in"], 0, dagger=c["dagger"], prec=p, links=c["links"], out=s["out"][0])
        return e, ctx.apply_H(e, 1, dagger=c["dagger"], prec=p, links=c["links"], out=s["out"][1])
    if kind == "hopm":
        return ctx.apply_H_multi(s["in"], 0, c["nrhs"], out=s["out"])
    if kind == "cg":
        return ctx.cg_solve(s["in"], s["kappas"], s["params"], x=s["out"])[0]
    if kind == "force":
        return ctx.force(s["in"], 2, c["n_t"], 29, c["kappa"], _BETA, flags=whmc.FORCE_PF | whmc.FORCE_GAUGE, out=s["out"])
    if kind == "gauge":
        s["pi"].copy_(s["in"])
        ctx.force(None, 2, 0, 0, 0.156, _BETA, flags=whmc.FORCE_GAUGE, out=s["F"])
        ctx.update_momenta(s["pi"], s["F"], 0.02)
        ctx.update_links(s["pi"], 0.02)
        ctx.force(None, 2, 0, 0, 0.156, _BETA, flags=whmc.FORCE_GAUGE, out=s["F"])
        ctx.update_links(s["pi"], -0.02)   # back, so that the links stay those of the state
        ctx.update_momenta(s["pi"], s["F"], 0.02)
        return s["F"], s["pi"]
    if kind == "io":
        ctx.load_gauge(s["U"], unitarity_tol=1e-11)
        b = ctx.pack_spinor(s["in"], -1)
        p = ctx.pack_algebra(s["pi"])
        return b, ctx.unpack_spinor(b, -1, c["nrhs"]), p, ctx.unpack_algebra(p), ctx.export_gauge()
    ctx.load_gauge(s["U"], unitarity_tol=0.0)
    s["pi"].copy_(s["pi0"])
    ctx.md_integrate(s["params"], s["pi"], s["in"])
    return s["pi"], ctx.export_gauge()


# ------------------------------------------------------------------ unavoidable work
# an even/odd hop: each output site reads its eight links and (once) a spinor and writes one; 1320 operations
_SPINOR = {"f64": 192, "f32": 96, "f16": 52}
_REAL = {"f64": 8, "f32": 4, "f16": 2}


def _hop(vh, prec="f64", links=18, nrhs=1):
    return {"bytes": vh * (8 * links * _REAL[prec] + 2 * nrhs * _SPINOR[prec]), "flops": 1320.0 * vh * nrhs}


def _plus(*ws):
    return {k: float(sum(w[k] for w in ws)) for k in ("bytes", "flops")}


def _times(n, w):
    return {k: n * v for k, v in w.items()}


def _solve(vh, prec, links, nrhs, iters):
    """iters steps of conjugate gradients: four hops and the vector updates of p, r and x"""
    v = {"bytes": 6 * nrhs * vh * _SPINOR[prec], "flops": 240.0 * nrhs * vh}
    return _times(iters, _plus(_times(4, _hop(vh, prec, links, nrhs)), v))


def _iters(c):
    """steps that a solve of these kappas and widths takes, about"""
    return 60 if c["width"] < 0.5 else 100


def work(case):
    c, kind = case, case["kind"]
    v = math.prod(_dims(c))
    vh = v // 2
    lk, alg = v * 4 * 144, v * 4 * 64   # links and an algebra field
    gauge = {"bytes": lk + alg, "flops": v * 4 * 2800.0}
    links = {"bytes": 2 * lk + alg, "flops": v * 4 * 1500.0}
    if kind == "mdagm":
        # two applications of M, each with its links and spinors once
        if c["eo"]:
            return _times(4, _hop(vh, nrhs=c["nrhs"]))
        return _times(2, {"bytes": lk + c["nrhs"] * 2 * v * 192, "flops": 1368.0 * v * c["nrhs"]})
    if kind == "hop":
        return _times(2, _hop(vh, c["prec"], c["links"]))
    if kind == "hopm":
        return _hop(vh, nrhs=c["nrhs"])
    if kind == "cg":
        return _solve(vh, c["prec"], c["links"], c["nrhs"], _iters(c))
    force = _plus(_times(4 * c.get("n_t", 0), _hop(vh)), {"bytes": (c.get("n_t", 0) + 1) * 2 * v * 192 + lk + alg,
                                                         "flops": (c.get("n_t", 0) + 1) * v * 4 * 400.0})
    if kind == "force":
        return _plus(_solve(vh, "f64", 18, 2, _iters(c)), force, gauge)
    if kind == "gauge":
        return _plus(_times(2, gauge), _times(2, links), {"bytes": 8 * alg, "flops": 0})
    if kind == "io":
        return {"bytes": float(4 * lk + 4 * alg + 4 * c["nrhs"] * v * 192), "flops": 0.0}
    n_pf, n_g = 2 * c["m"] + 1, 4 * c["m"] * c["m0"] + 1
    return _plus(_times(n_pf, _plus(_solve(vh, "f16", 12, 2, _iters(c)), force)), _times(n_g, _plus(gauge, links)),
                 {"bytes": 4 * lk + 2 * alg, "flops": 0})


# ------------------------------------------------------------------ the same in plain torch, 64 bits
# gamma_mu psi: row s is coef * psi[perm]; gamma_0 = [[0,1],[1,0]], gamma_k = [[0,-i s_k],[i s_k,0]]
_GAMMA = [([2, 3, 0, 1], [1, 1, 1, 1]), ([3, 2, 1, 0], [-1j, -1j, 1j, 1j]),
          ([3, 2, 1, 0], [-1, 1, 1, -1]), ([2, 3, 0, 1], [-1j, 1j, 1j, -1j])]


def _gamma(mu, psi):
    perm, coef = _GAMMA[mu]
    return psi[..., perm, :] * torch.tensor(coef, dtype=psi.dtype, device=psi.device)[:, None]


def _shift(f, mu, d, fermion=True):
    """f(x + d mu); fermions change sign across the time boundary"""
    out = torch.roll(f, -d, dims=mu)
    if fermion and mu == 0:
        out[-1 if d > 0 else 0] *= -1
    return out


def _mv(U, psi):
    return sum(U[..., None, :, k] * psi[..., k:k + 1] for k in range(3))


def _dag(U):
    return U.mH


def _h(U, psi, dagger=False):
    """H psi (H^dag psi) on the full lattice"""
    sg = -1 if dagger else 1
    out = torch.zeros_like(psi)
    for mu in range(4):
        Um = U[..., mu, :, :]
        v = _mv(Um, _shift(psi, mu, 1))
        out += v - sg * _gamma(mu, v)
        v = _shift(_mv(_dag(Um), psi), mu, -1)
        out += v + sg * _gamma(mu, v)
    return out


def _sites(dims):
    """canonical indices of the even and of the odd sites, in checkerboard order"""
    g = torch.meshgrid(*[torch.arange(d, device=DEV) for d in dims], indexing="ij")
    p = (sum(g) % 2).reshape(-1)
    return [torch.nonzero(p == q).reshape(-1) for q in (0, 1)]


class _Exact:
    def __init__(self, c, seed):
        self.c, self.dims, self.U = c, _dims(c), _links(c, seed)
        self.V = math.prod(self.dims)
        self.idx = _sites(self.dims)

    def full(self, half, p):
        out = torch.zeros((self.V, 4, 3), dtype=torch.complex128, device=DEV)
        out[self.idx[p]] = half
        return out.reshape(self.dims + (4, 3))

    def half(self, full, p):
        return full.reshape(self.V, 4, 3)[self.idx[p]]

    def hop(self, half, p, dagger=False):
        """the block of H onto parity p"""
        return self.half(_h(self.U, self.full(half, 1 - p), dagger), p)

    def K(self, x, k, dagger=False):
        return k * k * self.hop(self.hop(x, 0, dagger), 1, dagger)

    def A(self, x, k):
        u = x - self.K(x, k)
        return u - self.K(u, k, True)

    def solve(self, b, k):
        x, r = torch.zeros_like(b), b.clone()
        p, rr = r.clone(), r.abs().square().sum()
        stop = rr * 1e-28
        for _ in range(3000):
            ap = self.A(p, k)
            al = rr / torch.sum(p.conj() * ap).real
            x += al * p
            r -= al * ap
            new = r.abs().square().sum()
            p = r + (new / rr) * p
            rr = new
            if float(rr) <= float(stop):
                break
        return x

    # forces: coordinates f_a = Im Tr(lambda_a G) of the traceless antihermitian part of G
    def coords(self, G):
        s = 1 / math.sqrt(3.0)
        g = lambda a, b: G[..., a, b]   # noqa: E731
        return torch.stack([g(0, 1).imag + g(1, 0).imag, g(0, 1).real - g(1, 0).real, g(0, 0).imag - g(1, 1).imag,
                            g(0, 2).imag + g(2, 0).imag, g(0, 2).real - g(2, 0).real, g(1, 2).imag + g(2, 1).imag,
                            g(1, 2).real - g(2, 1).real, s * (g(0, 0).imag + g(1, 1).imag - 2 * g(2, 2).imag)], -1)

    def gauge_force(self, beta):
        out = []
        for mu in range(4):
            S, Um = 0, self.U[..., mu, :, :]
            for nu in range(4):
                if nu != mu:
                    Un = self.U[..., nu, :, :]
                    S = S + _mm(_mm(_shift(Un, mu, 1, False), _dag(_shift(Um, nu, 1, False))), _dag(Un))
                    S = S + _shift(_mm(_mm(_dag(_shift(Un, mu, 1, False)), _dag(Um)), Un), nu, -1, False)
            out.append(beta / 6 * self.coords(_mm(Um, S)))
        return torch.stack(out, -2)

    def pair(self, X, Y):
        """sum over the spins of U (1 - g) Y(x+mu) X(x)^dag - (1 + g) Y(x) X(x+mu)^dag U^dag for all links"""
        out = []
        for mu in range(4):
            Yf, Xf, Um = _shift(Y, mu, 1), _shift(X, mu, 1), self.U[..., mu, :, :]
            a, b = Yf - _gamma(mu, Yf), Y + _gamma(mu, Y)
            Q = sum(a[..., s, :, None] * X[..., s, None, :].conj() for s in range(4))
            R = sum(b[..., s, :, None] * Xf[..., s, None, :].conj() for s in range(4))
            out.append(_mm(Um, Q) - _mm(R, _dag(Um)))
        return torch.stack(out, -3)

    def pf_force(self, phi, k, n_t):
        """force of |M~^{-1} phi|^2 with the kappa^4 filter, series truncated at n_t"""
        n = n_t + 60
        e = [Fraction(1)]
        for m in range(1, n + 1):
            e.append(-sum(e[m - j] for j in (1, 2) if j <= m) / m)
        b = [-float(sum(e[m + 1:])) for m in range(n_t + 1)]
        alpha = math.exp(-1.5)
        Y = [None] * (n_t + 1)
        Y[n_t] = b[n_t] * phi
        for i in range(n_t, 0, -1):
            Y[i - 1] = b[i - 1] * phi + self.K(Y[i], k)
        g5 = torch.tensor([-1, -1, 1, 1], dtype=phi.dtype, device=DEV)[:, None]
        s2, s3 = self.solve(Y[0], k), self.solve(g5 * phi, k)
        Yt = alpha * (g5 * s3 - self.K(g5 * s3, k, True))
        Xt = s2 - self.K(s2, k) + alpha * g5 * s3
        X = Y[0] + Yt
        pairs = [(Xt, Yt)]
        for i in range(1, n_t + 1):
            pairs.append((X, Y[i]))
            X = self.K(X, k, True)
        G = 0
        for x, y in pairs:
            G = G + self.pair(self.full(self.hop(x, 0, True), 0) + self.full(x, 1),
                              self.full(self.hop(y, 0), 0) + self.full(y, 1))
        return -k * k * self.coords(G)

    # device layouts: 64-site blocks of K entries per site; algebra fields [parity][mu][a][site]
    def pack(self, x, w=2):
        r = torch.view_as_real(x.reshape(-1, 12)).reshape(x.shape[0], 24 // w, w)
        n = x.shape[0] // 64 * 64
        a = r[:n].reshape(-1, 64, 24 // w, w).transpose(1, 2).reshape(-1)
        return torch.cat([a, r[n:].transpose(0, 1).reshape(-1)])

    def pack_full(self, x):
        return torch.cat([self.pack(x.reshape(-1, 4, 3)[self.idx[p]]) for p in (0, 1)])

    def pack_algebra(self, f):
        f = f.reshape(self.V, 4, 8)
        return torch.cat([f[self.idx[p]].permute(1, 2, 0).reshape(-1) for p in (0, 1)])


def exact(case, seed):
    c, kind = case, case["kind"]
    E = _Exact(c, seed)
    if kind == "mdagm":
        out = []
        for x, k in zip(_sources(c, seed), _kappas(c)):
            if c["eo"]:
                out.append(E.pack(E.A(x, k)))
            else:
                x = x.reshape(E.dims + (4, 3))
                u = x - k * _h(E.U, x)
                out.append(E.pack_full(u - k * _h(E.U, u, True)))
        return torch.cat(out)
    if kind == "hop":
        w = 2 if c["prec"] == "f64" else 4
        x = _sources(c, seed)[0]
        if c["prec"] == "f32":
            x = x.to(torch.complex64).to(torch.complex128)
        e = E.hop(x, 0, c["dagger"])
        return E.pack(e, w), E.pack(E.hop(e, 1, c["dagger"]), w)
    if kind == "hopm":
        return torch.cat([E.pack(E.hop(x, 0)) for x in _sources(c, seed)])
    if kind == "cg":
        return torch.cat([E.pack(E.solve(x, k)) for x, k in zip(_sources(c, seed), _kappas(c))])
    if kind == "force":
        f = E.gauge_force(_BETA + 96 * c["kappa"] ** 4)
        return E.pack_algebra(f + E.pf_force(_sources(c, seed)[0], c["kappa"], c["n_t"]))
    if kind == "gauge":
        beta = _BETA + 96 * 0.156 ** 4
        pi = _momenta(c, seed) - 0.02 * E.gauge_force(beta)
        for t in range(c["t"]):   # a time slice at a time
            E.U[t] = _mm(_exp(0.02 * _algebra(pi[t])), E.U[t])
        f = E.gauge_force(beta)
        return E.pack_algebra(f), E.pack_algebra(pi - 0.02 * f)
    if kind == "io":
        s, p = _sources(c, seed), _momenta(c, seed)
        return torch.cat([E.pack_full(x) for x in s]), s if c["nrhs"] > 1 else s[0], E.pack_algebra(p), p, E.U
    # Omelyan (lambda = 1/6): P steps of the pseudo-fermion force around m0 gauge steps in each half
    beta, phi, pi = _BETA + 96 * c["kappa"] ** 4, _sources(c, seed)[0], _momenta(c, seed)
    lam, dt = 1.0 / 6.0, 0.2

    def inner(pi, span):
        h = span / c["m0"]
        for _ in range(c["m0"]):
            pi = pi - lam * h * E.gauge_force(beta)
            E.U = _mm(_exp(h / 2 * _algebra(pi)), E.U)
            pi = pi - (1 - 2 * lam) * h * E.gauge_force(beta)
            E.U = _mm(_exp(h / 2 * _algebra(pi)), E.U)
            pi = pi - lam * h * E.gauge_force(beta)
        return pi

    F = E.pf_force(phi, c["kappa"], c["n_t"])
    for _ in range(c["m"]):
        pi = inner(pi - lam * dt * F, dt / 2)
        pi = inner(pi - (1 - 2 * lam) * dt * E.pf_force(phi, c["kappa"], c["n_t"]), dt / 2)
        F = E.pf_force(phi, c["kappa"], c["n_t"])
        pi = pi - lam * dt * F
    return E.pack_algebra(pi), E.U
