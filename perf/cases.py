"""The work that users of this library have it do, as cases to be timed.

Three kinds of case, each through the public Python entry points:

* ``apply``: one application of D_S, D_W or D_B (or its adjoint) to a block of
  N_v right-hand sides, into a buffer that the program keeps.  Forms: plain
  links, two-row compressed links (D_S, D_W), with the clover term (D_W).
* ``step``: one differentiable step.  The operator is applied with gradients
  on, and the gradients with respect to the links V and to the right-hand
  sides follow for a given upstream gradient.  For D_B the step runs through
  the construction of the off-axis links W.
* ``solve``: the mixed-precision solve of D x = b.

Lattices are written (nx, ny, nz, nt).  They go from 8^4, where a call is
mostly latency, to 34^3 x 68, the lattice of the figures of the paper
(arXiv:1808.05506).  Links are SU(3): Haar-distributed (a rough field) or
near 1 (a smeared field); right-hand sides are complex Gaussian noise of unit
variance, as stochastic sources are.  All fields are drawn on the GPU.
"""
from __future__ import annotations

import itertools
import math

import torch

from paper_1808_05506_amd import dslash as D

MASS = {"staggered": 0.1, "wilson": 0.1, "brillouin": 0.1}
SOLVE_MASS = {"staggered": 0.2, "wilson": 0.05}
C_SW = 1.0
# Inner tolerances of the solves, the ones that are fastest for each storage.
INNER_TOL = {(False, "c64"): 3e-4, (False, "bf16"): 0.02, (False, "f16"): 2e-3,
             (True, "c64"): 3e-4, (True, "bf16"): 5e-3, (True, "f16"): 5e-3}
SOLVE_TOL = 1e-12
WORD = {"c64": 8, "c128": 16, "bf16": 4, "f16": 4}          # bytes of a complex number
HOP_FLOPS = {"staggered": 570, "wilson": 1320, "brillouin": 28224}   # per site and right-hand side
LINK_WORDS = {"staggered": 36, "wilson": 36, "brillouin": 360}


def _apply(name, op, nx, ny, nz, nt, nv, dtype, adjoint=False, form="plain", links="smooth"):
    return {"name": name, "kind": "apply", "op": op, "nx": nx, "ny": ny, "nz": nz, "nt": nt, "nv": nv,
            "dtype": dtype, "adjoint": adjoint, "form": form, "links": links}


def _step(name, op, nx, ny, nz, nt, nv, dtype, links="smooth"):
    return {"name": name, "kind": "step", "op": op, "nx": nx, "ny": ny, "nz": nz, "nt": nt, "nv": nv,
            "dtype": dtype, "links": links}


def _solve(name, op, nx, ny, nz, nt, nv, inner, eo, links="smooth"):
    return {"name": name, "kind": "solve", "op": op, "nx": nx, "ny": ny, "nz": nz, "nt": nt, "nv": nv,
            "inner": inner, "eo": eo, "links": links}


def listed():
    return [
        # The smallest call: D_S on a test-size lattice with few right-hand sides (an inner loop of small calls).
        _apply("ds_8_nv4", "staggered", 8, 8, 8, 8, 4, "c64", links="haar"),
        # D_S with the twelve right-hand sides of the paper on a production-size box.
        _apply("ds_32_nv12", "staggered", 32, 32, 32, 32, 12, "c64", links="haar"),
        # The paper's Wilson operator on a medium lattice: twelve columns, one propagator.
        _apply("dw_16x32_nv12", "wilson", 16, 16, 16, 32, 12, "c64"),
        # The same on the paper's own lattice, the largest call; 34 is no multiple of a power of two.
        _apply("dw_34x68_nv12", "wilson", 34, 34, 34, 68, 12, "c64"),
        # D_W^dag in double precision: residuals, and the normal equations of a double-precision solver.
        _apply("dw_24x48_nv12_c128", "wilson", 24, 24, 24, 48, 12, "c128", adjoint=True),
        # Wilson-clover, the usual production action, on a box whose extents all differ.
        _apply("dw_clover_ragged_nv12", "wilson", 18, 14, 20, 26, 12, "c64", form="clover"),
        # An odd lattice and an odd block: what is left of a sweep over sources.
        _apply("dw_odd_nv5", "wilson", 21, 15, 13, 27, 5, "c64"),
        # The Brillouin operator in single precision, W stored.
        _apply("db_32_nv12", "brillouin", 32, 32, 32, 32, 12, "c64", links="haar"),
        # The Brillouin operator in double precision.
        _apply("db_16x32_nv12_c128", "brillouin", 16, 16, 16, 32, 12, "c128", links="haar"),
        # A differentiable Wilson layer: forward, gradients of links and right-hand sides.
        _step("dw_step_24x48_nv12", "wilson", 24, 24, 24, 48, 12, "c64"),
        # A differentiable Brillouin layer on changing links: W construction, D_B, and both gradients back to V.
        _step("db_step_16x32_nv12", "brillouin", 16, 16, 16, 32, 12, "c64", links="haar"),
        # A propagator: twelve columns of D_W x = b on the checkerboard, 16-bit inner solve.
        _solve("solve_eo_16x32_nv12", "wilson", 16, 16, 16, 32, 12, "f16", True),
    ]


def _volume(case):
    return case["nx"] * case["ny"] * case["nz"] * case["nt"]


def _extents(rng, lo, hi, even):
    """Four extents of a volume spread over its logarithm, the time extent up to twice the longest other."""
    while True:
        side = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        ext = [min(34, max(lo, round(side * rng.uniform(0.75, 1.3)))) for _ in range(3)]
        ext.append(min(68, max(lo, round(side * rng.uniform(0.8, 2.0)))))
        if even:
            ext = [e + e % 2 for e in ext]
        if lo ** 4 <= math.prod(ext):
            return ext


def _unnamed(case):
    return {k: v for k, v in case.items() if k != "name"}


def draw(rng):
    kind = rng.choice(["apply", "apply", "apply", "apply", "step", "solve"])
    nv = rng.choice([12, 12, rng.randint(1, 24), rng.randint(1, 24), rng.choice([1, 4, 8, 16, 24])])
    if kind == "solve":
        op = rng.choice(["wilson", "wilson", "wilson", "staggered"])
        eo = op == "wilson" and rng.random() < 0.6
        nx, ny, nz, nt = _extents(rng, 8, 17, True)
        return _unnamed(_solve("", op, nx, ny, nz, nt, min(nv, 12), rng.choice(["c64", "bf16", "f16"]), eo))
    op = rng.choice(["staggered", "wilson", "wilson", "brillouin"])
    if kind == "step":
        dtype = rng.choice(["c64", "c64", "c128"])
        top = 17 if op == "brillouin" else 26
        nx, ny, nz, nt = _extents(rng, 8, top, op == "staggered")
        case = _step("", op, nx, ny, nz, nt, min(nv, 12), dtype, rng.choice(["smooth", "haar"]))
    else:
        dtype = rng.choice(["c64", "c64", "c64", "c128", "c128", "bf16", "f16"])
        if op == "brillouin":
            dtype = rng.choice(["c64", "c64", "c128"])
        top = {"staggered": 34, "wilson": 34, "brillouin": 20}[op] if dtype != "c128" else 22
        nx, ny, nz, nt = _extents(rng, 8, top, op == "staggered")
        form = rng.choice(["plain", "plain", "plain", {"staggered": "compressed", "wilson": "clover"}.get(op, "plain"),
                           "plain" if op == "brillouin" else "compressed"])
        case = _apply("", op, nx, ny, nz, nt, nv, dtype, rng.random() < 0.4, form, rng.choice(["smooth", "haar"]))
    if work(case)["flops"] > 3.5e11 or work(case)["bytes"] > 6.9e9:
        return draw(rng)
    return _unnamed(case)


# --- fields -----------------------------------------------------------------

def _gaussian(shape, gen):
    """Complex Gaussian of unit variance, complex64."""
    return torch.randn(shape, dtype=torch.complex64, device="cuda", generator=gen)


def _su3(n, kind, gen):
    """n SU(3) matrices, complex128: Gram-Schmidt on Gaussian rows (Haar), or on those of 1 and small noise (near 1)."""
    z = _gaussian((n, 2, 3), gen).to(torch.complex128)
    if kind == "smooth":
        z = 0.15 * z
        z[:, 0, 0] += 1.0
        z[:, 1, 1] += 1.0
    a = z[:, 0] / z[:, 0].abs().square().sum(-1, keepdim=True).sqrt()
    b = z[:, 1] - (a.conj() * z[:, 1]).sum(-1, keepdim=True) * a
    b = b / b.abs().square().sum(-1, keepdim=True).sqrt()
    c = torch.stack([a[:, (j + 1) % 3] * b[:, (j + 2) % 3] - a[:, (j + 2) % 3] * b[:, (j + 1) % 3] for j in range(3)],
                    dim=-1).conj()
    return torch.stack([a, b, c], dim=1)


def _store(x, dtype):
    """x in the storage of ``dtype``."""
    if dtype in ("c64", "c128"):
        return x.to(torch.complex64 if dtype == "c64" else torch.complex128).contiguous()
    return torch.view_as_real(x.to(torch.complex64)).to(torch.bfloat16 if dtype == "bf16" else torch.float16).contiguous()


def _wide(x):
    """A stored field in complex128."""
    if x.is_complex():
        return x.to(torch.complex128)
    return torch.view_as_complex(x.to(torch.float64).contiguous())


def _fields(case, seed, dtype):
    """Links and right-hand sides (and, for a step, the upstream gradient) in storage ``dtype``."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    lat = (case["nt"], case["nz"], case["ny"], case["nx"])
    n = math.prod(lat) * 4
    V = torch.empty((n, 3, 3), dtype=torch.complex128 if dtype == "c128" else torch.complex64, device="cuda")
    for i in range(0, n, 1 << 21):          # in pieces, for the memory
        V[i:i + (1 << 21)] = _su3(min(1 << 21, n - i), case["links"], gen).to(V.dtype)
    V = _store(V.view(lat + (4, 3, 3)), dtype)
    shape = lat + ((3, case["nv"]) if case["op"] == "staggered" else (4, 3, case["nv"]))
    psi = _store(_gaussian(shape, gen), dtype)
    g = _store(_gaussian(shape, gen), dtype) if case["kind"] == "step" else None
    return V, psi, g


def prepare(case, seed):
    if case["kind"] == "solve":
        V, b, _ = _fields(case, seed, "c128")
        return {"case": case, "U": V, "b": b}
    V, psi, g = _fields(case, seed, case["dtype"])
    if case["kind"] == "step":
        return {"case": case, "V": V.requires_grad_(), "psi": psi.requires_grad_(), "g": g}
    state = {"case": case, "U": V, "psi": psi, "out": torch.empty_like(psi), "clover": None}
    if case["op"] == "brillouin":
        state["U"] = D.brillouin_links(V)
    elif case["form"] == "clover":
        state["clover"] = D.clover_field(V, C_SW)
    elif case["form"] == "compressed":
        state["U"] = D.compress_links(V)
    return state


# --- one pass ---------------------------------------------------------------

def run(state):
    case = state["case"]
    op = case["op"]
    if case["kind"] == "solve":
        x, info = D.solve(op, state["U"], state["b"], SOLVE_MASS[op], inner=case["inner"], tol=SOLVE_TOL,
                          inner_tol=INNER_TOL[case["eo"], case["inner"]], eo=case["eo"])
        return {"x": x}
    if case["kind"] == "step":
        links = D.brillouin_links_autograd(state["V"]) if op == "brillouin" else state["V"]
        out = D.dslash(op, links, state["psi"], MASS[op])
        grad_V, grad_psi = torch.autograd.grad(out, (state["V"], state["psi"]), state["g"])
        return {"out": out, "grad_V": grad_V, "grad_psi": grad_psi}
    if case["form"] == "compressed":
        return D.apply_compressed(op, state["U"], state["psi"], MASS[op], case["adjoint"], out=state["out"])
    return D.apply(op, state["U"], state["psi"], MASS[op], case["adjoint"], out=state["out"], clover=state["clover"])


def work(case):
    """Every stored link and right-hand side read once, every output written once; operator flops only."""
    vol, op, nv = _volume(case), case["op"], case["nv"]
    spinor = (3 if op == "staggered" else 12) * nv
    if case["kind"] == "solve":
        # U, b and x; the flops of forty applications of D^dag D, which a solve of this kind cannot do without
        return {"bytes": (36 + 2 * spinor) * 16 * vol, "flops": 80.0 * HOP_FLOPS[op] * vol * nv}
    word = WORD[case["dtype"]]
    if case["kind"] == "step":
        # V, psi and the upstream gradient read; out, grad_V and grad_psi written; forward and two products back
        return {"bytes": (2 * 36 + 4 * spinor) * word * vol, "flops": 3.0 * HOP_FLOPS[op] * vol * nv}
    links = LINK_WORDS[op] * (2 / 3 if case["form"] == "compressed" else 1) + (36 if case["form"] == "clover" else 0)
    flops = HOP_FLOPS[op] + (576 if case["form"] == "clover" else 0)
    return {"bytes": (links + 2 * spinor) * word * vol, "flops": float(flops) * vol * nv}


# --- the same in 64 bits, with torch alone -----------------------------------

# gamma_mu psi: component s is phase[s] * psi[source[s]] (chiral basis)
_GAMMA = (((3, 2, 1, 0), (-1j, -1j, 1j, 1j)), ((3, 2, 1, 0), (-1, 1, 1, -1)),
          ((2, 3, 0, 1), (-1j, 1j, 1j, -1j)), ((2, 3, 0, 1), (1, 1, 1, 1)))
_RHO = (0, 64 / 432, 16 / 432, 4 / 432, 1 / 432)
_LAMBDA = (-240 / 64, 8 / 64, 4 / 64, 2 / 64, 1 / 64)
_ONE_HOP = [tuple(s if m == mu else 0 for m in range(4)) for mu in range(4) for s in (1, -1)]
_ALL_HOPS = [d for d in itertools.product((-1, 0, 1), repeat=4) if any(d)]


def _shift(f, d):
    """g(x) = f(x + d)."""
    moves = [(-s, 3 - mu) for mu, s in enumerate(d) if s]
    return torch.roll(f, [m[0] for m in moves], [m[1] for m in moves]) if moves else f


def _dagger(u):
    return u.conj().transpose(-1, -2)


def _product(a, b):
    return (a[..., :, :, None] * b[..., None, :, :]).sum(-2)


def _hop_link(V, mu, s):
    d = tuple(s if m == mu else 0 for m in range(4))
    return V[..., mu, :, :] if s > 0 else _dagger(_shift(V[..., mu, :, :], d))


def _off_axis(V):
    """{d: W_d}, the mean over the orderings of the hops, built from the first hop down."""
    W = {}
    for d in sorted(_ALL_HOPS, key=lambda d: sum(map(abs, d))):
        total, k = 0, sum(map(abs, d))
        for mu, s in enumerate(d):
            if s:
                rest = tuple(0 if m == mu else c for m, c in enumerate(d))
                hop = tuple(s if m == mu else 0 for m in range(4))
                first = _hop_link(V, mu, s)
                total = total + (_product(first, _shift(W[rest], hop)) if any(rest) else first)
        W[d] = total / k
    return W


def _gamma(mu, p):
    source, phase = _GAMMA[mu]
    return torch.stack([phase[s] * p[..., source[s], :, :] for s in range(4)], dim=-3)


def _colour(u, p):
    """u acting on the colour index of [..., 3, nv] or [..., 4, 3, nv]."""
    u = u if p.dim() == u.dim() else u.unsqueeze(-3)
    rows = [sum(u[..., a, b, None] * p[..., b, :] for b in range(3)) for a in range(3)]
    return torch.stack(rows, dim=-2)


def _eta(mu, lat):
    t, z, y, x = (torch.arange(n, device="cuda") for n in lat)
    t, z, y, x = t[:, None, None, None], z[:, None, None], y[:, None], x
    s = (x * 0 + y * 0 + z * 0 + t * 0) + (x if mu > 0 else 0) + (y if mu > 1 else 0) + (z if mu > 2 else 0)
    return (1 - 2 * (s % 2)).to(torch.float64)[..., None, None]


def _hop(op, d, u, p, sign):
    """The part of D (sign 1) or D^dag (sign -1) that hops by d: a spin matrix times u(x) p(x + d)."""
    chi = _colour(u, _shift(p, d))
    k = sum(map(abs, d))
    if op == "staggered":
        mu = [m for m in range(4) if d[m]][0]
        return sign * 0.5 * d[mu] * _eta(mu, p.shape[:4]) * chi
    diagonal, slope = (-0.5, 0.5) if op == "wilson" else (-0.5 * _LAMBDA[k], _RHO[k])
    out = diagonal * chi
    for mu, c in enumerate(d):
        if c:
            out = out + sign * slope * c * _gamma(mu, chi)
    return out


def _links(op, V):
    """{d: the link of the hop by d}."""
    if op == "brillouin":
        return _off_axis(V)
    return {d: _hop_link(V, [m for m in range(4) if d[m]][0], sum(d)) for d in _ONE_HOP}


def _diagonal(op, mass):
    return mass + {"staggered": 0.0, "wilson": 4.0, "brillouin": -0.5 * _LAMBDA[0]}[op]


def _operator(op, links, p, mass, sign=1.0):
    out = _diagonal(op, mass) * p
    for d, u in links.items():
        out += _hop(op, d, u, p, sign)
    return out


def _clover_term(V, p, c_sw):
    """-(c_SW / 2) sum_{mu < nu} sigma_{mu nu} F_{mu nu} p."""
    def plaquette(a, b):
        (m, s), (n, r) = a, b
        da = tuple(s if k == m else 0 for k in range(4))
        db = tuple(r if k == n else 0 for k in range(4))
        first = _product(_hop_link(V, m, s), _shift(_hop_link(V, n, r), da))
        second = _product(_hop_link(V, n, r), _shift(_hop_link(V, m, s), db))
        return _product(first, _dagger(second))
    out = torch.zeros_like(p)
    for mu, nu in itertools.combinations(range(4), 2):
        m, n, mm, nn = (mu, 1), (nu, 1), (mu, -1), (nu, -1)
        q = plaquette(m, n) + plaquette(n, mm) + plaquette(mm, nn) + plaquette(nn, m)
        f = (q - _dagger(q)) / 8j
        # sigma_{mu nu} = i gamma_mu gamma_nu for mu != nu
        out += -0.5 * c_sw * 1j * _gamma(mu, _gamma(nu, _colour(f, p)))
    return out


def _solve_exact(op, links, b, mass):
    """D x = b by CG on D^dag D in 64 bits, restarted on the true residual."""
    dims = tuple(range(b.dim() - 1))

    def dot(u, v):
        return (u.conj() * v).sum(dims).real

    x = torch.zeros_like(b)
    for _ in range(3):
        r = _operator(op, links, b - _operator(op, links, x, mass), mass, -1.0)
        if not bool((dot(r, r) > 0).all()):
            break
        p, rr, e = r.clone(), dot(r, r), torch.zeros_like(b)
        stop = 1e-16 * float(rr.max())
        for _ in range(600):
            q = _operator(op, links, _operator(op, links, p, mass), mass, -1.0)
            alpha = rr / dot(p, q)
            e += alpha * p
            r -= alpha * q
            new = dot(r, r)
            if float(new.max()) < stop:
                break
            p = r + (new / rr) * p
            rr = new
        x += e
    return x


def exact(case, seed):
    op = case["op"]
    if case["kind"] == "solve":
        V, b, _ = _fields(case, seed, "c128")
        if _volume(case) * case["nv"] > 1 << 21:
            return None          # over the time that this may take
        return {"x": _solve_exact(op, _links(op, V), b, SOLVE_MASS[op])}
    V, psi, g = _fields(case, seed, case["dtype"])
    V, psi = _wide(V), _wide(psi)
    mass = MASS[op]
    if case["kind"] == "apply":
        if case["form"] == "compressed":     # the third row follows from the stored two
            a, b = V[..., 0, :], V[..., 1, :]
            c = torch.stack([a[..., (j + 1) % 3] * b[..., (j + 2) % 3] - a[..., (j + 2) % 3] * b[..., (j + 1) % 3]
                             for j in range(3)], dim=-1).conj()
            V = torch.stack([a, b, c], dim=-2)
        out = _operator(op, _links(op, V), psi, mass, -1.0 if case["adjoint"] else 1.0)
        if case["form"] == "clover":
            out += _clover_term(V, psi, C_SW)
        return out if case["dtype"] in ("c64", "c128") else torch.view_as_real(out)
    g = _wide(g)
    V.requires_grad_()
    links = _links(op, V)
    out = torch.zeros_like(psi)
    grad_psi = _diagonal(op, mass) * g
    grad_links = []
    for d, u in links.items():               # hop by hop, so that one hop's intermediates are held at a time
        ud, pd = u.detach().requires_grad_(), psi.detach().requires_grad_()
        h = _hop(op, d, ud, pd, 1.0)
        gu, gp = torch.autograd.grad(h, (ud, pd), g)
        out += h.detach()
        grad_psi += gp
        grad_links.append(gu)
    out += _diagonal(op, mass) * psi
    grad_V, = torch.autograd.grad(list(links.values()), V, grad_links)
    return {"out": out, "grad_V": grad_V, "grad_psi": grad_psi}
