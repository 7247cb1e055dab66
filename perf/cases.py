"""Workloads by which the speed of the library is followed.

Every case is work that a user's program has the library do through its Python entry points, on
synthetic fields of the kind the benchmark uses (links exp(i eps H), antiperiodic in t):

* ``wilson``      one application of D or D^dagger (qmg_wilson_apply / _adj), in the canonical
                  layout that the entry points take by default or in the native layout;
* ``schur``       one application of the even-odd Schur complement, Wilson or clover;
* ``krylov``      a solve without a hierarchy: double-precision GMRES on the even-odd operator;
* ``twogrid``     restrict, coarse operator, prolong: a coarse-grid correction without its solve;
* ``propagator``  setup of a hierarchy and the solve of all sources of one gauge field;
* ``grad``        a differentiable solve and its backward (adjoint solve and link force);
* ``batch``       setup and solve of many small lattices at once.

``listed`` names one case for each part of the range, ``draw`` gives others of the same ranges.
Outputs are the entry points' own; ``exact`` gives the same in 64 bits from plain torch.
"""
import math

import numpy as np
import torch

import paper_2505_14399_amd as q
from paper_2505_14399_amd import autograd as qgrad

_BYTES = {"f64": 16, "f32": 8, "bf16": 4, "f16": 4}  # of one complex number


# --------------------------------------------------------------------------------- the cases

def listed():
    return [
        # the smallest call: one D on 4^4 in double precision, canonical layout; latency of a call
        {"name": "wilson_4x4_f64", "kind": "wilson", "lx": 4, "ly": 4, "lz": 4, "lt": 4, "nrhs": 1,
         "prec": "f64", "layout": "canonical", "adj": False, "eps": 0.3, "mass": 0.05, "xi": 1.0},
        # one single-precision D on a mid-size anisotropic lattice: the step of a Krylov solver
        {"name": "wilson_16x32_f32", "kind": "wilson", "lx": 16, "ly": 16, "lz": 16, "lt": 32, "nrhs": 1,
         "prec": "f32", "layout": "native", "adj": False, "eps": 0.6, "mass": 0.05, "xi": 3.5},
        # the same lattice through the default (canonical, double) layout for the twelve
        # spin-colour columns of a propagator: residual checks, contractions
        {"name": "wilson_16x32_canonical", "kind": "wilson", "lx": 16, "ly": 16, "lz": 16, "lt": 32, "nrhs": 12,
         "prec": "f64", "layout": "canonical", "adj": False, "eps": 0.6, "mass": 0.05, "xi": 3.5},
        # twelve right-hand sides at once on the benchmark's lattice
        {"name": "wilson_32x64_f32_12", "kind": "wilson", "lx": 32, "ly": 32, "lz": 32, "lt": 64, "nrhs": 12,
         "prec": "f32", "layout": "native", "adj": False, "eps": 0.6, "mass": 0.05, "xi": 1.0},
        # D^dagger in 16-bit storage on the lattice of the 16-bit workload
        {"name": "wilson_24x64_bf16_adj", "kind": "wilson", "lx": 24, "ly": 24, "lz": 24, "lt": 64, "nrhs": 1,
         "prec": "bf16", "layout": "native", "adj": True, "eps": 0.7, "mass": 0.05, "xi": 1.0},
        # the even-odd operator on a group of four sources: the smoother's operator in a solve
        {"name": "schur_32x64_f32_4", "kind": "schur", "lx": 32, "ly": 32, "lz": 32, "lt": 64, "nrhs": 4,
         "prec": "f32", "clover": False, "dagger": False, "eps": 0.6, "mass": 0.05, "xi": 1.0},
        # a single solve where no hierarchy pays: GMRES in double precision on the even-odd operator
        {"name": "krylov_16x32_f64", "kind": "krylov", "lx": 16, "ly": 16, "lz": 16, "lt": 32, "nrhs": 1,
         "clover": False, "eo": True, "eps": 0.6, "mass": 0.05, "xi": 3.5},
        # coarse-grid correction of one vector on the mid-size lattice ...
        {"name": "twogrid_16x32_f32", "kind": "twogrid", "lx": 16, "ly": 16, "lz": 16, "lt": 32, "block": 4,
         "rank": 24, "nrhs": 1, "prec": "f32", "eps": 0.6, "mass": 0.05, "xi": 3.5},
        # ... and of the twelve columns of a propagator on the benchmark's lattice
        {"name": "twogrid_32x64_f32_12", "kind": "twogrid", "lx": 32, "ly": 32, "lz": 32, "lt": 64, "block": 4,
         "rank": 24, "nrhs": 12, "prec": "f32", "eps": 0.6, "mass": 0.05, "xi": 1.0},
        # the whole job for one gauge field: hierarchy and twelve point sources (the benchmark)
        {"name": "propagator_32x64_f32", "kind": "propagator", "lx": 32, "ly": 32, "lz": 32, "lt": 64, "block": 4,
         "n_test": 48, "batch": 8, "rank": 24, "nrhs": 12, "inner": "f32", "eps": 0.6, "mass": 0.05, "xi": 1.0},
        # solve and its backward on the differentiation workload's lattice, hierarchy in hand
        {"name": "grad_16x32_f32", "kind": "grad", "lx": 16, "ly": 16, "lz": 16, "lt": 32, "block": 4,
         "n_test": 48, "batch": 8, "rank": 24, "nrhs": 1, "inner": "f32", "eps": 0.5, "mass": 0.03, "xi": 1.0},
        # 64 small lattices of uneven size, set up and solved together
        {"name": "batch_64_f32", "kind": "batch", "n": 64, "l0": 8, "l1": 10, "l2": 12, "n_test": 16, "batch": 4,
         "rank": 8, "nrhs": 1, "inner": "f32", "eps": 0.3, "m0": 0.01, "m1": 0.1},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _extents(rng, lo, hi, step, most):
    """Four extents, multiples of `step`, with a volume of at most `most`."""
    while True:
        e = [step * max(1, round(_log_int(rng, lo, hi) / step)) for _ in range(3)]
        e.append(step * max(1, round(_log_int(rng, lo, 2 * hi) / step)))
        if e[0] * e[1] * e[2] * e[3] <= most:
            return e


def draw(rng):
    """One more case of the same ranges."""
    kind = rng.choice(["wilson", "wilson", "schur", "krylov", "twogrid", "propagator", "grad", "batch"])
    c = {"kind": kind}
    big = 32 ** 3 * 64
    if kind in ("wilson", "schur", "krylov"):
        nrhs = rng.choice([1, 1, 2, 3, 4, 5, 8, 12]) if kind != "krylov" else rng.choice([1, 1, 2, 4])
        most = 16 ** 3 * 48 // nrhs if kind == "krylov" else big
        e = _extents(rng, 4, 33, 1 if kind == "wilson" else 2, most)
        if rng.random() < 0.5:  # as often a lattice of the usual extents
            e = [2 * max(2, v // 2) for v in e]
        c.update(lx=e[0], ly=e[1], lz=e[2], lt=e[3], nrhs=nrhs)
        if kind != "krylov":
            c["prec"] = rng.choice(["f32", "f32", "f64", "bf16", "f16"])
        if kind == "wilson":
            c["layout"] = rng.choice(["native", "canonical"]) if c["prec"] in ("f32", "f64") else "native"
            c["adj"] = rng.random() < 0.3
        elif kind == "schur":
            c["clover"] = rng.random() < 0.4
            c["dagger"] = rng.random() < 0.3
        else:
            c["clover"] = rng.random() < 0.4
            c["eo"] = rng.random() < 0.7
    elif kind in ("twogrid", "propagator", "grad"):
        block = rng.choice([4, 4, 2])
        most = {"twogrid": big, "propagator": 24 ** 3 * 48, "grad": 16 ** 3 * 32}[kind]
        if block == 2:
            most = min(most, 12 ** 3 * 24)
        e = _extents(rng, 8, 32, block if block == 4 else 2, most)
        e = [max(2 * block, v) for v in e]
        rank = rng.choice([8, 16, 20, 24]) if block == 4 else rng.choice([8, 12])
        c.update(lx=e[0], ly=e[1], lz=e[2], lt=e[3], block=block, rank=rank)
        if kind == "twogrid":
            c.update(nrhs=rng.choice([1, 2, 3, 4, 8, 12]), prec=rng.choice(["f32", "f32", "f64"]))
        else:
            batch = rng.choice([4, 8])
            c.update(n_test=2 * rank, batch=batch)
            if kind == "propagator":
                c.update(nrhs=rng.choice([1, 3, 4, 12]), inner=rng.choice(["f32", "f32", "f64", "bf16"]))
            else:
                c.update(nrhs=rng.choice([1, 2]), inner=rng.choice(["f32", "f32", "f64"]))
    else:
        ls = sorted(rng.sample([6, 8, 10, 12], 3))
        c.update(n=_log_int(rng, 4, 64), l0=ls[0], l1=ls[1], l2=ls[2], n_test=16, batch=4, rank=8,
                 nrhs=rng.choice([1, 2]), inner=rng.choice(["f32", "f64"]), m0=0.01, m1=0.1)
    c["eps"] = round(rng.uniform(0.2, 0.6), 3)
    if kind != "batch":
        c.update(mass=round(rng.uniform(0.03, 0.1), 4), xi=rng.choice([1.0, 1.0, 3.5]))
    return c


# -------------------------------------------------------------------------------- the inputs

def _dims(c):
    return (c["lx"], c["ly"], c["lz"], c["lt"])


def _volume(dims):
    return dims[0] * dims[1] * dims[2] * dims[3]


def _rng(seed, tag):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + tag)
    return g


def _gaussian(shape, g):
    """Complex Gaussian numbers, real and imaginary part N(0, 1)."""
    return torch.view_as_complex(torch.randn(tuple(shape) + (2,), generator=g, device="cuda", dtype=torch.float64))


def _mul3(a, b):
    """Products of 3 x 3 matrices, element by element."""
    return (a[..., :, :, None] * b[..., None, :, :]).sum(-2)


def _links(V, eps, g):
    """Random SU(3) links exp(i eps H), H Gaussian, Hermitian and traceless: [4, V, 3, 3]."""
    out = torch.empty((4, V, 3, 3), dtype=torch.complex128, device="cuda")
    one = torch.eye(3, dtype=torch.complex128, device="cuda")
    for mu in range(4):
        for s in range(0, V, 1 << 20):
            n = min(V, s + (1 << 20)) - s
            a = _gaussian((n, 3, 3), g)
            h = 0.5 * (a + a.mH)
            h = h - (h.diagonal(dim1=-2, dim2=-1).sum(-1) / 3.0)[:, None, None] * one
            m = h * (1j * eps / 32.0)
            e = one + m / 10.0
            for k in range(9, 0, -1):
                e = one + _mul3(m, e) / k
            for _ in range(5):
                e = _mul3(e, e)
            r0 = e[:, 0] / torch.linalg.vector_norm(e[:, 0], dim=-1, keepdim=True)
            r1 = e[:, 1] - (r0.conj() * e[:, 1]).sum(-1, keepdim=True) * r0
            r1 = r1 / torch.linalg.vector_norm(r1, dim=-1, keepdim=True)
            r2 = torch.stack([r0[:, 1] * r1[:, 2] - r0[:, 2] * r1[:, 1], r0[:, 2] * r1[:, 0] - r0[:, 0] * r1[:, 2],
                              r0[:, 0] * r1[:, 1] - r0[:, 1] * r1[:, 0]], -1).conj()
            out[mu, s:s + n] = torch.stack([r0, r1, r2], 1)
    return out


def _sources(V, nrhs, g):
    """The spin-colour point sources at the origin for a propagator's twelve columns, Gaussian noise else."""
    if nrhs == 12:
        b = torch.zeros((12, V * 12), dtype=torch.complex128, device="cuda")
        b[torch.arange(12), torch.arange(12)] = 1.0
        return b.reshape(12, V, 4, 3)
    return _gaussian((nrhs, V, 4, 3), g)


def _lattice(c):
    return q.Lattice(_dims(c), c["mass"], c["xi"], -1)


def _half(lat, psi, prec):
    return q.eo_pack_spinor(lat, psi, prec)[0]


def _small(c):
    """Extents and masses of the small lattices: the same for every field."""
    r = np.random.default_rng([c["n"], 7])
    ext = r.choice([c["l0"], c["l1"], c["l2"]], size=c["n"])
    return [int(v) for v in ext], [float(v) for v in r.uniform(c["m0"], c["m1"], size=c["n"])]


def _inputs(c, seed):
    """(gauge field, vectors) in double precision and the canonical layout."""
    V = _volume(_dims(c))
    U = _links(V, c["eps"], _rng(seed, 1))
    g = _rng(seed, 2)
    if c["kind"] in ("propagator", "grad", "krylov"):
        b = _sources(V, c["nrhs"], g)
    else:
        b = _gaussian((c["nrhs"], V, 4, 3), g)
    return U, b


def prepare(case, seed):
    c = case
    k = c["kind"]
    if k == "batch":
        ext, masses = _small(c)
        lats = [q.Lattice((L, L, L, L), m, 1.0, -1) for L, m in zip(ext, masses)]
        g, h = _rng(seed, 1), _rng(seed, 2)
        Us = [_links(L ** 4, c["eps"], g) for L in ext]
        bs = [_gaussian((c["nrhs"], L ** 4, 4, 3), h) for L in ext]
        return {"case": c, "lats": lats, "U": Us, "b": bs, "seed": int(seed)}
    lat = _lattice(c)
    U, b = _inputs(c, seed)
    s = {"case": c, "lat": lat, "seed": int(seed)}
    if k == "wilson":
        if c["layout"] == "native":
            s.update(U=q.pack_gauge(lat, U, c["prec"]), psi=q.pack_spinor(lat, b, c["prec"]))
        else:
            t = torch.complex128 if c["prec"] == "f64" else torch.complex64
            s.update(U=U.to(t), psi=b.to(t))
        s["out"] = torch.empty_like(s["psi"])
    elif k == "schur":
        s.update(U=q.eo_pack_gauge(lat, U, c["prec"]), psi=_half(lat, b, c["prec"]), A=None, Ainv=None)
        if c["clover"]:
            s["A"], s["Ainv"] = q.eo_site_term(lat, U, 1.0, prec=c["prec"])
        s["out"] = torch.empty_like(s["psi"])
    elif k == "krylov":
        s.update(U=U, b=b)
    elif k == "twogrid":
        # what the transfers move does not depend on how smooth the vectors are, so the
        # hierarchy is made from unsmoothed ones in one batch: it spans exactly these vectors
        phi = _gaussian((c["rank"], _volume(_dims(c)), 4, 3), _rng(seed, 3))
        s["mg"] = q.mg_setup_stream_chiral_svd(lat, U, (c["block"],) * 4, c["rank"], c["rank"], c["rank"],
                                               n_setup_iter=0, inner=c["prec"], seed=s["seed"], test_vectors=phi)
        s["psi"] = b if c["prec"] == "f64" else b.to(torch.complex64)
    elif k == "propagator":
        s.update(U=U, b=b)
    else:
        s.update(U=U.requires_grad_(True), b=b.requires_grad_(True), mg=_hierarchy(c, lat, U.detach(), s["seed"]))
        s["eta"] = _gaussian(tuple(b.shape), _rng(seed, 4))
    return s


def _hierarchy(c, lat, U, seed):
    mg = q.mg_setup_stream_chiral_svd(lat, U, (c["block"],) * 4, c["n_test"], c["batch"], c["rank"],
                                      inner=c["inner"], seed=seed)
    mg.set_smoother(eo=True, sstep=True)
    return mg


def run(state):
    s, c = state, state["case"]
    k = c["kind"]
    if k == "wilson":
        f = q.wilson_apply_adj if c["adj"] else q.wilson_apply
        return f(s["lat"], s["U"], s["psi"], layout=c["layout"], out=s["out"])
    if k == "schur":
        return q.schur_apply(s["lat"], s["U"], s["psi"], s["A"], s["Ainv"], dagger=c["dagger"], out=s["out"])
    if k == "krylov":
        return q.eo_solve(s["lat"], s["U"], s["b"], 1.0 if c["clover"] else None, tol=1e-12, eo=c["eo"])[0]
    if k == "twogrid":
        r = q.restrict(s["mg"], s["psi"])
        v = q.coarse_apply(s["mg"], r)
        return [r, v, q.prolong(s["mg"], v)]
    if k == "propagator":
        mg = _hierarchy(c, s["lat"], s["U"], s["seed"])
        x, _ = q.mg_solve(mg, s["b"], tol=1e-12)
        mg.close()
        return x
    if k == "grad":
        x = qgrad.solve(s["U"], s["b"], s["mg"])
        gU, gb = torch.autograd.grad(x, (s["U"], s["b"]), s["eta"])
        return [x.detach(), gU, gb]
    bt = q.batch_setup(s["lats"], s["U"], (2, 2, 2, 2), c["n_test"], c["batch"], c["rank"], inner=c["inner"],
                       seed=s["seed"])
    xs, _ = q.batch_solve(bt, s["b"], tol=1e-12)
    bt.close()
    return xs


# ---------------------------------------------------------------------------------- the work

def work(case):
    """Bytes (inputs and outputs once) and operations that one pass cannot do without."""
    c = case
    k = c["kind"]
    if k == "batch":
        V = sum(L ** 4 for L in _small(c)[0])
        n, it = c["nrhs"], 16 * c["n_test"] + 60 * c["nrhs"]
        return {"bytes": V * 16.0 * (36 + 24 * n), "flops": 1368.0 * V * it}
    V = float(_volume(_dims(c)))
    n = c["nrhs"]
    if k == "wilson":
        return {"bytes": V * _BYTES[c["prec"]] * (36 + 24 * n), "flops": 1368.0 * V * n}
    if k == "schur":
        site = 36 if c["clover"] else 0
        return {"bytes": V * _BYTES[c["prec"]] * (36 + site + 12 * n),
                "flops": V * n * (1320.0 + (504 if c["clover"] else 48))}
    if k == "krylov":
        return {"bytes": V * 16.0 * (36 + 24 * n), "flops": 1368.0 * V * n * 60}
    block, rank = c["block"], c["rank"]
    d = V / block ** 4
    cb = _BYTES[c["prec"] if k == "twogrid" else "f64"]
    if k == "twogrid":
        return {"bytes": cb * (12 * rank * V + 24 * V * n + 36 * rank * rank * d + 8 * rank * d * n),
                "flops": 8.0 * n * (2 * 12 * rank * V + 36 * rank * rank * d)}
    solve = 1368.0 * V * n * 60 * (2 if k == "grad" else 1)
    if k == "grad":
        return {"bytes": 16.0 * V * (2 * 36 + 48 * n), "flops": solve}
    setup = V * (1368.0 * 16 * c["n_test"] + 8 * 12 * 3 * rank * c["n_test"] + 8 * 6 * 16 * rank * rank)
    return {"bytes": 16.0 * V * (36 + 24 * n), "flops": setup + solve}


# ------------------------------------------------------------- the same in 64 bits, in torch

def _gamma(mu, v):
    """gamma_mu on [..., 4, 3] in the chiral basis [[0, A], [A^dag, 0]]."""
    u0, u1, d0, d1 = v[..., 0, :], v[..., 1, :], v[..., 2, :], v[..., 3, :]
    if mu == 0:
        r = (-1j * d1, -1j * d0, 1j * u1, 1j * u0)
    elif mu == 1:
        r = (-d1, d0, u1, -u0)
    elif mu == 2:
        r = (-1j * d0, 1j * d1, 1j * u0, -1j * u1)
    else:
        r = (d0, d1, u0, u1)
    return torch.stack(r, -2)


class _Dirac:
    """D in 64 bits on one lattice (U [4, V, 3, 3])."""

    def __init__(self, dims, U, mass, xi):
        self.dims = dims
        lx, ly, lz, lt = dims
        self.U = U.reshape(4, lt, lz, ly, lx, 3, 3)
        self.c = [1.0 / xi] * 3 + [1.0]
        self.diag = mass + 1.0 + 3.0 / xi
        self.sign = torch.ones((lt, 1, 1, 1, 1, 1), dtype=torch.float64, device="cuda")
        self.sign[lt - 1] = -1.0

    def grid(self, v):
        lx, ly, lz, lt = self.dims
        return v.reshape(lt, lz, ly, lx, 4, 3)

    def hop(self, v, dagger=False):
        """Sum over the eight hops of one spinor field on the grid."""
        out = torch.zeros_like(v)
        s = -1.0 if not dagger else 1.0
        for mu in range(4):
            ax = 3 - mu
            U = self.U[mu]
            w = torch.roll(v, -1, ax)
            w = (U[..., None, :, :] * w[..., :, None, :]).sum(-1)
            if mu == 3:
                w = w * self.sign
            out += self.c[mu] * (w + s * _gamma(mu, w))
            w = (U.conj()[..., None, :, :] * v[..., :, :, None]).sum(-2)
            if mu == 3:
                w = w * self.sign
            w = torch.roll(w, 1, ax)
            out += self.c[mu] * (w - s * _gamma(mu, w))
        return -0.5 * out

    def __call__(self, v, dagger=False):
        g = self.grid(v)
        return (self.diag * g + self.hop(g, dagger)).reshape(v.shape)


def _parity(dims):
    lx, ly, lz, lt = dims
    i = torch.arange(_volume(dims), device="cuda")
    x, i = i % lx, i // lx
    y, i = i % ly, i // ly
    return (x + y + i % lz + i // lz) % 2


def _native(v):
    """[n, V, 4, 3] -> [n, 12, V]."""
    n, V = v.shape[:2]
    return v.reshape(n, V, 12).transpose(1, 2).contiguous()


def _solve(D, b, dagger=False):
    """x with D x = b to about 1e-14 by BiCGStab; None if it does not get there."""
    x = torch.zeros_like(b)
    bn = float(torch.linalg.vector_norm(b))
    for _ in range(4):
        r = b - D(x, dagger)
        if float(torch.linalg.vector_norm(r)) <= 2e-14 * bn:
            return x
        r0, p = r.clone(), r.clone()
        rho = torch.vdot(r0.flatten(), r.flatten())
        for _ in range(600):
            Ap = D(p, dagger)
            alpha = rho / torch.vdot(r0.flatten(), Ap.flatten())
            s = r - alpha * Ap
            As = D(s, dagger)
            omega = torch.vdot(As.flatten(), s.flatten()) / torch.vdot(As.flatten(), As.flatten())
            x = x + alpha * p + omega * s
            r = s - omega * As
            if float(torch.linalg.vector_norm(r)) <= 5e-15 * bn:
                break
            new = torch.vdot(r0.flatten(), r.flatten())
            p = r + (new / rho) * (alpha / omega) * (p - omega * Ap)
            rho = new
    r = b - D(x, dagger)
    return x if float(torch.linalg.vector_norm(r)) <= 1e-13 * bn else None


def _blocks(v, dims, block):
    """[n, V, 4, 3] -> [d, 2, rows, n]: aggregates, chirality, (site, spin, colour)."""
    lx, ly, lz, lt = dims
    n, b = v.shape[0], block
    w = v.reshape(n, lt // b, b, lz // b, b, ly // b, b, lx // b, b, 2, 6)
    w = w.permute(1, 3, 5, 7, 9, 2, 4, 6, 8, 10, 0)
    return w.reshape(_volume(dims) // b ** 4, 2, 6 * b ** 4, n).contiguous()


def _unblocks(w, dims, block):
    lx, ly, lz, lt = dims
    n, b = w.shape[-1], block
    v = w.reshape(lt // b, lz // b, ly // b, lx // b, 2, b, b, b, b, 6, n)
    v = v.permute(10, 0, 5, 1, 6, 2, 7, 3, 8, 4, 9)
    return v.reshape(n, _volume(dims), 4, 3).contiguous()


def exact(case, seed):
    c = case
    k = c["kind"]
    if k == "batch":
        if sum(L ** 4 for L in _small(c)[0]) * c["nrhs"] > 800000:
            return None
        ext, masses = _small(c)
        g, h = _rng(seed, 1), _rng(seed, 2)
        Us = [_links(L ** 4, c["eps"], g) for L in ext]
        out = []
        for L, m, U in zip(ext, masses, Us):
            D = _Dirac((L, L, L, L), U, m, 1.0)
            b = _gaussian((c["nrhs"], L ** 4, 4, 3), h)
            xs = [_solve(D, b[i]) for i in range(c["nrhs"])]
            out.append(None if any(x is None for x in xs) else torch.stack(xs))
        return out
    dims = _dims(c)
    V = _volume(dims)
    if k in ("propagator", "grad", "krylov") and V * c["nrhs"] > 1_600_000:
        return None
    if k in ("schur", "krylov") and c["clover"]:
        return None
    U, b = _inputs(c, seed)
    D = _Dirac(dims, U, c["mass"], c["xi"])
    if k == "wilson":
        t = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[c["prec"]]
        D.U = torch.view_as_complex(torch.view_as_real(D.U).to(t).double())
        b = torch.view_as_complex(torch.view_as_real(b).to(t).double())
        out = torch.stack([D(v, c["adj"]) for v in b])
        if c["layout"] == "native":
            out = _native(out)
            if t in (torch.bfloat16, torch.float16):
                out = torch.view_as_real(out)
        return out
    if k == "schur":
        t = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[c["prec"]]
        D.U = torch.view_as_complex(torch.view_as_real(D.U).to(t).double())
        par = _parity(dims)
        even, odd = (par == 0), (par == 1)
        out = []
        for v in b:
            v = torch.view_as_complex(torch.view_as_real(v).to(t).double())
            ve = v[even]
            f = torch.zeros_like(v)
            f[even] = ve
            wo = D.hop(D.grid(f), c["dagger"]).reshape(V, 4, 3)[odd]
            f = torch.zeros_like(v)
            f[odd] = wo / D.diag
            he = D.hop(D.grid(f), c["dagger"]).reshape(V, 4, 3)[even]
            out.append(D.diag * ve - he)
        out = _native(torch.stack(out))
        return torch.view_as_real(out) if t in (torch.bfloat16, torch.float16) else out
    if k == "twogrid":
        phi = _gaussian((c["rank"], V, 4, 3), _rng(seed, 3))
        W = _blocks(phi, dims, c["block"])
        del phi
        Wd = W.conj().transpose(-1, -2).contiguous()
        G = torch.matmul(Wd, W)
        Gi = torch.from_numpy(np.linalg.inv(G.cpu().numpy())).cuda()

        def onto(v):
            return _unblocks(torch.matmul(W, torch.matmul(Gi, torch.matmul(Wd, _blocks(v, dims, c["block"])))),
                             dims, c["block"])

        if c["prec"] == "f32":
            b = b.to(torch.complex64).to(torch.complex128)
        v = onto(b)
        v = torch.stack([D(w) for w in v])
        return [None, None, onto(v)]
    xs = [_solve(D, v) for v in b]
    if any(x is None for x in xs):
        return None
    x = torch.stack(xs)
    if k in ("propagator", "krylov"):
        return x
    eta = _gaussian(tuple(b.shape), _rng(seed, 4))
    ls = [_solve(D, v, True) for v in eta]
    if any(v is None for v in ls):
        return [x, None, None]
    gU = torch.zeros_like(D.U)
    for xv, lv in zip(xs, ls):
        xg, lg = D.grid(xv), D.grid(lv)
        for mu in range(4):
            ax = 3 - mu
            xp, lp = torch.roll(xg, -1, ax), torch.roll(lg, -1, ax)
            a, e = xp - _gamma(mu, xp), lp + _gamma(mu, lp)
            G = (a[..., :, :, None] * lg.conj()[..., :, None, :]).sum(-3)
            G = G + (e[..., :, :, None] * xg.conj()[..., :, None, :]).sum(-3)
            w = 0.5 * D.c[mu] * G.mH
            gU[mu] += w * D.sign if mu == 3 else w
    return [x, gU.reshape(4, V, 3, 3), torch.stack(ls)]
