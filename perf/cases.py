"""Timed workloads of the framework's public entry points on one GPU.

listed() names the workloads, draw() gives more of the same ranges, prepare() makes what a program
has in hand before the call (a context with its links loaded and its launch configuration chosen,
vectors on the device, a network's weights), run() is one pass through the entry points, work() the
bytes and operations the pass cannot do without, and exact() the same outputs in 64 bits from plain
torch (Eq. 3 written out with index arrays; nothing of the library).

Inputs are random from the seed, made on the GPU: fat links exp(i eps H) + 0.05 G (near SU(3), as
smeared links are), Naik links -U / 24 with U in SU(3), complex Gaussian or Z2 sources.
"""
from __future__ import annotations

import ctypes
import math

import numpy as np
import torch

from paper_1409_1510_amd import hisq

DEV = "cuda:0"
PREC = {"f64": hisq.HISQ_F64, "f32": hisq.HISQ_F32, "f16": hisq.HISQ_F16}
COPY = {"f64": hisq.HISQ_LINKS_F64, "f32": hisq.HISQ_LINKS_F32, "f16": hisq.HISQ_LINKS_F16}
CHANNELS = 8


def listed():
    return [
        # the smallest operator application: one right-hand side on a test lattice, where launches
        # and host work are all there is
        dict(name="m_f64_8x8x8x8_n1", op="m", dims="8x8x8x8", n=1, prec="f64", recon=18, mass=0.1),
        # a lattice whose extents fill no tile, an odd number of right-hand sides, 14-real Naik links
        dict(name="dslash_f32r14_20x10x18x10_n5", op="dslash", dims="20x10x18x10", n=5, prec="f32", recon=14),
        # a single right-hand side on the paper's smaller lattice: bound by the links
        dict(name="dslash_f32_32x32x32x8_n1", op="dslash", dims="32x32x32x8", n=1, prec="f32", recon=18),
        # the benchmark's workload: both half Dslash on 16 right-hand sides
        dict(name="dslash_f32_32x32x32x8_n16", op="dslash", dims="32x32x32x8", n=16, prec="f32", recon=18),
        # the mixed solver's inner operator on the paper's smaller lattice
        dict(name="m_f16_32x32x32x8_n8", op="m", dims="32x32x32x8", n=8, prec="f16", recon=18, mass=0.02),
        # the operator of plain FP64 CG and of the reliable updates
        dict(name="m_f64_32x32x32x8_n8", op="m", dims="32x32x32x8", n=8, prec="f64", recon=18, mass=0.02),
        # the inner operator of the 48^3 x 12 solves with 16 sources
        dict(name="m_f32_48x48x48x12_n16", op="m", dims="48x48x48x12", n=16, prec="f32", recon=18, mass=0.01),
        # the largest lattice and bundle of the solver study: nothing stays in a cache
        dict(name="dslash_f16_64x64x64x16_n32", op="dslash", dims="64x64x64x16", n=32, prec="f16", recon=18),
        # the smallest solve, bound by launches: plain FP64 CG with one source
        dict(name="cg_f64_8x8x8x8_n1", op="cg", dims="8x8x8x8", n=1, kind="f64", link="f32", mass=0.1, tol=1e-10),
        # a production solve: mixed CG with FP16 links on 8 sources to a true residual of 1e-8
        dict(name="cg_mixed_32x32x32x8_n8", op="cg", dims="32x32x32x8", n=8, kind="mixed", link="f16", mass=0.02,
             tol=1e-8),
        # one application of the 4-layer learned preconditioner inside the flexible CG on 16 sources
        dict(name="nn_apply_48x48x48x12_n16", op="nn_apply", dims="48x48x48x12", n=16, layers=4, form="gram",
             bf16=True),
        # one training minibatch of that network: loss and gradient
        dict(name="nn_grad_32x32x32x8_n16", op="nn_grad", dims="32x32x32x8", n=16, layers=4, form="gram", bf16=True,
             loss="residual", mass=0.02),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_dims(rng, vmin, vmax):
    """Even extents >= 4 near a volume drawn over its logarithm; most of them fill no tile."""
    v = _log_uniform(rng, vmin, vmax)
    lt = 2 * rng.randint(2, 8)
    side = (v / lt) ** (1 / 3)
    ext = [max(4, 2 * round(side * rng.uniform(0.8, 1.25) / 2)) for _ in range(3)]
    while ext[0] * ext[1] * ext[2] * lt > 1.25 * vmax and max(ext) > 4:
        ext[ext.index(max(ext))] -= 2
    return "x".join(str(e) for e in ext + [lt]), ext[0] * ext[1] * ext[2] * lt


def draw(rng):
    op = rng.choices(["dslash", "m", "cg", "nn_apply", "nn_grad"], [4, 4, 2, 1, 1])[0]
    if op in ("dslash", "m"):
        dims, v = _draw_dims(rng, 4096, 1.3e6)
        n = min(round(_log_uniform(rng, 1, 32)), max(1, int(2.1e7 / v)))
        prec = rng.choice(["f64", "f32", "f16"])
        recon = 18 if prec == "f64" else rng.choice([18, 18, 14, 13, 9])
        c = dict(op=op, dims=dims, n=n, prec=prec, recon=recon)
        if op == "m":
            c["mass"] = round(_log_uniform(rng, 0.005, 0.2), 4)
        return c
    if op == "cg":
        dims, v = _draw_dims(rng, 4096, 1.5e5)
        kind = rng.choice(["f64", "mixed"])
        return dict(op=op, dims=dims, n=rng.randint(1, 12), kind=kind, link=rng.choice(["f32", "f16"]),
                    mass=round(_log_uniform(rng, 0.05, 0.2), 3), tol=1e-9)
    dims, v = _draw_dims(rng, 4096, 2.6e5)
    n = min(rng.randint(1, 16), max(1, int(4e6 / v)))
    c = dict(op=op, dims=dims, n=n, layers=rng.randint(1, 4), form=rng.choice(["gram", "direct"]),
             bf16=rng.random() < 0.7)
    if op == "nn_grad":
        c.update(loss=rng.choice(["residual", "solution"]), mass=round(_log_uniform(rng, 0.02, 0.2), 3))
    return c


# ---- inputs -----------------------------------------------------------------------------------

def _dims(case):
    return tuple(int(e) for e in case["dims"].split("x"))


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _normal(g, shape):
    """Standard complex normal: Re, Im ~ N(0, 1/2)."""
    return torch.view_as_complex(torch.randn(tuple(shape) + (2,), generator=g, dtype=torch.float64, device=DEV)
                                 * math.sqrt(0.5))


def _mm(a, b):
    return (a.unsqueeze(-1) * b.unsqueeze(-3)).sum(-2)


def _su3(z):
    """Haar SU(3) from complex normal 3x3 matrices: Gram-Schmidt on two rows, the third from det = 1."""
    r0 = z[..., 0, :]
    r0 = r0 / r0.abs().square().sum(-1, keepdim=True).sqrt()
    r1 = z[..., 1, :]
    r1 = r1 - (r0.conj() * r1).sum(-1, keepdim=True) * r0
    r1 = r1 / r1.abs().square().sum(-1, keepdim=True).sqrt()
    r2 = torch.stack([r0[..., 1] * r1[..., 2] - r0[..., 2] * r1[..., 1],
                      r0[..., 2] * r1[..., 0] - r0[..., 0] * r1[..., 2],
                      r0[..., 0] * r1[..., 1] - r0[..., 1] * r1[..., 0]], -1).conj()
    return torch.stack([r0, r1, r2], -2)


def _links(dims, seed, eps=0.4, chunk=1 << 18):
    v = math.prod(dims)
    g = _gen(seed)
    fat = torch.empty((v, 4, 3, 3), dtype=torch.complex128, device=DEV)
    naik = torch.empty_like(fat)
    eye = torch.eye(3, dtype=torch.complex128, device=DEV)
    for lo in range(0, v, chunk):
        m = min(v, lo + chunk) - lo
        a = _normal(g, (m, 4, 3, 3))
        h = 0.5 * (a + a.mH)
        h = 1j * eps * (h - (h.diagonal(dim1=-2, dim2=-1).sum(-1).real / 3)[..., None, None] * eye)
        e, term = eye + h, h
        for k in range(2, 18):
            term = _mm(term, h) / k
            e = e + term
        fat[lo:lo + m] = e + 0.05 * _normal(g, (m, 4, 3, 3))
        naik[lo:lo + m] = _su3(_normal(g, (m, 4, 3, 3))) / -24.0
    return fat, naik


def _source(dims, n, seed, kind="gaussian"):
    shape = (n, 3, math.prod(dims) // 2)
    if kind == "z2":
        return (torch.randint(0, 2, shape, generator=_gen(seed), device=DEV) * 2 - 1).to(torch.complex128)
    return _normal(_gen(seed), shape)


def _inputs(case, seed):
    """Links and the vectors of a case (complex128)."""
    dims, n = _dims(case), case["n"]
    fat, naik = _links(dims, 7919 * seed + 1)
    op = case["op"]
    if op in ("dslash", "m", "nn_apply"):
        vecs = [_source(dims, n, 7919 * seed + 2)]
        if op == "dslash":
            vecs.append(_source(dims, n, 7919 * seed + 3))
        if op != "nn_apply" and case["prec"] == "f64":
            return fat, naik, vecs
        return fat, naik, [v.to(torch.complex64) for v in vecs]
    if op == "cg":
        return fat, naik, [_source(dims, n, 7919 * seed + 2, "z2" if seed % 2 else "gaussian")]
    y = _source(dims, n, 7919 * seed + 2)  # a training pair: r = M y
    hops = _hops(dims)
    return fat, naik, [_apply_m(fat, naik, hops, y, case["mass"]), y]


def _weights(case, seed):
    """Complex64 parameters near the identity network, in the library's order."""
    nc, layers = CHANNELS, case["layers"]
    rng = np.random.default_rng(seed)
    count = nc + layers * 9 * nc + (layers - 1) * nc * nc + nc
    w = 0.05 * math.sqrt(0.5) * (rng.standard_normal(count) + 1j * rng.standard_normal(count))
    k = 0
    w[k] += 1.0
    k += nc
    for l in range(layers):
        if l:
            w[k] += 1.0
            k += nc * nc
        w[k] += 1.0
        k += 9 * nc
    w[k] += 1.0
    return w.astype(np.complex64)


# ---- the passes -------------------------------------------------------------------------------

class State:
    pass


def prepare(case, seed):
    s = State()
    s.case, op, n = case, case["op"], case["n"]
    dims = _dims(case)
    fat, naik, vecs = _inputs(case, seed)
    s.lat = hisq.Lattice(dims, 0)
    if op in ("dslash", "m"):
        copies = COPY[case["prec"]]
    elif op == "cg":
        copies = hisq.HISQ_LINKS_F64 | (COPY["f32"] | COPY[case["link"]] if case["kind"] == "mixed" else 0)
    else:
        copies = hisq.HISQ_LINKS_F32 | hisq.HISQ_LINKS_F16
    s.lat.load_links(fat, naik, copies, case.get("recon", 18))
    del fat, naik
    s.vecs = vecs
    if op in ("dslash", "m"):
        s.outs = [torch.empty_like(v) for v in vecs]
    elif op in ("nn_apply", "nn_grad"):
        lib, ctx = hisq.library(), s.lat.ctx
        w = _weights(case, seed).view(np.float32).astype(np.float64)
        hisq._check(ctx, lib.hisq_nn_init(ctx, case["layers"], CHANNELS, 1))
        hisq._check(ctx, lib.hisq_nn_set_precision(ctx, 1 if case["bf16"] else 0))
        hisq._check(ctx, lib.hisq_nn_set_form(ctx, hisq.HISQ_NN_FORM_GRAM if case["form"] == "gram"
                                              else hisq.HISQ_NN_FORM_DIRECT))
        hisq._check(ctx, lib.hisq_nn_set_params(ctx, w.ctypes.data_as(ctypes.POINTER(ctypes.c_double)), w.size))
        s.nreal = w.size
        if op == "nn_apply":
            s.outs = [torch.empty_like(vecs[0])]
        else:
            hisq._check(ctx, lib.hisq_nn_set_loss(
                ctx, hisq.HISQ_NN_LOSS_RESIDUAL if case["loss"] == "residual" else hisq.HISQ_NN_LOSS_SOLUTION,
                case["mass"]))
    if op != "cg" or math.prod(dims) <= 200000:
        run(s)  # a context outlives its first call, which chooses the launch configuration
        torch.cuda.synchronize()
    return s


def run(s):
    case, lat = s.case, s.lat
    op, n = case["op"], case["n"]
    if op == "dslash":  # D_oe on an even bundle and D_eo on an odd one
        prec = PREC[case["prec"]]
        return [lat.dslash(1, prec, s.vecs[0], s.outs[0]), lat.dslash(0, prec, s.vecs[1], s.outs[1])]
    if op == "m":
        return list(lat.apply_m(PREC[case["prec"]], case["mass"], s.vecs[0], s.outs[0], with_pq=True))
    if op == "cg":
        x, info = lat.cg(case["mass"], s.vecs[0],
                         kind=hisq.HISQ_CG_MIXED if case["kind"] == "mixed" else hisq.HISQ_CG_F64,
                         tol=case["tol"], link_prec=PREC[case["link"]])
        return [x, np.array(info["iters"], np.int64)]
    hisq.hisq_set_stream(lat.ctx)
    lib = hisq.library()
    if op == "nn_apply":
        hisq._check(lat.ctx, lib.hisq_nn_apply(lat.ctx, n, hisq.HISQ_F32, hisq._ptr(s.vecs[0]), hisq._ptr(s.outs[0])))
        return s.outs[0]
    loss, grad = ctypes.c_double(), (ctypes.c_double * s.nreal)()
    hisq._check(lat.ctx, lib.hisq_nn_loss_grad(lat.ctx, n, hisq._ptr(s.vecs[0]), hisq._ptr(s.vecs[1]),
                                               ctypes.byref(loss), grad))
    # the network's arithmetic and master weights are FP32: loss and gradient at that precision
    return [np.array([loss.value], np.float32), np.ctypeslib.as_array(grad).astype(np.float32)]


# ---- what a pass cannot do without ------------------------------------------------------------

def work(case):
    dims, n, op = _dims(case), case["n"], case["op"]
    vh = math.prod(dims) / 2
    cplx = 16 if case.get("prec") == "f64" or (op == "cg" and case["kind"] == "f64") else 8
    link = {"f64": 16, "f32": 8, "f16": 4}

    def half(prec, recon, nvec=2):
        planes = 72 + 8 * recon / 2
        return vh * (planes * link[prec] + nvec * 3 * cplx * n)
    if op == "dslash":
        return {"bytes": 2 * half(case["prec"], case["recon"]), "flops": 2 * vh * n * 1146.0}
    if op == "m":  # the links of both parities, p in and q out (and p, t once more between the halves)
        return {"bytes": half(case["prec"], case["recon"], 2) + half(case["prec"], case["recon"], 2),
                "flops": 2 * vh * n * (1146.0 + 12)}
    if op == "cg":
        iters = -math.log(case["tol"]) / math.log(10) * 9.1 / case["mass"]
        prec = case["link"] if case["kind"] == "mixed" else "f64"
        per = 2 * half(prec, 18) + vh * 3 * cplx * n * 8  # r: 2 reads, 1 write; p, x: 3 reads, 2 writes
        return {"bytes": iters * per, "flops": iters * 2 * vh * n * 1150.0}
    v, layers = 2 * vh, case["layers"]
    act = 2 if case["bf16"] else 4
    passes = 2 if case["form"] == "gram" else 1
    # a site and sample of a layer: 8 hops x 8 channels x (a 3x3 product and a complex scale), the
    # self term and the channel mix
    layer = 8 * CHANNELS * (66 + 24) + CHANNELS * 18 + 3 * 8 * CHANNELS * CHANNELS
    fl = passes * layers * v * n * layer
    io = v * 72 * (4 if case["bf16"] else 8) + n * 3 * v * 8
    if op == "nn_apply":
        return {"bytes": io, "flops": fl}
    # gradient: a forward and an adjoint pass, then forward and backward for each of the passes, the
    # activations of every layer written once and read once
    keep = 2 * layers * v * n * 3 * CHANNELS * 2 * act
    return {"bytes": io + passes * 2 * keep, "flops": 3.0 * fl}


# ---- 64-bit values ----------------------------------------------------------------------------

def _hops(dims):
    """Per parity: lexicographic sites, and the neighbours (lexicographic) at +1, -1, +3, -3 along
    each direction."""
    lx, ly, lz, lt = dims
    lex = torch.arange(math.prod(dims), device=DEV)
    c = [lex % lx, (lex // lx) % ly, (lex // (lx * ly)) % lz, lex // (lx * ly * lz)]
    stride = [1, lx, lx * ly, lx * ly * lz]
    par = (c[0] + c[1] + c[2] + c[3]) % 2
    sites = [torch.nonzero(par == p).flatten() for p in (0, 1)]
    nbr = {}
    for p in (0, 1):
        s = sites[p]
        for mu in range(4):
            cm = c[mu][s]
            for d in (1, -1, 3, -3):
                nbr[p, mu, d] = s + ((cm + d) % dims[mu] - cm) * stride[mu]
    return sites, nbr


def _add_mv(out, u, v, dag, sign):
    """out += sign u v (u^dag v), u [S][3][3], v and out [n][3][S]."""
    for a in range(3):
        for b in range(3):
            e = u[:, b, a].conj() if dag else u[:, a, b]
            out[:, a] += sign * e * v[:, b]


def _half(fat, naik, hops, v, out_parity, step=4):
    """Eq. 3 restricted to one output parity, complex128."""
    sites, nbr = hops
    s = sites[out_parity]
    out = torch.zeros_like(v)
    for lo in range(0, v.shape[0], step):
        o, w = out[lo:lo + step], v[lo:lo + step]
        for mu in range(4):
            for links, d in ((fat, 1), (naik, 3)):
                f, b = nbr[out_parity, mu, d], nbr[out_parity, mu, -d]
                _add_mv(o, links[s, mu], w[:, :, f >> 1], False, 1.0)
                _add_mv(o, links[b, mu], w[:, :, b >> 1], True, -1.0)
    return out


def _apply_m(fat, naik, hops, v, mass):
    return mass * mass * v - _half(fat, naik, hops, _half(fat, naik, hops, v, 1), 0)


def _solve(fat, naik, hops, b, mass):
    """CG in complex128 to the rounding level."""
    x, r = torch.zeros_like(b), b.clone()
    p, rho = r.clone(), (r.abs() ** 2).sum((1, 2))
    stop = 1e-28 * rho
    for it in range(1, 20001):
        q = _apply_m(fat, naik, hops, p, mass)
        alpha = (rho / (p.conj() * q).sum((1, 2)).real)[:, None, None]
        x += alpha * p
        r -= alpha * q
        new = (r.abs() ** 2).sum((1, 2))
        if it % 50 == 0 and bool((new <= stop).all()):
            break
        p = r + (new / rho)[:, None, None] * p
        rho = new
    return x


class _Net:
    """The network on one sample, on the full lattice in lexicographic order ([3][V][C])."""

    def __init__(self, case, fat, hops, w):
        nc = CHANNELS
        self.fat, self.layers, self.v = fat, case["layers"], fat.shape[0]
        sites, nbr = hops
        self.even = sites[0]
        self.nb = {}
        for mu in range(4):
            for d in (1, -1):
                full = torch.empty(self.v, dtype=torch.long, device=DEV)
                for p in (0, 1):
                    full[sites[p]] = nbr[p, mu, d]
                self.nb[mu, d] = full
        k = 0
        self.win = w[k:k + nc]
        k += nc
        self.w, self.a = [], []
        for l in range(self.layers):
            self.w.append(w[k:k + nc * nc].reshape(nc, nc) if l else None)
            k += nc * nc if l else 0
            self.a.append(w[k:k + 9 * nc].reshape(9, nc))
            k += 9 * nc
        self.wout = w[k:k + nc]

    def stencil(self, a, phi, adj):
        out = (a[0].conj() if adj else a[0]) * phi
        for mu in range(4):
            for d in (1, -1):
                nb = self.nb[mu, d]
                g = phi[:, nb]
                rows = []
                for i in range(3):
                    t = 0
                    for j in range(3):
                        e = self.fat[:, mu, i, j] if d == 1 else self.fat[nb, mu, j, i].conj()
                        t = t + e[:, None] * g[j]
                    rows.append(t)
                h = (1 + mu) if d == 1 else (5 + mu)
                if adj:  # the adjoint of the forward hop is the backward hop with the conjugate weight
                    c = a[5 + mu if d == 1 else 1 + mu].conj()
                else:
                    c = a[h]
                out = out + c * torch.stack(rows)
        return out

    def forward(self, r):
        """N r on the full lattice for an even-site r [3][V/2]."""
        full = torch.zeros((3, self.v), dtype=torch.complex128, device=DEV)
        full = full.index_copy(1, self.even, r)
        phi = full[..., None] * self.win
        for l in range(self.layers):
            if l:
                phi = psi @ self.w[l].T
            psi = self.stencil(self.a[l], phi, False)
        return psi @ self.wout

    def adjoint(self, u):
        """N^dag u on the even sites for a full-lattice u [3][V]."""
        g = u[..., None] * self.wout.conj()
        for l in range(self.layers - 1, -1, -1):
            g = self.stencil(self.a[l], g, True)
            if l:
                g = g @ self.w[l].conj()
        return (g @ self.win.conj())[:, self.even]

    def apply(self, r, gram):
        u = self.forward(r)
        return self.adjoint(u) if gram else u[:, self.even]


def exact(case, seed):
    dims, op = _dims(case), case["op"]
    if op == "cg" and math.prod(dims) * case["n"] > 70000:
        return None  # thousands of iterations on a large lattice
    if op == "nn_grad" and math.prod(dims) * case["n"] > 5e6:
        return None
    fat, naik, vecs = _inputs(case, seed)
    hops = _hops(dims)
    vecs = [v.to(torch.complex128) for v in vecs]
    if op == "dslash":
        return [_half(fat, naik, hops, vecs[0], 1), _half(fat, naik, hops, vecs[1], 0)]
    if op == "m":
        q = _apply_m(fat, naik, hops, vecs[0], case["mass"])
        return [q, (vecs[0].conj() * q).sum((1, 2)).real]
    if op == "cg":
        return [_solve(fat, naik, hops, vecs[0], case["mass"]), None]
    w = torch.from_numpy(_weights(case, seed)).to(DEV).to(torch.complex128)
    gram = case["form"] == "gram"
    if op == "nn_apply":
        net = _Net(case, fat, hops, w)
        return torch.stack([net.apply(r, gram) for r in vecs[0]])
    w.requires_grad_(True)
    net = _Net(case, fat, hops, w)
    total = 0.0
    for r, y in zip(*vecs):
        z = net.apply(r, gram)
        if case["loss"] == "residual":
            d = _grad_m(fat, naik, hops, z - y, case["mass"])
            norm = r
        else:
            d, norm = z - y, y
        part = (d.abs() ** 2).sum() / (norm.abs() ** 2).sum() / case["n"]
        part.backward()
        total += float(part.detach())
    return [np.array([total]), torch.view_as_real(w.grad).reshape(-1)]


class _GradM(torch.autograd.Function):
    """M v for one sample; M is Hermitian, so its gradient is M too."""

    @staticmethod
    def forward(ctx, v, f):
        ctx.f = f
        return f(v)

    @staticmethod
    def backward(ctx, g):
        return ctx.f(g), None


def _grad_m(fat, naik, hops, v, mass):
    return _GradM.apply(v, lambda u: _apply_m(fat, naik, hops, u[None], mass)[0])
