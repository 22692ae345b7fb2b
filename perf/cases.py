"""The work that users of this framework have it do, as cases that can be timed and checked.

listed() names the cases, draw(rng) makes one more of the same ranges, prepare(case, seed) builds what a program
holds before the call, run(state) is one pass through the public entry points, work(case) counts what a pass cannot
do without, and exact(case, seed) gives the same outputs in 64 bits from plain torch, without the library.

Fields are synthetic, with the structure of the benchmark's: one-link matrices 0.6 U + 0.1 Z and three-link matrices
U with U Haar SU(3) and Z complex Gaussian, staggered phases and the antiperiodic time boundary folded in, and
complex Gaussian sources.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1411_2087_amd as hq
from paper_1411_2087_amd import train

PREC = {"f64": hq.HISQ_F64, "f32": hq.HISQ_F32, "f16s": hq.HISQ_F16S, "i16s": hq.HISQ_I16S, "f64c": hq.HISQ_F64C,
        "f32c": hq.HISQ_F32C, "i16sc": hq.HISQ_I16SC}
# solver form -> (mode, outer links, inner links)
FORMS = {"f64": (hq.HISQ_CG_PLAIN_F64, "f64", None), "f64c": (hq.HISQ_CG_PLAIN_F64C, "f64c", None),
         "f32": (hq.HISQ_CG_MIXED_F32, "f64", "f32"), "f16s": (hq.HISQ_CG_MIXED_F16S, "f64", "f16s"),
         "i16s": (hq.HISQ_CG_MIXED_I16S, "f64", "i16s"), "f32c": (hq.HISQ_CG_MIXED_F32C, "f64c", "f32c"),
         "i16sc": (hq.HISQ_CG_MIXED_I16SC, "f64c", "i16sc")}
# fat7 weights with a Lepage term
FAT7 = (1 / 8, 1 / 16, 1 / 64, 1 / 384, -1 / 16)
LINK_BYTES = {"f64": 2304, "f32": 1152, "f16s": 640, "i16s": 640, "f64c": 1920, "f32c": 960, "i16sc": 544}


def listed():
    """
    dslash-small      one operator application on the smallest workload lattice: launch and latency
    dslash-paper      the paper's 32x40x24x96 lattice in its single precision
    cg-small          the small workload's solve, plain FP64
    cg-mid            a solve whose links fit the last-level cache
    cg-large          the 32^4 workload in its fastest form (16-bit two-row links, FP64 updates)
    multi-rhs         eight masses solved as one batch, FP32 inner links
    mdslash           the batched operator at 16 right-hand sides (a batch of training pairs)
    net-forward       the network applied to a batch (evaluation of a preconditioner)
    train-step        one Adam step of the residual objective at the training shape
    fcg               a solve preconditioned by the network's built polynomial
    fat-paths         path-summed one-link matrices of a new gauge field
    links-pack        its three-link matrices, phases and the packing of both link forms of a mixed solve
    """
    return [
        dict(name="dslash-small", kind="dslash", lx=8, ly=8, lz=8, lt=8, prec="f64", parity=1),
        dict(name="dslash-paper", kind="dslash", lx=32, ly=40, lz=24, lt=96, prec="f32", parity=0),
        dict(name="cg-small", kind="cg", lx=8, ly=8, lz=8, lt=8, form="f64", mass=0.05, tol=1e-10),
        dict(name="cg-mid", kind="cg", lx=16, ly=16, lz=16, lt=16, form="f64", mass=0.02, tol=1e-10),
        dict(name="cg-large", kind="cg", lx=32, ly=32, lz=32, lt=32, form="i16sc", mass=0.01, tol=1e-10),
        dict(name="multi-rhs", kind="multi", lx=24, ly=24, lz=24, lt=24, form="f32", nrhs=8, shift=False, lo=0.02,
             hi=0.2, tol=1e-10),
        dict(name="mdslash", kind="mdslash", lx=32, ly=32, lz=32, lt=32, nrhs=16, parity=1),
        dict(name="net-forward", kind="forward", lx=16, ly=16, lz=16, lt=16, channels=16, batch=16),
        dict(name="train-step", kind="train", lx=16, ly=16, lz=16, lt=16, channels=16, batch=16, mass=0.05),
        dict(name="fcg", kind="fcg", lx=16, ly=16, lz=16, lt=16, channels=4, mass=0.02, tol=1e-10),
        dict(name="fat-paths", kind="fat", lx=32, ly=32, lz=32, lt=32, lepage=True),
        dict(name="links-pack", kind="pack", lx=32, ly=32, lz=32, lt=32, form="i16sc"),
    ]


def _extents(rng, lo, hi):
    """Four even extents whose product is spread over [lo, hi] in its logarithm; rows of x may be short and ragged."""
    while True:
        side = math.exp(rng.uniform(math.log(lo), math.log(hi))) ** 0.25
        d = [max(4, 2 * round(side * math.exp(rng.uniform(-0.35, 0.35)) / 2)) for _ in range(4)]
        if lo <= d[0] * d[1] * d[2] * d[3] <= hi:
            return dict(lx=d[0], ly=d[1], lz=d[2], lt=d[3])


def draw(rng):
    kind = rng.choice(["dslash", "dslash", "apply", "cg", "cg", "multi", "mdslash", "forward", "train", "fcg", "fat",
                       "pack"])
    if kind == "dslash":
        return dict(kind=kind, **_extents(rng, 4 ** 4, 1500000), prec=rng.choice(sorted(PREC)), parity=rng.randrange(2))
    if kind == "apply":
        return dict(kind=kind, **_extents(rng, 4 ** 4, 1048576), prec=rng.choice(sorted(PREC)),
                    mass=rng.uniform(0.005, 0.2))
    if kind == "cg":
        return dict(kind=kind, **_extents(rng, 4 ** 4, 400000), form=rng.choice(["f64", "f64c", "f32", "i16s", "f32c",
                                                                                 "i16sc"]),
                    mass=rng.uniform(0.03, 0.2), tol=1e-10)
    if kind == "multi":
        return dict(kind=kind, **_extents(rng, 1000, 70000), form=rng.choice(["f32", "f32c", "i16s", "i16sc"]),
                    nrhs=rng.randrange(2, 17), shift=rng.random() < 0.4, lo=rng.uniform(0.04, 0.08), hi=0.2, tol=1e-10)
    if kind == "mdslash":
        return dict(kind=kind, **_extents(rng, 4 ** 4, 1048576), nrhs=rng.choice([1, 2, 4, 8, 16]),
                    parity=rng.randrange(2))
    if kind in ("forward", "train"):
        c = dict(kind=kind, **_extents(rng, 4 ** 4, 65536), channels=rng.choice([4, 8, 16]), batch=rng.randrange(1, 17))
        if kind == "train":
            c["mass"] = rng.uniform(0.02, 0.2)
        return c
    if kind == "fcg":
        return dict(kind=kind, **_extents(rng, 1000, 65536), channels=rng.choice([4, 8]), mass=rng.uniform(0.05, 0.1),
                    tol=1e-10)
    if kind == "fat":
        return dict(kind=kind, **_extents(rng, 4 ** 4, 1048576), lepage=rng.random() < 0.5)
    return dict(kind=kind, **_extents(rng, 4 ** 4, 1048576), form=rng.choice(["f64", "f32", "i16s", "f32c", "i16sc"]))


# ------------------------------------------------------------------ synthetic fields
def _dims(case):
    return case["lx"], case["ly"], case["lz"], case["lt"]


def _sites(case):
    return case["lx"] * case["ly"] * case["lz"] * case["lt"]


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(1000003 * int(seed) + 17)


def _gauss(g, *shape):
    """Complex Gaussian of unit mean square modulus."""
    return torch.view_as_complex(torch.randn(*shape, 2, dtype=torch.float64, device="cuda", generator=g)) * 0.5 ** 0.5


def _su3(g, n):
    """n Haar-random SU(3) matrices: two orthonormalised Gaussian rows and the conjugate of their cross product."""
    a, b = _gauss(g, n, 3), _gauss(g, n, 3)
    a = a / torch.linalg.vector_norm(a, dim=1, keepdim=True)
    for _ in range(2):
        b = b - (a.conj() * b).sum(1, keepdim=True) * a
    b = b / torch.linalg.vector_norm(b, dim=1, keepdim=True)
    c = torch.linalg.cross(a, b, dim=1).conj()
    return torch.stack((a, b, c.resolve_conj()), 1)


def _thin(case, seed):
    """Thin links [mu][t][z][y][x][3][3]."""
    lx, ly, lz, lt = _dims(case)
    return _su3(_gen(seed), 4 * _sites(case)).reshape(4, lt, lz, ly, lx, 3, 3).contiguous()


def _phases(case):
    """Staggered phases [mu][t][z][y][x]: 1, (-1)^x, (-1)^(x+y), (-1)^(x+y+z)."""
    lx, ly, lz, lt = _dims(case)
    x = torch.arange(lx, device="cuda").reshape(1, 1, 1, lx)
    y = torch.arange(ly, device="cuda").reshape(1, 1, ly, 1)
    z = torch.arange(lz, device="cuda").reshape(1, lz, 1, 1)
    e = [torch.zeros((), dtype=torch.long, device="cuda"), x, x + y, x + y + z]
    return torch.stack([(1.0 - 2.0 * (v % 2)).to(torch.float64).expand(lt, lz, ly, lx) for v in e])


def _fold(case, links, hop):
    """Phases and the antiperiodic time boundary into [mu][t][z][y][x][3][3] links, in place."""
    ph = _phases(case).clone()
    ph[3, case["lt"] - hop:] *= -1
    links *= ph[..., None, None]
    return links


def _links(case, seed, naive=False):
    """Folded one- and three-link fields (three-link matrices zero for the naive operator)."""
    lx, ly, lz, lt = _dims(case)
    g, n = _gen(seed), 4 * _sites(case)
    fat = (0.6 * _su3(g, n) + 0.1 * _gauss(g, n, 3, 3)).reshape(4, lt, lz, ly, lx, 3, 3)
    lng = torch.zeros_like(fat) if naive else _su3(g, n).reshape(4, lt, lz, ly, lx, 3, 3)
    return _fold(case, fat, 1).contiguous(), _fold(case, lng, 3).contiguous()


def _source(case, seed, n=None):
    shape = (_sites(case) // 2, 3) if n is None else (n, _sites(case) // 2, 3)
    return _gauss(_gen(seed + 500009), *shape)


def _masses(case):
    n = case["nrhs"]
    return [case["lo"] * (case["hi"] / case["lo"]) ** (i / max(1, n - 1)) for i in range(n)]


def _weights(case, seed):
    """The network's weights near the identity it starts training from, with noise."""
    r = np.random.RandomState(seed % (1 << 31))
    w = train.flatten(train.identity_weights(case["channels"], 0.05))
    z = (r.standard_normal(w.size) + 1j * r.standard_normal(w.size)) * 0.5 ** 0.5
    return (w + 0.05 * z).astype(np.complex64)


def _fcg_weights(case):
    """The built polynomial of the naive operator (its largest eigenvalue with these fields is below 11.8)."""
    return train.chebyshev_weights(case["channels"], case["mass"], 11.8)[0].astype(np.complex64)


# ------------------------------------------------------------------ what a program holds, and one pass
def prepare(case, seed):
    kind, dims = case["kind"], _dims(case)
    s = {"case": case, "dims": dims}
    if kind in ("dslash", "apply"):
        prec = PREC[case["prec"]]
        s["links"] = hq.fields.Links.pack(*_links(case, seed), dims, prec)
        s["src"] = _source(case, seed).to(hq.fields.VEC_DTYPE[prec])
        s["dst"], s["tmp"] = torch.empty_like(s["src"]), torch.empty_like(s["src"])
    elif kind in ("cg", "multi"):
        mode, outer, inner = FORMS[case["form"]]
        links = _links(case, seed)
        s["hi"] = hq.fields.Links.pack(*links, dims, PREC[outer])
        s["lo"] = hq.fields.Links.pack(*links, dims, PREC[inner]) if inner else None
        s["opts"] = hq.CGOpts(mode=mode, max_iter=0, check_every=0, use_graph=1, delta=0.0)
        if kind == "cg":
            s["b"] = _source(case, seed)
            s["x"] = torch.empty_like(s["b"])
            s["ws"] = hq.fields.workspace("cg", dims, 1, mode)
        else:
            n = case["nrhs"]
            s["mode"] = hq.HISQ_MULTI_SHIFT if case["shift"] else hq.HISQ_MULTI_RHS
            s["b"] = _source(case, seed, None if case["shift"] else n)
            s["x"] = torch.empty((n, _sites(case) // 2, 3), dtype=torch.complex128, device="cuda")
            s["ws"] = hq.fields.workspace("cg_multi", dims, n, s["mode"])
    elif kind == "mdslash":
        s["links"] = hq.fields.Links.pack(*_links(case, seed), dims, hq.HISQ_F32)
        s["src"] = _gauss(_gen(seed + 500009), _sites(case) // 2, case["nrhs"], 3).to(torch.complex64)
        s["dst"] = torch.empty_like(s["src"])
        s["ws"] = torch.empty(4096, dtype=torch.uint8, device="cuda")
    elif kind in ("forward", "train"):
        c, n = case["channels"], case["batch"]
        s["links"] = hq.fields.Links.pack(*_links(case, seed), dims, hq.HISQ_F32)
        s["b"] = _source(case, seed, n).to(torch.complex64)
        if kind == "train":
            s["trainer"] = train.Trainer(dims, c, s["links"].fat, _weights(case, seed), batch=n, objective="residual",
                                         links32=s["links"], mass=case["mass"])
        else:
            s["w"] = torch.from_numpy(_weights(case, seed)).cuda()
            s["y"] = torch.empty_like(s["b"])
            s["acts"] = torch.empty(hq.net_act_bytes(dims, c, n), dtype=torch.uint8, device="cuda")
    elif kind == "fcg":
        links = _links(case, seed, naive=True)
        s["hi"] = hq.fields.Links.pack(*links, dims, hq.HISQ_F64)
        s["lo"] = hq.fields.Links.pack(*links, dims, hq.HISQ_F32)
        s["b"] = _source(case, seed)
        s["x"] = torch.empty_like(s["b"])
        s["w"] = torch.from_numpy(_fcg_weights(case)).cuda()
        s["ws"] = hq.fields.workspace("fcg", dims, 1, 0, case["channels"])
    else:
        s["thin"] = _thin(case, seed)
        if kind == "fat":
            s["fat"] = torch.empty_like(s["thin"])
            s["coeff"] = FAT7 if case["lepage"] else FAT7[:4] + (0.0,)
            s["ws"] = hq.fields.workspace("fat_paths", dims)
        else:
            s["fat"], s["lng"] = _links(case, seed)[0], torch.empty_like(s["thin"])
            _, outer, inner = FORMS[case["form"]]
            s["packed"] = [(PREC[p], *(torch.zeros(hq.hisq_packed_link_bytes(dims, PREC[p]), dtype=torch.uint8,
                                                   device="cuda") for _ in range(2))) for p in (outer, inner) if p]
    return s


def run(s):
    case, dims = s["case"], s["dims"]
    kind = case["kind"]
    if kind == "dslash":
        hq.dslash_apply(s["links"].fat, s["links"].lng, s["src"], s["dst"], case["parity"], dims, s["links"].prec)
        return s["dst"]
    if kind == "apply":
        hq.hisq_apply_A(case["mass"], s["links"].fat, s["links"].lng, s["src"], s["dst"], s["tmp"], dims,
                        s["links"].prec)
        return s["dst"]
    if kind == "cg":
        s["x"].zero_()
        lo = s["lo"]
        hq.cg_solve(case["mass"], case["tol"], s["hi"].fat, s["hi"].lng, lo.fat if lo else None, lo.lng if lo else None,
                    s["b"], s["x"], dims, s["opts"], s["ws"], raise_on_noconv=True)
        return s["x"]
    if kind == "multi":
        hq.cg_solve_multi(case["nrhs"], _masses(case), case["tol"], s["mode"], s["hi"].fat, s["hi"].lng, s["lo"].fat,
                          s["lo"].lng, s["b"], s["x"], dims, s["opts"], s["ws"], raise_on_noconv=True)
        return s["x"]
    if kind == "mdslash":
        hq.hisq_dslash_multi(s["links"].fat, s["links"].lng, s["src"], s["dst"], case["parity"], case["nrhs"], dims,
                             s["ws"])
        return s["dst"]
    if kind == "forward":
        hq.net_forward(s["links"].fat, s["w"], case["channels"], s["b"], s["y"], s["acts"], case["batch"], dims)
        return s["y"]
    if kind == "train":
        t = s["trainer"]
        t.step(s["b"], None, 1e-4)
        return {"y": t.y, "grad": t.gw, "weights": t.w}
    if kind == "fcg":
        s["x"].zero_()
        hq.fcg_solve(case["mass"], case["tol"], s["hi"].fat, s["hi"].lng, s["lo"].fat, s["w"], case["channels"], s["b"],
                     s["x"], dims, None, s["ws"], raise_on_noconv=True)
        return s["x"]
    if kind == "fat":
        hq.hisq_fat_paths(s["thin"], s["coeff"], s["fat"], dims, s["ws"])
        return s["fat"]
    hq.hisq_three_link(s["thin"], s["lng"], dims)
    hq.hisq_fold_links(s["lng"], dims, 3)
    out = {"long": s["lng"]}
    for prec, fat, lng in s["packed"]:
        hq.hisq_pack_links(s["fat"], s["lng"], dims, prec, fat, lng)
        if prec == hq.HISQ_F64:  # whole doubles; the others pack integers and scales
            fat, lng = fat.view(torch.float64), lng.view(torch.float64)
        out[f"fat{prec}"], out[f"long{prec}"] = fat, lng
    return out


# ------------------------------------------------------------------ what a pass cannot do without
def _iterations(mass, tol):
    """CG iterations of these fields: 38 / mass at 1e-10 (741 at 0.05, 3804 at 0.01), in proportion to log(tol)."""
    return 38.0 / mass * math.log(2.0 / tol) / math.log(2e10)


def work(case):
    kind, vh = case["kind"], _sites(case) / 2
    if kind in ("dslash", "apply"):
        v = 48 if case["prec"] in ("f64", "f64c") else 24
        n = 1 if kind == "dslash" else 2
        return {"bytes": vh * n * (LINK_BYTES[case["prec"]] + 2 * v), "flops": vh * n * 1146}
    if kind == "cg":
        inner = FORMS[case["form"]][2] or FORMS[case["form"]][1]
        v = 48 if inner in ("f64", "f64c") else 24
        it = _iterations(case["mass"], case["tol"])
        return {"bytes": vh * it * (2 * LINK_BYTES[inner] + 10 * v), "flops": vh * it * (2 * 1146 + 60)}
    if kind == "multi":
        its = [_iterations(m, case["tol"]) for m in _masses(case)]
        return {"bytes": vh * (max(its) * 2 * LINK_BYTES[FORMS[case["form"]][2]] + sum(its) * 10 * 24),
                "flops": vh * sum(its) * (2 * 1146 + 60)}
    if kind == "mdslash":
        return {"bytes": vh * (1152 + 48 * case["nrhs"]), "flops": vh * 1146 * case["nrhs"]}
    if kind in ("forward", "train", "fcg"):
        c, b, v = case["channels"], case.get("batch", 1), 2 * vh
        # per site: links once per layer, features once each way; per channel and transport 66 flops, 24 per mix
        layer = {"bytes": v * (4 * 288 + b * 24 * (2 + 6 * c)), "flops": v * b * (8 * 66 * (2 + 2 * c) + 9 * 24 * (2 * c + 2 * c * c))}
        if kind == "forward":
            return layer
        if kind == "train":
            a = {"bytes": 4 * vh * b * (48 + 48) + 4 * vh * 1152, "flops": 4 * vh * b * 1146}
            return {"bytes": 2.5 * layer["bytes"] + a["bytes"], "flops": 2.5 * layer["flops"] + a["flops"]}
        it = 0.38 * 20.0 / case["mass"]
        return {"bytes": it * (layer["bytes"] + vh * (2 * 2304 + 10 * 48)), "flops": it * (layer["flops"] + vh * 2400)}
    if kind == "fat":
        # the nested 3-staples of the path families, shared between them: 12 (both signs, 2 products each) per link
        return {"bytes": 2 * vh * 4 * 2 * 144, "flops": 2 * vh * 4 * (12 * 4 * 198 + 12 * 2 * 36)}
    out = sum(LINK_BYTES[p] for p in FORMS[case["form"]][1:] if p)
    return {"bytes": 2 * vh * (4 * 144 * 3 + out), "flops": 2 * vh * 4 * 2 * 198}


# ------------------------------------------------------------------ the same outputs in 64 bits
DIM = (3, 2, 1, 0)  # torch dimension of x, y, z, t in [t][z][y][x]


def _shift(f, mu, k):
    """f(n + k mu) of a field [t][z][y][x]..."""
    return torch.roll(f, -k, DIM[mu])


def _parity(case):
    lx, ly, lz, lt = _dims(case)
    ax = [torch.arange(n, device="cuda") for n in (lt, lz, ly, lx)]
    return (ax[0][:, None, None, None] + ax[1][:, None, None] + ax[2][:, None] + ax[3]) % 2


class _Operator:
    """D between the parities as gathers: for each direction the matrices at the sites and the neighbours' numbers."""

    def __init__(self, case, fat, lng, hops=((0, 1), (1, 3))):
        par = _parity(case)
        lx, ly, lz, lt = _dims(case)
        h = (torch.arange(_sites(case), device="cuda") // 2).reshape(lt, lz, ly, lx)
        self.m, self.idx = {}, {}
        for p in (0, 1):
            at, ms, ids = par == p, [], []
            for which, k in hops:
                u = (fat, lng)[which]
                for mu in range(4):
                    ms.append(u[mu][at])
                    ids.append(_shift(h, mu, k)[at])
                    ms.append(-_shift(u[mu], mu, -k)[at].conj().transpose(-1, -2))
                    ids.append(_shift(h, mu, -k)[at])
            self.m[p], self.idx[p] = torch.stack(ms, 1).contiguous(), torch.stack(ids, 1).contiguous()

    def d(self, v, p):
        """D v on the sites of parity p."""
        return (self.m[p] * v[self.idx[p]][:, :, None, :]).sum((1, 3))

    def a(self, mass, v):
        return 4 * mass * mass * v - self.d(self.d(v, 1), 0)


def _solve(op, mass, b, tol=1e-14, most=40000):
    x, r = torch.zeros_like(b), b.clone()
    p, rr = r.clone(), torch.linalg.vector_norm(b) ** 2
    stop = float(rr) * tol * tol
    for i in range(most):
        ap = op.a(mass, p)
        al = rr / (p.conj() * ap).sum().real
        x += al * p
        r -= al * ap
        new = (r.conj() * r).sum().real
        if i % 50 == 49 and float(new) <= stop:
            break
        p = r + (new / rr) * p
        rr = new
    return x


def _transports(case, fat):
    """The nine transports T_k of full-lattice fields [n][t][z][y][x][3]."""
    dn = [_shift(fat[mu], mu, -1).conj().transpose(-1, -2).contiguous() for mu in range(4)]

    def t(k, f):
        if k == 0:
            return f
        mu, m, hop = (k - 1, fat[k - 1], 1) if k < 5 else (k - 5, dn[k - 5], -1)
        return (m * torch.roll(f, -hop, DIM[mu] + 1)[..., None, :]).sum(-1)

    return t


def _layers(case, w):
    c, out, o = case["channels"], [], 0
    for co, ci in ((c, 1), (c, c), (c, c), (1, c)):
        out.append(w[o:o + 9 * co * ci].reshape(9, co, ci))
        o += 9 * co * ci
    return out


def _network(t, ws, f):
    """One sample [1][t][z][y][x][3] through the four layers."""
    for w in ws:
        g = 0
        for k in range(9):
            tf = t(k, f)
            g = g + (w[k] @ tf.reshape(tf.shape[0], -1)).reshape(w.shape[1], *tf.shape[1:])
        f = g
    return f


def _full(case, v):
    lx, ly, lz, lt = _dims(case)
    f = torch.zeros((lt, lz, ly, lx, 3), dtype=torch.complex128, device="cuda")
    f[_parity(case) == 0] = v
    return f[None]


def _exact_train(case, seed, fat, lng):
    w = torch.from_numpy(_weights(case, seed)).cuda().to(torch.complex128).requires_grad_(True)
    t, op, b = _transports(case, fat), _Operator(case, fat, lng), _source(case, seed, case["batch"])
    b = b.to(torch.complex64).to(torch.complex128)
    even, ys, grad = _parity(case) == 0, [], torch.zeros_like(w)
    for bi in b:
        y = _network(t, _layers(case, w), _full(case, bi))[0][even]
        res = op.a(case["mass"], y) - bi
        loss = (res.abs() ** 2).sum() / (bi.abs() ** 2).sum() / case["batch"]
        grad += torch.autograd.grad(loss, w)[0]
        ys.append(y.detach())
    g = torch.view_as_real(grad)
    step = 1e-4 * g / (g.abs() + 1e-8)  # Adam's first step
    return {"grad": grad, "weights": w.detach() - torch.view_as_complex(step), "y": torch.stack(ys)}


def _staple(u, v, mu, nu, sign):
    if sign > 0:
        return u[nu] @ _shift(v, nu, 1) @ _shift(u[nu], mu, 1).conj().transpose(-1, -2)
    un, vn = _shift(u[nu], nu, -1), _shift(v, nu, -1)
    return un.conj().transpose(-1, -2) @ vn @ _shift(un, mu, 1)


def _both(u, v, mu, nu):
    return _staple(u, v, mu, nu, 1) + _staple(u, v, mu, nu, -1)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("dslash", "apply"):
        fat, lng = _links(case, seed)
        op, b = _Operator(case, fat, lng), _source(case, seed).to(hq.fields.VEC_DTYPE[PREC[case["prec"]]])
        b = b.to(torch.complex128)
        return op.d(b, case["parity"]) if kind == "dslash" else op.a(case["mass"], b)
    if kind in ("cg", "fcg"):
        if _sites(case) > 300000:
            return None
        op = _Operator(case, *_links(case, seed, naive=kind == "fcg"), hops=((0, 1),) if kind == "fcg" else ((0, 1), (1, 3)))
        return _solve(op, case["mass"], _source(case, seed))
    if kind == "multi":
        if _sites(case) > 70000:
            return None
        op, b = _Operator(case, *_links(case, seed)), _source(case, seed, None if case["shift"] else case["nrhs"])
        return torch.stack([_solve(op, m, b if case["shift"] else b[i]) for i, m in enumerate(_masses(case))])
    if kind == "mdslash":
        op = _Operator(case, *_links(case, seed))
        b = _gauss(_gen(seed + 500009), _sites(case) // 2, case["nrhs"], 3).to(torch.complex64).to(torch.complex128)
        return torch.stack([op.d(b[:, i], case["parity"]) for i in range(case["nrhs"])], 1)
    if kind == "forward":
        fat = _links(case, seed)[0]
        t, w = _transports(case, fat), torch.from_numpy(_weights(case, seed)).cuda().to(torch.complex128)
        b = _source(case, seed, case["batch"]).to(torch.complex64).to(torch.complex128)
        even = _parity(case) == 0
        return torch.stack([_network(t, _layers(case, w), _full(case, v))[0][even] for v in b])
    if kind == "train":
        return _exact_train(case, seed, *_links(case, seed))
    u = _thin(case, seed)
    if kind == "fat":
        c, out = FAT7 if case["lepage"] else FAT7[:4] + (0.0,), []
        for mu in range(4):
            f = c[0] * u[mu]
            for nu in range(4):
                if nu == mu:
                    continue
                s3 = _both(u, u[mu], mu, nu)
                f = f + c[1] * s3
                for rho in range(4):
                    if rho in (mu, nu):
                        continue
                    s5 = _both(u, s3, mu, rho)
                    f = f + c[2] * s5 + c[3] * _both(u, s5, mu, 6 - mu - nu - rho)
                if c[4]:
                    for sg in (1, -1):
                        f = f + c[4] * _staple(u, _staple(u, u[mu], mu, nu, sg), mu, nu, sg)
            out.append(f)
        return torch.stack(out)
    long = torch.stack([u[mu] @ _shift(u[mu], mu, 1) @ _shift(u[mu], mu, 2) for mu in range(4)])
    out = {"long": _fold(case, long, 3)}
    for p in FORMS[case["form"]][1:]:
        if p:
            out[f"fat{PREC[p]}"] = out[f"long{PREC[p]}"] = None
    return out
