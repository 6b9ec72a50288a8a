"""Performance cases of the density-fitting library: what its users have it do, with their sizes.

A case is a dict of plain values: "op" names the call, the rest are sizes.  `listed()` gives the fixed
cases, `draw(rng)` one more of the same ranges, `prepare(case, seed)` what a program holds before the
call (inputs on the GPU, int8 planes of B where the call takes them), `run(state)` one pass through the
public entry points with its outputs, `work(case)` the bytes and FP64 operations the pass cannot do
without, and `exact(case, seed)` the same outputs in plain FP64 torch, without this library.

Inputs follow the workloads of paper_2505_03755_amd/synth.py: B[P, pair(i, j)] = N(0,1) exp(-|i-j| / L),
orthonormal orbitals, 8-fold symmetric Gamma, a Coulomb metric with a geometric spectrum.  N_aux is
about 4 N_ao and N_occ about N_ao / 4 throughout, as in those workloads.
"""
from __future__ import annotations

import math

import torch

from paper_2505_03755_amd import dfmi

DEV = "cuda:0"


def listed():
    return [
        # one contraction step of a small molecule or fragment: launches and latency count
        {"name": "step-120", "op": "step", "nao": 120, "naux": 480, "nocc": 30, "nac": 8},
        # the same for a medium system
        {"name": "step-600", "op": "step", "nao": 600, "naux": 2400, "nocc": 150, "nac": 20},
        # the benchmark: forward step with X kept, then the adjoint for the energy's cotangents
        {"name": "grad-1200", "op": "grad", "nao": 1200, "naux": 4800, "nocc": 300, "nac": 40},
        # an orbital-optimisation step through autograd, X recomputed in the backward; ragged sizes
        {"name": "autograd-341", "op": "autograd", "nao": 341, "naux": 1365, "nocc": 85, "nac": 13},
        # one Fock build of an SCF iteration on a small, ragged basis
        {"name": "jk-77", "op": "jk", "nao": 77, "naux": 310, "nocc": 19, "ndm": 1, "weighted": False},
        # a Fock build for two densities with signed occupation weights (spin, or a general density)
        {"name": "jk-455x2w", "op": "jk", "nao": 455, "naux": 1822, "nocc": 113, "ndm": 2, "weighted": True},
        # the fragment batch: 8 uneven embedding problems ("N_emb x N_ac"), 64 densities each
        {"name": "fragments-8x64", "op": "batch", "frags": "80x4,120x4,160x6,200x6,240x6,280x8,340x8,400x8",
         "ndm": 64, "ppaa": False},
        # a small batch with few densities, (pq|uv) asked for too
        {"name": "fragments-4x2", "op": "batch", "frags": "80x4,120x4,160x6,200x6", "ndm": 2, "ppaa": True},
        # the full (pu|qv) block of an AO2MO call, all orbitals on both general indices
        {"name": "papa-500", "op": "papa", "nao": 500, "naux": 2000, "nac": 12},
        # (pq|uv) over all orbitals of a medium system
        {"name": "ppaa-600", "op": "ppaa", "nao": 600, "naux": 2400, "nac": 20},
        # forming B once per geometry, from the metric and the three-centre integrals
        {"name": "build-600", "op": "build", "nao": 600, "naux": 2400},
        # the gradient step in split precision (7 int8 slices, B split once beforehand)
        {"name": "split-grad-800", "op": "split", "nao": 800, "naux": 3200, "nocc": 200, "nac": 24},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["step", "step", "grad", "autograd", "jk", "jk", "batch", "batch", "papa", "ppaa", "build", "split"])
    top = {"step": 1200, "grad": 1150, "autograd": 700, "jk": 700, "papa": 560, "ppaa": 700, "build": 800, "split": 800}
    if op == "batch":
        n = rng.randint(2, 8)
        frags = [(_log(rng, 40, 400), rng.randint(2, 8)) for _ in range(n)]
        ndm = _log(rng, 1, 64)
        return {"op": op, "frags": ",".join("%dx%d" % f for f in frags), "ndm": ndm, "ppaa": rng.random() < 0.3}
    nao = _log(rng, {"step": 48, "jk": 32, "grad": 120, "autograd": 100, "papa": 64, "ppaa": 64, "build": 64,
                     "split": 200}[op], top[op])
    naux = max(4, int(nao * rng.uniform(3.2, 4.0)))
    nocc = max(1, int(nao * rng.uniform(0.12, 0.25)))
    nac = max(2, min(40, nao // 8, _log(rng, 4, 40)))
    if op == "jk":
        ndm = rng.choice([1, 1, 1, 2, 2, 3, 4])
        return {"op": op, "nao": nao, "naux": naux, "nocc": nocc, "ndm": ndm, "weighted": rng.random() < 0.4}
    if op == "papa":
        return {"op": op, "nao": nao, "naux": naux, "nac": min(nac, 12)}
    if op == "ppaa":
        return {"op": op, "nao": nao, "naux": naux, "nac": min(nac, 20)}
    if op == "build":
        return {"op": op, "nao": nao, "naux": naux}
    return {"op": op, "nao": nao, "naux": naux, "nocc": nocc, "nac": nac}


# ---- inputs ----

def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1_000_003 + 7919 * int(stream)) % (1 << 62))
    return g


def _randn(shape, g):
    return torch.randn(shape, generator=g, dtype=torch.float64, device=DEV)


def _npair(n):
    return n * (n + 1) // 2


def _tril(nao):
    return torch.tril_indices(nao, nao, device=DEV)


def _packed(naux, nao, g, L):
    """B or (Q|mu nu): N(0,1) exp(-|i - j| / L) over the packed pairs."""
    il, jl = _tril(nao)
    env = torch.exp(-(il - jl).double() / L)
    out = torch.empty((naux, _npair(nao)), dtype=torch.float64, device=DEV)
    for r in range(0, naux, 512):
        torch.randn(out[r:r + 512].shape, generator=g, dtype=torch.float64, device=DEV, out=out[r:r + 512])
        out[r:r + 512].mul_(env)
    return out


def _orthonormal(batch, n, m, g):
    """batch x n x m with orthonormal columns: A (A^T A)^(-1/2) in Cholesky form, twice."""
    a = _randn((batch, n, m), g)
    for _ in range(2):
        l = torch.linalg.cholesky_ex(a.transpose(1, 2) @ a)[0]
        a = torch.linalg.solve_triangular(l, a.transpose(1, 2), upper=False).transpose(1, 2).contiguous()
    return a


def _orbitals(nao, g):
    return torch.linalg.qr(_randn((nao, nao), g))[0].contiguous()


def _gamma(nac, g):
    """Random two-body density with the 8-fold symmetry of (uv|wx)."""
    x = _randn((nac,) * 4, g)
    x = x + x.transpose(0, 1)
    x = x + x.transpose(2, 3)
    return ((x + x.permute(2, 3, 0, 1)) / 8.0).contiguous()


def _decay(nao):
    return 20.0 if nao <= 400 else 40.0


def _frags(case):
    return [tuple(int(v) for v in f.split("x")) for f in case["frags"].split(",")]


def _inputs(case, seed):
    op = case["op"]
    g = _gen(seed, 1)
    if op == "batch":
        probs = []
        for nemb, nac in _frags(case):
            nocc = nemb // 4
            C = _orbitals(nemb, g)
            probs.append({"B": _packed(4 * nemb, nemb, g, 20.0), "nao": nemb,
                          "Cocc": _orthonormal(case["ndm"], nemb, nocc, g),
                          "Cact": C[:, nocc:nocc + nac].contiguous(), "Cp": C})
        return {"probs": probs}
    nao, naux = case["nao"], case["naux"]
    if op == "build":
        q = torch.linalg.qr(_randn((naux, naux), g))[0]
        lam = torch.logspace(0.0, -6.0, naux, dtype=torch.float64, device=DEV)
        m = (q * lam) @ q.T
        return {"metric": ((m + m.T) * 0.5).contiguous(), "E": _packed(naux, nao, g, _decay(nao))}
    s = {"B": _packed(naux, nao, g, _decay(nao))}
    if op == "jk":
        s["Cocc"] = _orthonormal(case["ndm"], nao, case["nocc"], g)
        if case["weighted"]:   # signed occupations of a general symmetric density
            s["w"] = torch.rand((case["ndm"], case["nocc"]), generator=g, dtype=torch.float64, device=DEV) * 2.2 - 0.2
        return s
    C = _orbitals(nao, g)
    nocc, nac = case.get("nocc", nao // 4), case["nac"]
    s["C"] = C
    s["Cact"] = C[:, nocc:nocc + nac].contiguous()
    if op in ("papa", "ppaa"):
        return s
    s["Cocc"] = C[:, :nocc].contiguous()
    if op != "step":   # cotangents of the model energy: gJ = D/2, gK = -D/4, geri = Gamma/2
        D = s["Cocc"] @ s["Cocc"].T
        s["gJ"], s["gK"], s["ge"] = (0.5 * D).contiguous(), (-0.25 * D).contiguous(), (0.5 * _gamma(nac, g)).contiguous()
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    if case["op"] == "split":   # split once per B, like B itself
        s["Bs"], s["Be"] = dfmi.split_cholesky(s["B"], case["nao"])
        s["Bt"], s["Bte"] = dfmi.split_cholesky_t(s["B"], case["nao"])
    if case["op"] == "autograd":
        s["Cocc"].requires_grad_(True)
        s["Cact"].requires_grad_(True)
    return s


# ---- one pass ----

def run(s):
    case = s["case"]
    op = case["op"]
    if op == "batch":
        return dfmi.batched_step(s["probs"], ppaa=case["ppaa"])
    if op == "build":
        L, B, _ = dfmi.build_cholesky(s["metric"], s["E"], case["nao"])
        return {"L": L, "B": B}
    B, nao = s["B"], case["nao"]
    if op == "jk":
        J, K, v = dfmi.jk(B, nao, s["Cocc"], w=s.get("w"))
        return {"J": J, "K": K, "v": v}
    if op == "papa":
        return {"papa": dfmi.papa(B, nao, s["C"], s["Cact"], Cq=s["C"])}
    if op == "ppaa":
        return {"ppaa": dfmi.ppaa(B, nao, s["C"], s["Cact"])}
    Cocc, Cact = s["Cocc"], s["Cact"]
    if op == "step":
        return dfmi.step(B, nao, Cocc, Cact, s["C"])
    if op == "grad":
        o = dfmi.step(B, nao, Cocc, Cact, s["C"], keep_x=True)
        Xo, Xa = o.pop("Xocc"), o.pop("Xact")
        o["dCocc"], o["dCact"] = dfmi.step_backward(B, nao, Cocc, Cact, s["gJ"], s["gK"], s["ge"], Xo, Xa)
        return o
    if op == "split":
        o = dfmi.step_split(B, s["Bs"], s["Be"], nao, Cocc, Cact, s["C"], keep_x=True)
        Xo, Xa = o.pop("Xocc"), o.pop("Xact")
        o["dCocc"], o["dCact"] = dfmi.step_backward_split(B, s["Bt"], s["Bte"], nao, Cocc, Cact, s["gJ"], s["gK"],
                                                          s["ge"], Xo, Xa)
        return o
    J, K, eri = dfmi.dfstep_apply(B, nao, Cocc, Cact, keep_x=False)
    dCocc, dCact = torch.autograd.grad((J, K, eri), (Cocc, Cact), (s["gJ"], s["gK"], s["ge"]))
    return {"J": J.detach(), "K": K.detach(), "eri": eri.detach(), "dCocc": dCocc, "dCact": dCact}


# ---- what a pass cannot do without ----

def _forward_work(naux, nao, nocc, nac, nmo):
    npair = _npair(nao)
    f = (2 * naux * nao * nao * (nocc + nac) + 2 * naux * nao * nocc + 2 * naux * npair
         + naux * nocc * nao * (nao + 1) + 2 * naux * nao * nac * nac + 2 * naux * nac ** 4)
    b = naux * npair + nao * (nocc + nac) + 2 * nao * nao + naux + nac ** 4
    if nmo:
        f += 2 * naux * nao * nmo * nac + 2 * naux * nmo * nac ** 3
        b += nao * nmo + nmo * nac ** 3
    return f, b


def _ppaa_work(naux, nao, nac, nmo):
    npair, nuv = _npair(nao), _npair(nac)
    f = (2 * naux * nao * nao * nac + 2 * naux * nao * nac * nac + 2 * naux * npair * nuv
         + 2 * nuv * nao * nmo * (nao + nmo))
    return f, naux * npair + nao * (nac + nmo) + nuv * nmo * nmo


def work(case):
    op = case["op"]
    if op == "batch":
        f = b = 0
        for n, nac in _frags(case):
            naux, nocc, ndm, npair = 4 * n, n // 4, case["ndm"], _npair(n)
            f += (2 * naux * n * n * (ndm * nocc + nac) + ndm * (2 * naux * n * nocc + 2 * naux * npair)
                  + ndm * naux * nocc * n * (n + 1) + 2 * naux * n * n * nac + 2 * naux * (n * nac) ** 2
                  + 2 * naux * n * nac * nac + 2 * naux * nac ** 4)
            b += naux * npair + ndm * n * nocc + n * nac + n * n + 2 * ndm * n * n + nac ** 4 + (n * nac) ** 2
            if case["ppaa"]:
                nuv = _npair(nac)
                f += 2 * naux * npair * nuv + 4 * nuv * n ** 3
                b += nuv * n * n
        return {"bytes": 8 * b, "flops": f}
    nao, naux = case["nao"], case["naux"]
    npair = _npair(nao)
    if op == "build":
        return {"bytes": 8 * (2 * naux * npair + 2 * naux * naux), "flops": naux ** 3 / 3 + naux * naux * npair}
    if op == "jk":
        ndm, nocc = case["ndm"], case["nocc"]
        return {"bytes": 8 * (naux * npair + ndm * (nao * nocc + 2 * nao * nao + naux)),
                "flops": ndm * (2 * naux * nao * nao * nocc + 2 * naux * nao * nocc + 2 * naux * npair
                                + naux * nocc * nao * (nao + 1))}
    nac = case["nac"]
    if op == "papa":
        return {"bytes": 8 * (naux * npair + nao * (nao + nac) + (nao * nac) ** 2),
                "flops": 2 * naux * nao * nao * nac * 2 + 2 * naux * (nao * nac) ** 2}
    if op == "ppaa":
        f, b = _ppaa_work(naux, nao, nac, nao)
        return {"bytes": 8 * b, "flops": f}
    nocc = case["nocc"]
    f, b = _forward_work(naux, nao, nocc, nac, 0 if op == "autograd" else nao)
    if op != "step":
        f += (4 * naux * npair + 2 * nao * nao * nocc + 4 * naux * nao * nao * nocc + 2 * naux * nac ** 4
              + 2 * naux * nao * nac * nac)
        b += 2 * nao * nao + nac ** 4 + nao * (nocc + nac)
    return {"bytes": 8 * b, "flops": f}


# ---- the same outputs in plain FP64 torch ----

def _unpacked(B, nao, p0, p1):
    i = torch.arange(nao, device=DEV)
    hi, lo = torch.maximum(i[:, None], i[None, :]), torch.minimum(i[:, None], i[None, :])
    return B[p0:p1].index_select(1, (hi * (hi + 1) // 2 + lo).reshape(-1)).reshape(p1 - p0, nao, nao)


def _blocks(B, nao):
    per = max(1, min(B.shape[0], (1 << 27) // (nao * nao)))
    for p0 in range(0, B.shape[0], per):
        p1 = min(B.shape[0], p0 + per)
        yield p0, p1, _unpacked(B, nao, p0, p1)


def _sym(packed, nao):
    il, jl = _tril(nao)
    out = torch.empty((packed.shape[0], nao, nao), dtype=torch.float64, device=DEV)
    out[:, il, jl] = packed
    out[:, jl, il] = packed
    return out


def _exact_jk(B, nao, Cocc, w):
    """J, K, v of the densities Cocc [ndm, nao, nocc] with weights w [ndm, nocc] or None."""
    ndm, nocc = Cocc.shape[0], Cocc.shape[2]
    v = torch.empty((ndm, B.shape[0]), dtype=torch.float64, device=DEV)
    K = torch.zeros((ndm, nao, nao), dtype=torch.float64, device=DEV)
    for p0, p1, b in _blocks(B, nao):
        for z in range(ndm):
            X = b @ Cocc[z]
            Cw = Cocc[z] if w is None else Cocc[z] * w[z]
            v[z, p0:p1] = (X * Cw).sum((1, 2))
            Xr = X.permute(1, 0, 2).reshape(nao, -1)
            Xw = Xr if w is None else (X * w[z]).permute(1, 0, 2).reshape(nao, -1)
            K[z] += Xw @ Xr.T
    return _sym(v @ B, nao), K, v


def _exact_active(B, nao, Cp, Cact):
    """b_pu [naux, np, nac] (or None) and b_uv [naux, nac, nac]."""
    bpu, buv = [], []
    for _, _, b in _blocks(B, nao):
        X = b @ Cact
        buv.append(Cact.T @ X)
        if Cp is not None:
            bpu.append(Cp.T @ X)
    return torch.cat(bpu) if bpu else None, torch.cat(buv)


def _gram(a, b):
    return a.reshape(a.shape[0], -1).T @ b.reshape(b.shape[0], -1)


def _exact_step(s, nao, papa=True):
    B, Cocc, Cact = s["B"], s["Cocc"].detach(), s["Cact"].detach()
    J, K, v = _exact_jk(B, nao, Cocc[None], None)
    nac = Cact.shape[1]
    bpu, buv = _exact_active(B, nao, s["C"] if papa else None, Cact)
    o = {"J": J[0], "K": K[0], "v": v[0], "eri": _gram(buv, buv).reshape((nac,) * 4)}
    if papa:
        o["papa"] = _gram(bpu, buv).reshape(nao, nac, nac, nac)
    return o, buv


def _exact_vjp(s, nao, buv):
    B, Cocc, Cact = s["B"], s["Cocc"].detach(), s["Cact"].detach()
    nac = Cact.shape[1]
    il, jl = _tril(nao)
    gp = torch.where(il == jl, s["gJ"][il, jl], s["gJ"][il, jl] + s["gJ"][jl, il])
    M = _sym(((B @ gp) @ B)[None], nao)[0]
    dCocc, S = 2.0 * (M @ Cocc), s["gK"] + s["gK"].T
    G = s["ge"].reshape(nac * nac, nac * nac)
    Z = (buv.reshape(-1, nac * nac) @ (G + G.T)).reshape(-1, nac, nac)
    Z = Z + Z.transpose(1, 2)
    dCact = torch.zeros_like(Cact)
    for p0, p1, b in _blocks(B, nao):
        Y = S @ (b @ Cocc)
        dCocc += b.permute(1, 0, 2).reshape(nao, -1) @ Y.reshape(-1, Y.shape[2])
        X = b @ Cact
        dCact += X.permute(1, 0, 2).reshape(nao, -1) @ Z[p0:p1].reshape(-1, nac)
    return dCocc, dCact


def _exact_ppaa(B, nao, C, buv):
    u, v = _tril(buv.shape[1])
    W = buv[:, u, v].T @ B
    return torch.cat([C.T @ (_sym(W[k:k + 16], nao) @ C) for k in range(0, W.shape[0], 16)])


def exact(case, seed):
    op = case["op"]
    s = _inputs(case, seed)
    if op == "batch":
        outs = []
        for p in s["probs"]:
            B, n, Cact = p["B"], p["nao"], p["Cact"]
            J, K, _ = _exact_jk(B, n, p["Cocc"], None)
            nac = Cact.shape[1]
            bpu, buv = _exact_active(B, n, p["Cp"], Cact)
            o = {"J": J, "K": K, "eri": _gram(buv, buv).reshape((nac,) * 4),
                 "papa": _gram(bpu, bpu).reshape(n, nac, n, nac)}
            if case["ppaa"]:
                o["ppaa"] = _exact_ppaa(B, n, p["Cp"], buv)
            outs.append(o)
        return outs
    nao = case["nao"]
    if op == "build":
        L = torch.linalg.cholesky(s["metric"].cpu())
        eye = torch.eye(L.shape[0], dtype=torch.float64)
        Li, L = torch.linalg.solve_triangular(L, eye, upper=False).to(DEV), L.to(DEV)
        B = Li @ s["E"]
        B += Li @ (s["E"] - L @ B)   # one step of refinement: the inverse's own error drops out
        return {"L": L, "B": B}
    if op == "jk":
        J, K, v = _exact_jk(s["B"], nao, s["Cocc"], s.get("w"))
        return {"J": J, "K": K, "v": v}
    if op == "papa":
        nac = case["nac"]
        bpu, _ = _exact_active(s["B"], nao, s["C"], s["Cact"])
        return {"papa": _gram(bpu, bpu).reshape(nao, nac, nao, nac)}
    if op == "ppaa":
        _, buv = _exact_active(s["B"], nao, None, s["Cact"])
        return {"ppaa": _exact_ppaa(s["B"], nao, s["C"], buv)}
    o, buv = _exact_step(s, nao, papa=op != "autograd")
    if op == "step":
        return o
    o["dCocc"], o["dCact"] = _exact_vjp(s, nao, buv)
    if op == "autograd":
        o.pop("v")
    return o
