"""The work that this library's performance is judged on, as cases.

Each case goes through the public entry points the way a program does: the
specialization is requested once with the library's default structure and
tiles (the handle is kept), and a pass launches it on device buffers.  The
kinds:

  moments   LTimes, then LPlusTimes on its moments (FP64): the two moment
            operators of one transport iteration.  ``accumulate``: LPlusTimes
            adds into a source array that already holds values.
  bf16      LTimes on FP32 fluxes with BF16 products, plain or compensated.
  fused     LTimes and LPlusTimes in one launch, with or without the moments.
  scatter   the scattering source; materials in zone regions or drawn per zone.
  mass      the tensor-product mass operator over a mesh's elements.
  products  a batch of small square products through a kept plan.
  train     one training step of the cost model: gradient, then Adam.

Inputs come from the seed alone and are made on the GPU.
"""
import math

import numpy as np
import torch

from paper_1904_08555_amd import sj

LAYOUTS = ("DGZ", "DZG", "GDZ", "GZD", "ZDG", "ZGD")


def listed():
    return [
        # the smallest parity configuration: one launch moves 17 MB, so latency counts
        dict(name="moments_small_dgz", kind="moments", layout="DGZ", Z=4096, G=8, D=48, NM=16, accumulate=False),
        # one step of the six-nesting benchmark, a nesting whose zones are contiguous
        dict(name="moments_p3_dgz", kind="moments", layout="DGZ", Z=32768, G=32, D=96, NM=16, accumulate=False),
        # the next odd expansion order (25 moments) on 26^3 zones with directions contiguous, added into a source
        dict(name="moments_p4_gzd", kind="moments", layout="GZD", Z=17576, G=21, D=80, NM=25, accumulate=True),
        # the highest order of the range (64 moments), where FP64 arithmetic weighs as much as memory
        dict(name="moments_p7_dzg", kind="moments", layout="DZG", Z=64000, G=32, D=128, NM=64, accumulate=False),
        # FP32 fluxes at the same order, compensated BF16 products
        dict(name="ltimes_bf16x3_dgz", kind="bf16", layout="DGZ", Z=262144, G=16, D=128, NM=64, x3=True),
        # both operators in one launch, directions contiguous, moments wanted too
        dict(name="fused_p3_zgd", kind="fused", layout="ZGD", Z=32768, G=32, D=96, NM=16, phi=True),
        # the scattering benchmark: four materials in contiguous zone regions, moments contiguous
        dict(name="scatter_regions_zgd", kind="scatter", layout="ZGD", Z=32768, G=32, NM=16, nmat=4, mixed=False),
        # a fine group structure on a heterogeneous mesh: the material changes from zone to zone
        dict(name="scatter_mixed_dzg", kind="scatter", layout="DZG", Z=13824, G=44, NM=9, nmat=6, mixed=True),
        # cubic hexahedra, the mass-operator benchmark's mesh
        dict(name="mass_hex_d4q6", kind="mass", dim=3, D1D=4, Q1D=6, NE=500000),
        # high-order hexahedra: few elements, much arithmetic in each
        dict(name="mass_hex_d8q12", kind="mass", dim=3, D1D=8, Q1D=12, NE=20000),
        # 200,000 products of sizes 3 .. 16
        dict(name="products_200k", kind="products", count=200000, lo=3, hi=16),
        # a minibatch step as the picker trains (37 features, width 64)
        dict(name="train_b128", kind="train", rows=128, inputs=37, width=64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("moments",) * 4 + ("fused",) * 2 + ("scatter",) * 2 + ("mass",) * 2 + ("bf16", "products", "train"))
    layout = rng.choice(LAYOUTS)
    if kind in ("moments", "fused"):
        while True:
            c = dict(kind=kind, layout=layout, Z=_log(rng, 125, 65536), G=_log(rng, 1, 64), D=8 * rng.randint(2, 16),
                     NM=rng.choice((1, 4, 9, 16, 25, 36, 64)))
            if rng.random() < 0.15:
                c["D"] -= rng.randint(1, 7)
            if c["NM"] <= c["D"] and c["Z"] * c["G"] * (c["D"] + c["NM"]) <= 64000 * 32 * 192:
                break
        if kind == "moments":
            c["accumulate"] = rng.random() < 0.25
        else:
            c["phi"] = rng.random() < 0.5
        return c
    if kind == "bf16":
        return dict(kind=kind, layout=layout, Z=_log(rng, 4096, 131072), G=_log(rng, 2, 32), D=8 * rng.randint(4, 16),
                    NM=rng.choice((16, 25, 36, 64)), x3=rng.random() < 0.7)
    if kind == "scatter":
        return dict(kind=kind, layout=layout, Z=_log(rng, 512, 32768), G=rng.randint(6, 64), NM=rng.choice((1, 4, 9, 16, 25)),
                    nmat=rng.randint(1, 8), mixed=rng.random() < 0.4)
    if kind == "mass":
        dim = rng.choice((2, 3, 3))
        D1D = rng.randint(2, 9)
        Q1D = rng.randint(D1D, max(D1D, 2 * D1D - 2))
        most = 140000000 // (2 * D1D ** dim + Q1D ** dim)
        return dict(kind=kind, dim=dim, D1D=D1D, Q1D=Q1D, NE=_log(rng, 200, min(most, 1000000)))
    if kind == "products":
        lo = rng.randint(1, 12)
        return dict(kind=kind, count=_log(rng, 500, 200000), lo=lo, hi=rng.randint(lo, 16))
    return dict(kind=kind, rows=_log(rng, 16, 1024), inputs=rng.randint(8, 48), width=rng.choice((16, 32, 48, 64)))


# ------------------------------------------------------------- inputs

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _u01(g, n, dtype=torch.float64):
    return torch.rand(n, generator=g, device="cuda", dtype=dtype)


def _sym(g, n):
    return 2.0 * _u01(g, n) - 1.0


def _sizes(c):
    """Instance sizes of a batch: part of the case, the same for every seed."""
    return np.random.default_rng(c["count"]).integers(c["lo"], c["hi"] + 1, c["count"]).astype(np.int32)


def _inputs(c, seed):
    """The case's input arrays, by name."""
    g = _gen(seed)
    kind = c["kind"]
    if kind in ("moments", "fused", "bf16"):
        cols, D, NM = c["G"] * c["Z"], c["D"], c["NM"]
        # fluxes are positive, weights take both signs
        s = dict(L=_sym(g, NM * D), Lp=_sym(g, D * NM),
                 psi=_u01(g, D * cols, torch.float32 if kind == "bf16" else torch.float64))
        if kind == "moments":
            s["out"] = _u01(g, D * cols) if c["accumulate"] else torch.empty_like(s["psi"])
        return s
    if kind == "scatter":
        NM, G, Z, nmat = c["NM"], c["G"], c["Z"], c["nmat"]
        nl = math.isqrt(NM - 1) + 1
        s = dict(S=_u01(g, nmat * nl * G * G) / G, phi=_u01(g, NM * G * Z))
        if c["mixed"]:
            s["mat"] = torch.randint(0, nmat, (Z,), generator=g, device="cuda", dtype=torch.int32)
        else:
            s["mat"] = (torch.arange(Z, device="cuda") * nmat // Z).to(torch.int32)
        return s
    if kind == "mass":
        nd, nq = c["D1D"] ** c["dim"], c["Q1D"] ** c["dim"]
        return dict(B1=_sym(g, c["Q1D"] * c["D1D"]), Dq=_u01(g, c["NE"] * nq), X=_u01(g, c["NE"] * nd))
    if kind == "products":
        total = int((_sizes(c).astype(np.int64) ** 2).sum())
        return dict(A=torch.randn(total, generator=g, device="cuda", dtype=torch.float64),
                    B=torch.randn(total, generator=g, device="cuda", dtype=torch.float64))
    R, F, H = c["rows"], c["inputs"], c["width"]
    P = H * F + H * H + 3 * H + 1
    f32 = torch.float32
    lim = torch.cat([torch.full((H * F,), math.sqrt(6.0 / F)), torch.zeros(H), torch.full((H * H,), math.sqrt(6.0 / H)),
                     torch.zeros(H), torch.full((H,), math.sqrt(6.0 / H)), torch.zeros(1)]).to("cuda", f32)
    # optimizer state as in the middle of training
    return dict(theta=(2 * _u01(g, P, f32) - 1) * lim, X=torch.randn(R * F, generator=g, device="cuda", dtype=f32),
                t=torch.randn(R, generator=g, device="cuda", dtype=f32),
                m=0.02 * torch.randn(P, generator=g, device="cuda", dtype=f32), v=1e-3 * (0.5 + _u01(g, P, f32)))


_STEP, _LR = 100, 2e-3


def prepare(case, seed):
    sj.sj_init(0)
    c, s = case, _inputs(case, seed)
    s["case"] = c
    kind = c["kind"]
    dev = dict(device="cuda", dtype=torch.float64)
    if kind in ("moments", "fused", "bf16"):
        spec = dict(layout=c["layout"], Z=c["Z"], G=c["G"], D=c["D"], NM=c["NM"])
        cols = c["G"] * c["Z"]
        s["phi"] = torch.empty(c["NM"] * cols, device="cuda", dtype=s["psi"].dtype)
        if kind == "moments":
            s["hl"] = sj.sj_specialize(sj.SJ_LTIMES, **spec)
            s["hp"] = sj.sj_specialize(sj.SJ_LPLUSTIMES, flags=sj.SJ_FLAG_ACCUMULATE if c["accumulate"] else 0, **spec)
        elif kind == "fused":
            s["h"] = sj.sj_specialize(sj.SJ_LTIMES_LPLUS, **spec)
            s["out"] = torch.empty_like(s["psi"])
        else:
            s["h"] = sj.sj_specialize(sj.SJ_LTIMES, dtype=sj.SJ_BF16X3 if c["x3"] else sj.SJ_BF16, **spec)
    elif kind == "scatter":
        s["h"] = sj.sj_specialize(sj.SJ_SCATTERING, layout=c["layout"], Z=c["Z"], G=c["G"], NM=c["NM"], count=c["nmat"])
        s["out"] = torch.empty_like(s["phi"])
    elif kind == "mass":
        s["h"] = sj.sj_specialize(sj.SJ_MASS, D=c["D1D"], NM=c["Q1D"], inputs=c["dim"], count=c["NE"])
        s["Y"] = torch.empty_like(s["X"])
    elif kind == "products":
        mask = 0
        for n in range(c["lo"], c["hi"] + 1):
            mask |= 1 << n
        s["plan"] = _Plan(sj.sj_batch_plan(sj.sj_specialize(sj.SJ_BGEMM, class_mask=mask), _sizes(c)))
        s["C"] = torch.empty(s["A"].numel(), **dev)
    else:
        R, F, H = c["rows"], c["inputs"], c["width"]
        s["hb"] = sj.sj_specialize(sj.SJ_MLP_BWD, dtype=sj.SJ_F32, rows=R, inputs=F, width=H)
        s["ha"] = sj.sj_specialize(sj.SJ_ADAM, dtype=sj.SJ_F32, rows=s["theta"].numel())
        s["grad"] = torch.empty_like(s["theta"])
        s["loss"] = torch.empty(1, device="cuda", dtype=torch.float32)
        s["ws"] = torch.empty(R * (4 * H + 2), device="cuda", dtype=torch.float32)
        s["step"] = _STEP
    return s


class _Plan:
    """A batch plan that is given back with the state that holds it."""

    def __init__(self, plan):
        self.plan = plan

    def __del__(self):
        torch.cuda.synchronize()
        sj.sj_plan_destroy(self.plan)


def run(s):
    kind = s["case"]["kind"]
    if kind == "moments":
        sj.sj_run(s["hl"], [s["L"], s["psi"], s["phi"]])
        sj.sj_run(s["hp"], [s["Lp"], s["phi"], s["out"]])
        return s["phi"], s["out"]
    if kind == "fused":
        ptrs = [s["L"], s["Lp"], s["psi"], s["out"]]
        if s["case"]["phi"]:
            sj.sj_run(s["h"], ptrs + [s["phi"]])
            return s["phi"], s["out"]
        sj.sj_run(s["h"], ptrs)
        return s["out"]
    if kind == "bf16":
        sj.sj_run(s["h"], [s["L"], s["psi"], s["phi"]])
        return s["phi"]
    if kind == "scatter":
        sj.sj_run(s["h"], [s["S"], s["mat"], s["phi"], s["out"]])
        return s["out"]
    if kind == "mass":
        sj.sj_run(s["h"], [s["B1"], s["Dq"], s["X"], s["Y"]])
        return s["Y"]
    if kind == "products":
        sj.sj_batch_run(s["plan"].plan, s["A"], s["B"], s["C"])
        return s["C"]
    sj.sj_run(s["hb"], [s["theta"], s["X"], s["t"], s["grad"], s["loss"], s["ws"]])
    s["step"] += 1
    sj.sj_run_adam(s["ha"], [s["theta"], s["grad"], s["m"], s["v"]], s["step"], lr=_LR)
    return dict(grad=s["grad"], loss=s["loss"], theta=s["theta"], m=s["m"], v=s["v"])


def work(case):
    c, kind = case, case["kind"]
    if kind in ("moments", "fused", "bf16"):
        cols, D, NM = c["G"] * c["Z"], c["D"], c["NM"]
        w, one = 8 * D * NM, 2.0 * D * NM * cols
        if kind == "moments":   # psi in, phi out; phi in, psi' out (and in, when it accumulates)
            return dict(bytes=8 * cols * ((3 if c["accumulate"] else 2) * D + 2 * NM) + 2 * w, flops=2 * one)
        if kind == "fused":
            return dict(bytes=8 * cols * (2 * D + (NM if c["phi"] else 0)) + 2 * w, flops=2 * one)
        return dict(bytes=4 * cols * (D + NM) + w, flops=one)
    if kind == "scatter":
        NM, G, Z = c["NM"], c["G"], c["Z"]
        return dict(bytes=16 * NM * G * Z + 8 * c["nmat"] * (math.isqrt(NM - 1) + 1) * G * G + 4 * Z, flops=2.0 * NM * G * G * Z)
    if kind == "mass":
        d, D, Q = c["dim"], c["D1D"], c["Q1D"]
        chain = sum(D ** (d - i) * Q ** (i + 1) for i in range(d))   # one direction of the factorized operator
        return dict(bytes=8 * c["NE"] * (2 * D ** d + Q ** d) + 8 * D * Q, flops=c["NE"] * (4.0 * chain + Q ** d))
    if kind == "products":
        n = _sizes(c).astype(np.int64)
        return dict(bytes=int(24 * (n ** 2).sum()), flops=float(2 * (n ** 3).sum()))
    R, F, H = c["rows"], c["inputs"], c["width"]
    P = H * F + H * H + 3 * H + 1
    return dict(bytes=4 * (R * (F + 1) + 8 * P + 1), flops=2.0 * R * (2 * H * F + 3 * H * H + 2 * H) + 12.0 * P)


# ------------------------------------------------------------- 64-bit values

def _view(layout, Z, G):
    """Columns of a nesting as [B][rows][I]."""
    if layout in ("DGZ", "DZG"):
        return 1, G * Z
    if layout == "GDZ":
        return G, Z
    if layout == "ZDG":
        return Z, G
    return G * Z, 1


def _apply(W, x, B, I):
    """W times the rows of x [B][k][I]."""
    if I == 1:
        return (x.view(B, -1) @ W.t().contiguous()).reshape(-1)
    x = x.view(B, -1, I)
    y = torch.empty(B, W.shape[0], I, device=x.device, dtype=x.dtype)
    for b0 in range(0, B, 4096):
        torch.matmul(W, x[b0:b0 + 4096], out=y[b0:b0 + 4096])
    return y.reshape(-1)


def _axes(layout):
    """How an array stored in a nesting is permuted to (moment, group, zone)."""
    return [layout.index(a) for a in "DGZ"]


def exact(case, seed):
    c, s = case, _inputs(case, seed)
    kind = c["kind"]
    if kind in ("moments", "fused", "bf16"):
        B, I = _view(c["layout"], c["Z"], c["G"])
        L, Lp = s["L"].view(c["NM"], c["D"]), s["Lp"].view(c["D"], c["NM"])
        phi = _apply(L, s["psi"].double(), B, I)
        if kind == "bf16":
            return phi
        out = _apply(Lp, phi, B, I)
        if kind == "moments":
            return phi, (out + s["out"] if c["accumulate"] else out)
        return (phi, out) if c["phi"] else out
    if kind == "scatter":
        NM, G, Z = c["NM"], c["G"], c["Z"]
        size = dict(D=NM, G=G, Z=Z)
        phi = s["phi"].view([size[a] for a in c["layout"]]).permute(_axes(c["layout"]))
        out = torch.empty([size[a] for a in c["layout"]], device="cuda", dtype=torch.float64)
        res = out.permute(_axes(c["layout"]))
        S = s["S"].view(c["nmat"], -1, G, G)
        for k in range(c["nmat"]):
            zs = torch.nonzero(s["mat"] == k).reshape(-1)
            for nm in range(NM):
                res[nm][:, zs] = S[k, math.isqrt(nm)] @ phi[nm][:, zs].contiguous()
        return out.reshape(-1)
    if kind == "mass":
        NE, d, D, Q = c["NE"], c["dim"], c["D1D"], c["Q1D"]
        B1 = s["B1"].view(Q, D)

        def along(W, u):   # contract the fastest index and make it the slowest: after d turns the order is the first again
            u = u.reshape(NE, -1, W.shape[1]) @ W.t().contiguous()
            return u.transpose(1, 2).contiguous()

        u = s["X"].view(NE, -1)
        for _ in range(d):
            u = along(B1, u)
        u = u.reshape(NE, -1) * s["Dq"].view(NE, -1)
        for _ in range(d):
            u = along(B1.t().contiguous(), u)
        return u.reshape(-1)
    if kind == "products":
        n = torch.from_numpy(_sizes(c).astype(np.int64)).cuda()
        off = torch.cumsum(n * n, 0) - n * n
        out = torch.empty(s["A"].numel(), device="cuda", dtype=torch.float64)
        for k in range(c["lo"], c["hi"] + 1):
            at = off[n == k][:, None] + torch.arange(k * k, device="cuda")
            if at.numel():
                out[at] = torch.bmm(s["A"][at].view(-1, k, k), s["B"][at].view(-1, k, k)).view(-1, k * k)
        return out
    R, F, H = c["rows"], c["inputs"], c["width"]
    th = s["theta"].double().requires_grad_(True)
    W1, b1, W2, b2, w3, b3 = torch.split(th, [H * F, H, H * H, H, H, 1])
    h = torch.relu(s["X"].double().view(R, F) @ W1.view(H, F).t() + b1)
    y = torch.relu(h @ W2.view(H, H).t() + b2) @ w3 + b3
    loss = ((y - s["t"].double()) ** 2).mean()
    (g,) = torch.autograd.grad(loss, th)
    m = 0.9 * s["m"].double() + 0.1 * g
    v = 0.999 * s["v"].double() + 0.001 * g * g
    k = _STEP + 1
    p = th.detach() - _LR * (m / (1 - 0.9 ** k)) / (torch.sqrt(v / (1 - 0.999 ** k)) + 1e-8)
    return dict(grad=g, loss=loss.detach().reshape(1), theta=p, m=m, v=v)
