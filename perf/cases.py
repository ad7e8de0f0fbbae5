"""Performance cases of dexmi: the work a program has the library do, through its
public entry points (paper_2104_05372_amd.dex and .autograd), from the smallest
calls to the largest.

  listed()             the named cases
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  inputs, descriptor, buffers and workspaces, on the GPU
  run(state)           one pass; returns its outputs
  work(case)           bytes and flops the pass cannot do without
  exact(case, seed)    run's outputs in 64 bits, by plain torch
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2104_05372_amd import autograd, dex

VARIANT = {"plain": dex.DEX_GMM_PLAIN, "16bit": dex.DEX_GMM_BF16, "split16": dex.DEX_GMM_BF16X3}
BATCH_VARIANT = {"plain": dex.DEX_GMM_PLAIN, "f16x3": dex.DEX_GMM_F16X3}
DTYPE = {"f32": torch.float32, "f64": torch.float64}


def listed():
    return [
        # An FP64 mixture fit of a few parameters: one objective and gradient per
        # optimiser step, so launches and latency are what it costs.
        dict(name="gmm_f64_small", kind="gmm", N=1000, D=2, K=5, dtype="f64", variant="plain",
             mode="grad", api="dex"),
        # A medium FP64 fit (full double precision, ragged point count).
        dict(name="gmm_f64_mid", kind="gmm", N=20_011, D=16, K=25, dtype="f64", variant="plain",
             mode="grad", api="dex"),
        # An FP32 fit of odd sizes inside a torch training loop.
        dict(name="gmm_f32_ragged", kind="gmm", N=30_011, D=20, K=37, dtype="f32",
             variant="plain", mode="grad", api="autograd"),
        # The large fit: 16-bit products, 1e5 points, 64 dimensions, 200 components.
        dict(name="gmm_16bit_large", kind="gmm", N=100_000, D=64, K=200, dtype="f32",
             variant="16bit", mode="grad", api="dex"),
        # Forward mode: the objective and its derivative along a direction (line
        # searches, Hessian-free methods), FP32.
        dict(name="gmm_f32_tangent", kind="gmm", N=20_000, D=32, K=50, dtype="f32",
             variant="plain", mode="jvp", api="dex"),
        # 512 mixtures of uneven sizes fitted together, FP32.
        dict(name="gmm_batched", kind="batched", B=512, nmin=1000, nmax=50_000, shape_seed=3,
             variant="plain"),
        # An embedding table of a million rows: lookup, and its transpose.
        dict(name="gather_large", kind="gather", V=1_000_000, R=128, n=4_194_304, mode="grad"),
        # A small table with rows of odd length inside a training loop.
        dict(name="gather_ragged", kind="gather", V=50_021, R=50, n=100_003, mode="grad"),
        # Integer histogram of 2^26 skewed keys.
        dict(name="histogram", kind="hist", bins=65_536, n=1 << 26),
        # A long in-place diffusion loop with a non-linear term on the large grid:
        # forward with checkpoints, reverse with recomputation.
        dict(name="stencil_large", kind="stencil", H=4096, W=4096, steps=200, every=32, rho=-0.2,
             variant="recompute", mode="grad"),
        # The same loop, linear, on a small grid of odd sizes, in a training loop.
        dict(name="stencil_ragged", kind="stencil", H=601, W=333, steps=100, every=32, rho=0.0,
             variant="linear", mode="grad"),
        # Row sums of a tall matrix and the sum of everything.
        dict(name="reductions", kind="reduce", rows=1 << 20, cols=128),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["gmm", "gmm", "gmm", "batched", "gather", "gather", "accum", "hist",
                       "stencil", "stencil", "reduce"])
    if kind == "gmm":
        form = rng.choice([("f64", "plain"), ("f32", "plain"), ("f32", "16bit"), ("f32", "split16")])
        D = rng.choice([2, 3, 8, 13, 16, 20, 32, 47, 64]) if form[0] == "f32" else _log_int(rng, 2, 32)
        K = _log_int(rng, 2, 200)
        # the FP64 and FP32 forms at sizes up to that of the listed ones, the 16-bit
        # form up to the large fit
        top = {"f64": 1.2e8, "f32": 6e9 if form[1] == "16bit" else 3e9}[form[0]]
        N = min(_log_int(rng, 500, 100_000), max(500, int(top / (K * D * D))))
        return dict(kind="gmm", N=N, D=D, K=K, dtype=form[0], variant=form[1],
                    mode=rng.choice(["grad", "grad", "jvp"]), api=rng.choice(["dex", "autograd"]))
    if kind == "batched":
        return dict(kind="batched", B=_log_int(rng, 8, 512), nmin=500,
                    nmax=_log_int(rng, 1000, 50_000), shape_seed=rng.randrange(1 << 20),
                    variant=rng.choice(["plain", "f16x3"]))
    if kind in ("gather", "accum"):
        R = rng.choice([1, 3, 8, 17, 32, 50, 64, 100, 128, 256, 300])
        n = min(_log_int(rng, 1000, 4_000_000), 500_000_000 // R)
        V = min(_log_int(rng, 100, 1_000_000), 128_000_000 // R)
        if kind == "gather":
            return dict(kind=kind, V=V, R=R, n=n, mode=rng.choice(["grad", "grad", "jvp"]))
        return dict(kind=kind, V=V, R=R, n=n, deterministic=rng.random() < 0.5)
    if kind == "hist":
        return dict(kind=kind, bins=_log_int(rng, 16, 65_536), n=_log_int(rng, 1000, 1 << 26))
    if kind == "stencil":
        H, W = _log_int(rng, 64, 4096), _log_int(rng, 64, 4096)
        if rng.random() < 0.5:
            H, W = (H + 31) // 32 * 32, (W + 255) // 256 * 256
        rho = rng.choice([0.0, -0.05, -0.2])  # damping terms: the loop stays well conditioned
        return dict(kind=kind, H=H, W=W, steps=_log_int(rng, 10, 200), every=rng.choice([8, 20, 32]),
                    rho=rho, variant="recompute" if rho or rng.random() < 0.5 else "linear",
                    mode=rng.choice(["grad", "grad", "jvp"]))
    cols = _log_int(rng, 1, 4096)
    return dict(kind="reduce", rows=min(_log_int(rng, 100, 1 << 20), (1 << 27) // cols), cols=cols)


# ---- inputs ------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(g, *shape, scale=1.0):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float64) * scale


def _zipf(g, n, s=1.1):
    """k >= 1 drawn from Zipf(s) by Devroye's rejection method, int64."""
    b, got, have = 2.0 ** (s - 1.0), [], 0
    while have < n:
        m = int(1.6 * (n - have)) + 1024
        u = torch.rand(m, generator=g, device="cuda", dtype=torch.float64)
        v = torch.rand(m, generator=g, device="cuda", dtype=torch.float64)
        x = torch.floor((1.0 - u) ** (-1.0 / (s - 1.0)))
        t = (1.0 + 1.0 / x) ** (s - 1.0)
        x = x[(v * x * (t - 1.0) / (b - 1.0) <= t / b) & (x < 9e18)]
        got.append(x.to(torch.int64))
        have += x.numel()
    return torch.cat(got)[:n]


def _gmm_data(g, N, D, K, dtype):
    data = (_normal(g, K), _normal(g, K, D), _normal(g, K, D, scale=0.1),
            _normal(g, K, D * (D - 1) // 2, scale=0.1), _normal(g, N, D))
    return [t.to(dtype) for t in data]  # alphas, means, qd, l, x


def _shapes(c):
    r = np.random.default_rng(c["shape_seed"])
    B = c["B"]
    return np.stack([r.integers(c["nmin"], c["nmax"], size=B, endpoint=True),
                     r.choice(np.array([8, 16, 32]), size=B),
                     r.integers(10, 100, size=B, endpoint=True)], axis=1).astype(np.int64)


def _inputs(c, seed):
    g = _gen(seed)
    kind = c["kind"]
    if kind == "gmm":
        dt = DTYPE[c["dtype"]]
        data = _gmm_data(g, c["N"], c["D"], c["K"], dt)
        tangents = [_normal(g, *t.shape).to(dt) for t in data[:4]] if c["mode"] == "jvp" else []
        return dict(data=data, tangents=tangents)
    if kind == "batched":
        shapes = _shapes(c)
        N, D, K = (torch.from_numpy(shapes[:, i].copy()) for i in range(3))
        draw_ = lambda m, s=1.0: torch.randn(int(m), generator=g, device="cuda") * s  # noqa: E731
        return dict(shapes=shapes, alphas=draw_(K.sum()), means=draw_((K * D).sum()),
                    qd=draw_((K * D).sum(), 0.1), l=draw_((K * D * (D - 1) // 2).sum(), 0.1),
                    x=draw_((N * D).sum()))
    if kind in ("gather", "accum"):
        V, R, n = c["V"], c["R"], c["n"]
        f = lambda *s: torch.randn(*s, generator=g, device="cuda")  # noqa: E731
        i = dict(idx=((_zipf(g, n) - 1) % V).to(torch.int32),
                 w=torch.rand(n, generator=g, device="cuda") * 2 - 1, T=f(V, R))
        if kind == "gather" and c["mode"] == "jvp":
            i.update(tT=f(V, R), tw=f(n))
        else:
            i["g"] = f(n, R)
        return i
    if kind == "hist":
        return dict(keys=(_zipf(g, c["n"]) % c["bins"]).to(torch.int32))
    if kind == "stencil":
        m = 4 if c["mode"] == "jvp" else 2
        return dict(fields=[torch.randn(c["H"], c["W"], generator=g, device="cuda") for _ in range(m)])
    return dict(values=torch.randn(c["rows"], c["cols"], generator=g, device="cuda"))


def prepare(case, seed):
    s = dict(case=case, **_inputs(case, seed))
    kind = case["kind"]
    dev = torch.device("cuda")
    ws = lambda d, role: dex.workspace(dex.dex_workspace_bytes(d, role), dev)  # noqa: E731
    if kind == "gmm":
        if case["api"] == "autograd" and case["mode"] == "grad":
            s["params"] = [t.requires_grad_() for t in s["data"][:4]]
            return s
        dt = DTYPE[case["dtype"]]
        code = dex.DEX_F64 if dt == torch.float64 else dex.DEX_F32
        d = dex.gmm_desc(case["N"], case["D"], case["K"], code, VARIANT[case["variant"]])
        s["desc"] = d
        s["F"] = torch.empty(1, dtype=dt, device=dev)
        s["resid"] = [torch.empty(case["N"], dtype=dt, device=dev),
                      torch.empty(dex.dex_workspace_bytes(d, dex.DEX_WS_RESID), dtype=torch.uint8,
                                  device=dev)]
        s["ws_fwd"] = ws(d, dex.DEX_WS_FWD)
        if case["mode"] == "grad":
            s["ws_vjp"], s["ct"] = ws(d, dex.DEX_WS_VJP), torch.ones(1, dtype=dt, device=dev)
            s["grads"] = [torch.empty_like(t) for t in s["data"][:4]]
        else:
            s["ws_jvp"], s["dF"] = ws(d, dex.DEX_WS_JVP), torch.empty(1, dtype=dt, device=dev)
    elif kind == "batched":
        d, plan = dex.dex_gmm_batched_plan(s["shapes"], BATCH_VARIANT[case["variant"]])
        s["desc"] = d
        s["ins"] = [torch.from_numpy(plan).to(dev), s["alphas"], s["means"], s["qd"], s["l"], s["x"]]
        s["F"] = torch.empty(case["B"], device=dev)
        s["resid"] = [torch.empty(int(s["shapes"][:, 0].sum()), device=dev),
                      torch.empty(dex.dex_workspace_bytes(d, dex.DEX_WS_RESID), dtype=torch.uint8,
                                  device=dev)]
        s["ws"] = ws(d, dex.DEX_WS_FWD)
        s["ct"] = torch.ones(case["B"], device=dev)
        s["grads"] = [torch.empty_like(t) for t in s["ins"][1:5]]
    elif kind == "gather":
        if case["mode"] == "grad":
            s["T"].requires_grad_()
            s["w"].requires_grad_()
        else:
            s["desc"] = dex.gather_desc(case["V"], case["R"], case["n"])
            s["out"] = torch.empty(case["n"], case["R"], device=dev)
    elif kind == "accum":
        flags = dex.DEX_DETERMINISTIC if case["deterministic"] else 0
        nb = dex.dex_accum_scatter_workspace_bytes(dex.DEX_F32, case["V"], case["R"], case["n"],
                                                   True, flags)
        s["flags"], s["ws"] = flags, dex.workspace(nb, dev) if nb else None
    elif kind == "stencil" and case["mode"] == "grad":
        s["fields"][0].requires_grad_()
    elif kind == "stencil":
        s["desc"] = dex.stencil_desc(case["H"], case["W"], case["steps"], case["every"],
                                     rho=case["rho"])
        s["ws"], s["dL"] = ws(s["desc"], dex.DEX_WS_JVP), torch.empty(1, device=dev)
    elif kind == "reduce":
        s["out"], s["total"] = torch.empty(case["rows"], device=dev), torch.empty(1, device=dev)
        s["ws"] = dex.workspace(dex.DEX_REDUCE_WS_BYTES, dev)
    return s


# ---- one pass ------------------------------------------------------------------

def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "gmm":
        if "params" in s:
            F = autograd.gmm_loglik(*s["params"], s["data"][4], VARIANT[c["variant"]])
            return [F, *torch.autograd.grad(F, s["params"])]
        dex.dex_fwd(s["desc"], s["data"], [s["F"]], s["resid"], s["ws_fwd"])
        if c["mode"] == "grad":
            dex.dex_vjp(s["desc"], s["data"], s["resid"], [s["ct"]], s["grads"], 0, s["ws_vjp"])
            return [s["F"], *s["grads"]]
        dex.dex_jvp(s["desc"], s["data"], s["tangents"], [s["dF"]], s["ws_jvp"], resid=s["resid"])
        return [s["F"], s["dF"]]
    if kind == "batched":
        dex.dex_fwd(s["desc"], s["ins"], [s["F"]], s["resid"], s["ws"])
        dex.dex_vjp(s["desc"], s["ins"], s["resid"], [s["ct"]], s["grads"], 0, s["ws"])
        return [s["F"], *s["grads"]]
    if kind == "gather":
        if c["mode"] == "grad":
            out = autograd.gather_scale(s["T"], s["idx"], s["w"])
            return [out, *torch.autograd.grad(out, (s["T"], s["w"]), s["g"])]
        dex.dex_jvp(s["desc"], [s["T"], s["idx"], s["w"]], [s["tT"], s["tw"]], [s["out"]])
        return [s["out"]]
    if kind == "accum":
        acc = s["T"].clone()  # a copy, so that every pass adds to the same values
        dex.dex_accum_scatter(acc, s["idx"], s["g"], s["w"], s["flags"], ws=s["ws"])
        return [acc]
    if kind == "hist":
        return [autograd.histogram(s["keys"], c["bins"])]
    if kind == "stencil":
        if c["mode"] == "grad":
            u0, target = s["fields"]
            v = dex.DEX_STENCIL_LINEAR if c["variant"] == "linear" else dex.DEX_STENCIL_RECOMPUTE
            L, uT = autograd.diffusion_loss(u0, target, c["steps"], c["every"], rho=c["rho"],
                                            variant=v)
            return [L, uT, *torch.autograd.grad(L, (u0,))]
        u0, target, du0, dtarget = s["fields"]
        dex.dex_jvp(s["desc"], [u0, target], [du0, dtarget], [s["dL"]], s["ws"])
        return [s["dL"]]
    dex.dex_reduce_rows(s["out"], s["values"])
    dex.dex_reduce_all(s["total"], s["values"], s["ws"])
    return [s["out"], s["total"]]


# ---- what a pass cannot do without -------------------------------------------------

def work(case):
    c = case
    kind = c["kind"]
    if kind in ("gmm", "batched"):
        shapes = [(c["N"], c["D"], c["K"])] if kind == "gmm" else _shapes(c).tolist()
        size = 8 if kind == "gmm" and c["dtype"] == "f64" else 4
        nbytes = flops = 0
        for N, D, K in shapes:
            params = K * (1 + 2 * D + D * (D - 1) // 2)
            flops += D * (D + 1) * N * K  # y = Q r, Q lower triangular
            if c.get("mode") == "jvp":
                flops += D * (D + 1) * N * K  # its tangent
                nbytes += size * (N * D + 2 * params)
            else:
                flops += D * (D + 3) * N * K  # symmetric second and first moments
                nbytes += size * (N * D + 2 * params)
        return dict(bytes=nbytes, flops=flops)
    if kind in ("gather", "accum"):
        V, R, n = c["V"], c["R"], c["n"]
        if kind == "accum":
            return dict(bytes=4 * (n * R + 2 * n + 2 * V * R), flops=2 * n * R)
        if c["mode"] == "jvp":
            return dict(bytes=4 * (n * R + 3 * n + 2 * V * R), flops=3 * n * R)
        return dict(bytes=4 * (2 * n * R + 3 * n + 2 * V * R), flops=5 * n * R)
    if kind == "hist":
        return dict(bytes=4 * (c["n"] + c["bins"]), flops=0)
    if kind == "stencil":
        cells = c["H"] * c["W"]
        if c["mode"] == "jvp":
            return dict(bytes=16 * cells, flops=12 * cells * c["steps"])
        passes = 3 if c["variant"] == "recompute" else 2  # forward, (recomputation,) adjoint
        return dict(bytes=16 * cells, flops=6 * cells * c["steps"] * passes)
    m = c["rows"] * c["cols"]
    return dict(bytes=4 * (2 * m + c["rows"]), flops=2 * m)


# ---- the same in 64 bits -------------------------------------------------------------

def _gmm_exact(alphas, means, qd, l, x, tangents=None):
    """F and its gradients (or F and its derivative along the tangents) for ct = 1, FP64."""
    N, D = x.shape
    K = alphas.shape[0]
    lower = torch.tril_indices(D, D, -1, device=x.device)  # row-major over the strict lower part

    def factor(k):
        Q = torch.diag(torch.exp(qd[k]))
        Q[lower[0], lower[1]] = l[k]
        return Q

    beta = torch.empty(K, N, dtype=torch.float64, device=x.device)
    for k in range(K):
        y = (x - means[k]) @ factor(k).T
        beta[k] = alphas[k] + qd[k].sum() - 0.5 * (y * y).sum(1)
    f = torch.logsumexp(beta, 0)
    F = f.sum() - N * torch.logsumexp(alphas, 0)
    soft = torch.softmax(alphas, 0)
    if tangents:
        da, dm, dq, dl = tangents
        dF = torch.zeros((), dtype=torch.float64, device=x.device)
        for k in range(K):
            Q, r = factor(k), x - means[k]
            dQ = torch.diag(torch.exp(qd[k]) * dq[k])
            dQ[lower[0], lower[1]] = dl[k]
            dy = r @ dQ.T - Q @ dm[k]
            dbeta = da[k] + dq[k].sum() - ((r @ Q.T) * dy).sum(1)
            dF += (torch.exp(beta[k] - f) * dbeta).sum()
        return [F, dF - N * (soft * da).sum()]
    ga, gm, gq, gl = (torch.empty_like(t) for t in (alphas, means, qd, l))
    for k in range(K):
        Q, r, w = factor(k), x - means[k], torch.exp(beta[k] - f)
        wy = w[:, None] * (r @ Q.T)
        A, M = w.sum(), wy.T @ r
        ga[k] = A - N * soft[k]
        gm[k] = Q.T @ wy.sum(0)
        gq[k] = A - torch.exp(qd[k]) * torch.diagonal(M)
        gl[k] = -M[lower[0], lower[1]]
    return [F, ga, gm, gq, gl]


def _scatter_exact(acc, idx, vals, w):
    """acc[idx[j]] += w[j] vals[j] in FP64: sums of runs of the sorted indices."""
    order = torch.argsort(idx)
    rows, counts = torch.unique_consecutive(idx[order], return_counts=True)
    ends = torch.cumsum(counts, 0) - 1
    for c0 in range(0, acc.shape[1], 32):
        v = (vals[order, c0:c0 + 32].double() * w[order].double()[:, None]).cumsum(0)[ends]
        acc[rows.long(), c0:c0 + 32] += torch.diff(v, dim=0, prepend=torch.zeros_like(v[:1]))
    return acc


def _stencil_exact(u0, target, steps, rho, du0=None, dtarget=None, c=0.2):
    def lin(u):
        return u + c * (torch.roll(u, -1, 0) + torch.roll(u, 1, 0) + torch.roll(u, -1, 1)
                        + torch.roll(u, 1, 1) - 4.0 * u)

    u, du, kept = u0, du0, []
    for _ in range(steps):
        if du is not None:
            du = lin(du) + rho * torch.cos(u) * du if rho else lin(du)
        elif rho:
            kept.append(u)
        u = lin(u) + rho * torch.sin(u) if rho else lin(u)
    if du is not None:
        return [((u - target) * (du - dtarget)).sum().reshape(1)]
    lam = u - target
    for _ in range(steps):
        lam = lin(lam) + rho * torch.cos(kept.pop()) * lam if rho else lin(lam)
    return [0.5 * ((u - target) ** 2).sum(), u, lam]


def exact(case, seed):
    c, kind = case, case["kind"]
    i = _inputs(c, seed)
    if kind == "gmm":
        got = _gmm_exact(*(t.double() for t in i["data"]), [t.double() for t in i["tangents"]])
        scalar = c["mode"] == "grad" and c["api"] == "autograd"
        return [got[0] if scalar else got[0].reshape(1),
                *(t.reshape(1) if t.dim() == 0 else t for t in got[1:])]
    if kind == "batched":
        outs, at = [[], [], [], [], []], [0] * 4
        for N, D, K in i["shapes"].tolist():
            part = []
            for q, (name, m) in enumerate((("alphas", K), ("means", K * D), ("l", K * D * (D - 1) // 2),
                                           ("x", N * D))):
                part.append((name, slice(at[q], at[q] + m)))
                at[q] += m
            p = dict(part)
            got = _gmm_exact(i["alphas"][p["alphas"]].double(),
                             i["means"][p["means"]].double().reshape(K, D),
                             i["qd"][p["means"]].double().reshape(K, D),
                             i["l"][p["l"]].double().reshape(K, -1),
                             i["x"][p["x"]].double().reshape(N, D))
            for o, t in zip(outs, got):
                o.append(t.reshape(-1))
        return [torch.cat(o) for o in outs]
    if kind == "gather":
        T, idx = i["T"].double(), i["idx"].long()
        if c["mode"] == "jvp":
            return [i["tw"].double()[:, None] * T[idx]
                    + i["w"].double()[:, None] * i["tT"].double()[idx]]
        rows = T[idx]
        dw = (rows * i["g"]).sum(1)
        out = rows.mul_(i["w"].double()[:, None])
        return [out, _scatter_exact(torch.zeros_like(T), i["idx"], i["g"], i["w"]), dw]
    if kind == "accum":
        return [_scatter_exact(i["T"].double(), i["idx"], i["g"], i["w"])]
    if kind == "hist":
        return None  # whole numbers
    if kind == "stencil":
        return _stencil_exact(i["fields"][0].double(), i["fields"][1].double(), c["steps"], c["rho"],
                              *(t.double() for t in i["fields"][2:]))
    v = i["values"].double()
    return [v.sum(1), v.sum().reshape(1)]
