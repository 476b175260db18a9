"""Workloads of the hyper-connection path for timing it and for comparing two builds of it.

A case is one call pattern of a user's program at one size:

  train      a training step of one layer: the two fused forward calls around the caller's layer
             function, then the fused backward (what bench.py times)
  forward    the two fused forward calls alone (prefill, evaluation)
  serve      the forward through the allocation-free entry point (decode loops)
  separable  forward and backward through the separable calls (a caller that keeps H and inserts
             its own code between post, pre and the coefficients)
  stack      two layers under torch.autograd around an elementwise layer function
  diag       the doubly-stochasticity diagnostics of a few Sinkhorn-Knopp layers

Inputs are i.i.d. Gaussian streams with W ~ N(0, 0.02^2), b ~ N(0, 0.1^2) and alpha = 1, the
distributions of the repository's workloads; all are drawn on the GPU from the case's seed.
"""
import itertools
import math
import random
from types import SimpleNamespace

import torch

import paper_2601_05732_amd as mhcl
from paper_2601_05732_amd import diag

EPS = 1e-6
SK_ITERS = 20
DIAG_ALPHA = 8.0   # residual-logit scale at which Sinkhorn-Knopp matrices miss column sum 1 visibly


def _case(name, kind, mode, n, C, T, io="bf16", K=0, L=1):
    return dict(name=name, kind=kind, mode=mode, n=n, C=C, T=T, io=io, K=K, L=L)


def listed():
    return [
        # the benchmark's training step: four wide streams, a large micro-batch
        _case("train_n4_c4096", "train", "lite", 4, 4096, 32768),
        # evaluation / prefill over a large batch
        _case("forward_n4_c2048", "forward", "lite", 4, 2048, 32768),
        # few narrow streams, very many tokens
        _case("train_n3_c1024", "train", "lite", 3, 1024, 65536),
        # the largest full permutation set (130 logits)
        _case("train_n5_c2560", "train", "lite", 5, 2560, 16384),
        # the Sinkhorn-Knopp variant at the paper's middle width, a few ragged sequences
        _case("train_sk_n4_c768", "train", "sk", 4, 768, 3001),
        # all-fp32 check size: launches and latency
        _case("train_f32_n4_c64", "train", "lite", 4, 64, 256, io="f32"),
        # fp32 training at the paper's middle width
        _case("train_f32_n4_c768", "train", "lite", 4, 768, 4096, io="f32"),
        # eight streams with a subset of the permutations
        _case("train_n8_c1024_k64", "train", "subset", 8, 1024, 16384, K=64),
        # a decode step of a small batch at the widest streams
        _case("serve_n4_c4096", "serve", "lite", 4, 4096, 16),
        # separable calls at the paper's largest width, an odd token count
        _case("separable_n4_c1024", "separable", "lite", 4, 1024, 5003),
        # two layers under autograd, two sequences of 1024 tokens
        _case("stack_n4_c1024", "stack", "lite", 4, 1024, 2048, L=2),
        # column sums, l1 errors and products of six Sinkhorn-Knopp layers
        _case("diag_sk_n4_c512", "diag", "sk", 4, 512, 8192, L=6),
    ]


# per kind: token range, and the most n * C * T * M (the work of one projection) a case may have
_LIMITS = {
    "train": (1, 65536, 2 ** 33),
    "forward": (1, 65536, 2 ** 33),
    "serve": (1, 64, 2 ** 31),
    "separable": (1, 16384, 2 ** 29),
    "stack": (1, 8192, 2 ** 28),
    "diag": (64, 16384, 2 ** 28),
}


def _logspread(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["train", "train", "train", "forward", "forward", "serve", "separable", "stack", "diag"])
    mode = "sk" if kind == "diag" else rng.choice(["lite", "lite", "lite", "sk", "subset"])
    n = rng.choice([2, 3, 4, 4, 4, 5])
    K = 0
    if mode == "subset":
        n = rng.choice([5, 6, 7, 8])
        K = rng.randint(2, 100)
    io = "f32" if kind in ("train", "forward", "separable") and rng.random() < 0.25 else "bf16"
    C = _logspread(rng, 64, 4096)
    C = max(64, C // 64 * 64) if rng.random() < 0.75 else max(8, C // 8 * 8)
    lo, hi, most = _LIMITS[kind]
    if io == "f32" or C % 64:
        most = min(most, 2 ** 28)
    M = _logits(dict(mode=mode, n=n, K=K))
    hi = max(lo, min(hi, most // (n * C * M)))
    return dict(kind=kind, mode=mode, n=n, C=C, T=_logspread(rng, lo, hi), io=io, K=K,
                L={"stack": 2, "diag": rng.randint(2, 6)}.get(kind, 1))


def _logits(case):
    n = case["n"]
    R = {"lite": math.factorial(n), "sk": n * n, "subset": case["K"]}[case["mode"]]
    return R + 2 * n


def _perms(case, seed):
    """Rows sigma_k of the case's permutations: all n! in lexicographic order, or K distinct ones."""
    n = case["n"]
    if case["mode"] == "lite":
        return list(itertools.permutations(range(n)))
    rng, rows = random.Random(seed), [tuple(range(n))]
    while len(rows) < case["K"]:
        p = list(range(n))
        rng.shuffle(p)
        if tuple(p) not in rows:
            rows.append(tuple(p))
    return rows


def _inputs(case, seed):
    """The tensors of a case on the GPU, one dict per layer (x, y and gradients in the first only)."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    io = torch.bfloat16 if case["io"] == "bf16" else torch.float32
    n, C, T, M = case["n"], case["C"], case["T"], _logits(case)

    def normal(*shape, std=1.0, dtype=torch.float32):
        out = torch.empty(shape, device="cuda", dtype=dtype)
        if dtype == torch.float32:
            return out.normal_(0.0, std, generator=gen)
        rows = max(1, 2 ** 26 // max(1, out[0].numel()))
        for r in range(0, shape[0], rows):
            part = torch.empty((min(rows, shape[0] - r),) + shape[1:], device="cuda")
            out[r:r + rows].copy_(part.normal_(0.0, std, generator=gen))
        return out

    layers = []
    for layer in range(case["L"]):
        d = dict(W=normal(n * C, M, std=0.02), b=normal(M, std=0.1), alpha=torch.ones(3, device="cuda"))
        if case["kind"] == "diag":
            d["alpha"][0] = DIAG_ALPHA
            d["x"] = normal(T, n, C, dtype=io)
        layers.append(d)
    d = layers[0]
    if case["kind"] == "stack":
        d["x0"], d["g_out"] = normal(T, C, dtype=io), normal(T, C, dtype=io)
    elif case["kind"] != "diag":
        d["x"], d["y"] = normal(T, n, C, dtype=io), normal(T, C, dtype=io)
        if case["kind"] in ("train", "separable"):
            d["g_xout"], d["g_h"] = normal(T, n, C, dtype=io), normal(T, C, dtype=io)
    return layers


def prepare(case, seed):
    layers = _inputs(case, seed)
    n, C, T = case["n"], case["C"], case["T"]
    perm = None
    if case["mode"] == "subset":
        perm = torch.tensor(_perms(case, seed), dtype=torch.int8, device="cuda")
    if case["kind"] == "stack":
        net = mhcl.HyperConnectionStack(n, C, [torch.nn.functional.silu] * case["L"], case["mode"],
                                        sk_iters=SK_ITERS, eps=EPS, perm=perm)
        with torch.no_grad():
            for layer, d in zip(net.layers, layers):
                layer.W.copy_(d["W"])
                layer.b.copy_(d["b"])
                layer.alpha.copy_(d["alpha"])
        x0 = layers[0]["x0"].requires_grad_()
        params = [p for layer in net.layers for p in (layer.W, layer.b, layer.alpha)]
        return dict(kind="stack", net=net, x0=x0, g_out=layers[0]["g_out"], wrt=[x0] + params)
    wl = SimpleNamespace(n=n, C=C, T=T, M=_logits(case), io=case["io"], res_mode=case["mode"],
                         sk_iters=SK_ITERS, eps=EPS)
    if case["kind"] == "diag":
        return dict(kind="diag", wl=wl, L=case["L"], layers=layers)
    inp = layers[0]
    inp["x"] = mhcl.place_stream(inp["x"], mhcl.layer.PHASE_X)
    if "g_xout" in inp:
        inp["g_xout"] = mhcl.place_stream(inp["g_xout"], mhcl.layer.PHASE_G_XOUT)
    return dict(kind=case["kind"], layer=mhcl.GpuLayer(mhcl.desc_for(wl, perm=perm), inp))


_FORWARD = ("H_res", "H_pre", "H_post", "h", "x_out")
_BACKWARD = ("g_x", "g_y", "g_W", "g_b", "g_alpha")


def run(state):
    kind = state["kind"]
    if kind == "stack":
        out = state["net"](state["x0"])
        grads = torch.autograd.grad(out, state["wrt"], state["g_out"])
        return dict(out=out, grads=list(grads))
    if kind == "diag":
        H, z, spread = diag.layer_stack(state["wl"], state["L"], state["layers"])
        return dict(H=H, z=z, spread=spread, **diag.chain(H))
    L = state["layer"]
    names = _FORWARD
    if kind == "train":
        L.step()
        names = _FORWARD + _BACKWARD
    elif kind == "separable":
        L.forward_separable()
        L.backward_separable()
        names = _FORWARD + _BACKWARD + ("g_H_res", "g_H_pre", "g_H_post")
    elif kind == "forward":
        L.forward_fused()
    else:
        i, d = L.inp, L.d
        mhcl.mhcl_fwd_coeffs_pre_static(d, i["x"], i["W"], i["b"], i["alpha"], L.H_res, L.H_pre,
                                        L.H_post, L.h)
        mhcl.mhcl_post(d, i["x"], i["y"], L.H_res, L.H_post, L.x_out)
    return {k: getattr(L, k) for k in names}


def work(case):
    n, C, T, M, L = case["n"], case["C"], case["T"], _logits(case), case["L"]
    e = 2 if case["io"] == "bf16" else 4
    U = C * e                                  # one [C] row of a stream
    coef = 4 * (n * n + 2 * n)                 # coefficients of one token
    par = 4 * (n * C * M + M + 3)              # parameters, or their gradients
    proj = 2 * n * C * M                       # one thin product per token
    fwd_bytes = T * ((3 * n + 2) * U + coef) + par
    fwd_flops = T * (proj + 2 * n * C + 2 * n * C + 2 * n * (n + 1) * C)
    bwd_bytes = T * (3 * n + 3) * U + par
    bwd_flops = T * (2 * proj + 2 * (n * n + 2 * n) * C + 2 * (n * n + 3 * n) * C)
    if case["kind"] in ("forward", "serve"):
        return dict(bytes=fwd_bytes, flops=fwd_flops)
    if case["kind"] == "train":
        return dict(bytes=fwd_bytes + bwd_bytes, flops=fwd_flops + bwd_flops)
    if case["kind"] == "separable":            # the gradients on H are outputs too
        return dict(bytes=fwd_bytes + bwd_bytes + T * coef, flops=fwd_flops + bwd_flops)
    if case["kind"] == "stack":                # per layer: forward, backward; x0, out and their gradients
        f_bytes = 4 * T * U                    # the layer function and its backward
        return dict(bytes=L * (fwd_bytes + bwd_bytes + f_bytes) + 4 * T * U, flops=L * (fwd_flops + bwd_flops))
    per = T * (n * U + 4 * M + 4 + 4 * n * n + 8 * (n + 1)) + par     # diag: x, z, spread, H, sums
    return dict(bytes=L * per + 4 * T * n * n, flops=L * T * (proj + 2 * n * C + 2 * n ** 3))


def tolerance(case):
    # two-norm and largest deviations seen against 64 bits, times about four
    if case["kind"] == "stack":                # two layers of bf16 roundings, summed into gradients
        return dict(rel=2e-2, max=1e-1)
    if case["kind"] == "diag":                 # fp32 after a projection with 16 bits of W, logits times eight
        return dict(rel=4e-5, max=1e-2)
    if case["io"] == "f32":
        return dict(rel=5e-6, max=1e-4)
    return dict(rel=8e-3, max=4e-2)            # one rounding of bf16 outputs


# ---- the same in 64 bits, plain torch ------------------------------------------------------


def _coeffs64(case, x, W, b, alpha, stack):
    """H_res, H_pre, H_post, z of x [t, n, C] in float64."""
    n = case["n"]
    flat = x.reshape(x.shape[0], -1)
    r = torch.rsqrt(flat.square().mean(dim=1, keepdim=True) + EPS)
    M = W.shape[1]
    R = M - 2 * n
    scale = torch.cat([alpha[0].expand(R), alpha[1].expand(n), alpha[2].expand(n)])
    z = scale * (r * (flat @ W)) + b
    if case["mode"] == "sk":
        H = torch.exp(z[:, :R] - z[:, :R].amax(dim=1, keepdim=True).detach()).reshape(-1, n, n)
        for _ in range(SK_ITERS):
            H = H / H.sum(dim=1, keepdim=True)
            H = H / H.sum(dim=2, keepdim=True)
    else:
        H = (torch.softmax(z[:, :R], dim=1) @ stack).reshape(-1, n, n)
    return H, torch.sigmoid(z[:, R:R + n]), 2 * torch.sigmoid(z[:, R + n:]), z


def _perm_stack(case, seed):
    """The permutation matrices as rows of a [K, n*n] matrix."""
    if case["mode"] == "sk":
        return None
    rows, n = _perms(case, seed), case["n"]
    P = torch.zeros(len(rows), n, n, dtype=torch.float64)
    for k, row in enumerate(rows):
        for i, j in enumerate(row):
            P[k, i, j] = 1.0
    return P.reshape(len(rows), n * n).cuda()


def _mix(H, x):
    return (H.unsqueeze(-1) * x.unsqueeze(1)).sum(dim=2)      # H [t, n, n], x [t, n, C]


def exact(case, seed):
    layers = _inputs(case, seed)
    stack = _perm_stack(case, seed)
    f64 = lambda t: t.to(torch.float64)  # noqa: E731
    if case["kind"] == "stack":
        return _exact_stack(case, layers, stack)
    if case["kind"] == "diag":
        return _exact_diag(case, layers, stack)
    d = layers[0]
    T = case["T"]
    backward = case["kind"] in ("train", "separable")
    W, b, alpha = (f64(d[k]).requires_grad_(backward) for k in ("W", "b", "alpha"))
    rows = max(1, 2 ** 23 // (case["n"] * case["C"]))
    pieces, sums = [], None
    for t0 in range(0, T, rows):
        x, y = (f64(d[k][t0:t0 + rows]).requires_grad_(backward) for k in ("x", "y"))
        H, Hp, Hq, _ = _coeffs64(case, x, W, b, alpha, stack)
        h = (Hp.unsqueeze(-1) * x).sum(dim=1)
        x_out = _mix(H, x) + Hq.unsqueeze(-1) * y.unsqueeze(1)
        out = dict(H_res=H, H_pre=Hp, H_post=Hq, h=h, x_out=x_out)
        if backward:
            gxo, gh = f64(d["g_xout"][t0:t0 + rows]), f64(d["g_h"][t0:t0 + rows])
            g = torch.autograd.grad([x_out, h], [x, y, H, Hp, Hq, W, b, alpha], [gxo, gh])
            out.update(g_x=g[0], g_y=g[1])
            if case["kind"] == "separable":
                out.update(g_H_res=g[2], g_H_pre=g[3], g_H_post=g[4])
            sums = list(g[5:]) if sums is None else [p + q for p, q in zip(sums, g[5:])]
        pieces.append({k: v.detach() for k, v in out.items()})
    result = {k: torch.cat([p[k] for p in pieces]) for k in pieces[0]}
    if backward:
        result.update(g_W=sums[0], g_b=sums[1], g_alpha=sums[2])
    return result


def _exact_stack(case, layers, stack):
    x0 = layers[0]["x0"].to(torch.float64).requires_grad_()
    wrt = [x0]
    x = x0.unsqueeze(1).expand(-1, case["n"], -1)
    for d in layers:
        W, b, alpha = (d[k].to(torch.float64).requires_grad_() for k in ("W", "b", "alpha"))
        wrt += [W, b, alpha]
        H, Hp, Hq, _ = _coeffs64(case, x, W, b, alpha, stack)
        y = torch.nn.functional.silu((Hp.unsqueeze(-1) * x).sum(dim=1))
        x = _mix(H, x) + Hq.unsqueeze(-1) * y.unsqueeze(1)
    out = x.sum(dim=1)
    grads = torch.autograd.grad(out, wrt, layers[0]["g_out"].to(torch.float64))
    return dict(out=out.detach(), grads=list(grads))


def _exact_diag(case, layers, stack):
    n = case["n"]
    Hs, zs, spreads = [], [], []
    for d in layers:
        H, _, _, z = _coeffs64(case, *(d[k].to(torch.float64) for k in ("x", "W", "b", "alpha")), stack)
        R = z.shape[1] - 2 * n
        Hs.append(H)
        zs.append(z)
        spreads.append(z[:, :R].amax(dim=1) - z[:, :R].amin(dim=1))
    Q, Qs = torch.eye(n, dtype=torch.float64, device="cuda").expand(case["T"], n, n), []
    for H in Hs:
        Q = H @ Q
        Qs.append(Q)
    H, Q = torch.stack(Hs), torch.stack(Qs)
    l1 = lambda A: (A.sum(dim=3) - 1).abs().sum(dim=2) + (A.sum(dim=2) - 1).abs().sum(dim=2)  # noqa: E731
    return dict(H=H, z=torch.stack(zs), spread=torch.stack(spreads), colsum=H.sum(dim=2), l1=l1(H),
                prod=Q[-1], prod_colsum=Q.sum(dim=2), prod_l1=l1(Q))
