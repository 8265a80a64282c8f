"""The calls whose speed and results this repository keeps track of.

k-MIP attention as its users call it: inference and training steps over one
graph or a block-diagonal batch, through the public entry points of
``paper_2604_03815_amd`` (``fwd``, ``fwd_noalloc``, ``bwd`` and the layer).
Inputs follow the recipes of ``workloads.py``, drawn on the GPU:

  normal   Q, K, V i.i.d. N(0, 1)
  fourier  random Fourier features of 2-D positions plus N(0, 0.1^2) noise,
           randomly projected (city road networks)
  cloud    random projection of xyz uniform in the unit cube plus
           N(0, 0.05^2) noise, randomly projected again (point clouds)
  mixture  Q and K from a Gaussian mixture of 64 centres, sigma 0.1 (many
           near-tied scores)

A case is a dict:
  kind     infer (forward), serve (forward without allocation), train
           (forward and backward), layer (a training step of the layer);
  data     the recipe above;
  graphs   0 for one graph of ``lo`` nodes (no graph_offsets), else the number
           of graphs, their sizes uniform in [lo, hi];
  heads, d, dv (value width), k, drop (attention dropout rate).
"""
import math
import random

import torch

import paper_2604_03815_amd as kmip

DEVICE = "cuda:0"


def _case(name, kind, data, graphs, lo, hi, heads, d, dv, k, drop=0.0):
    c = dict(kind=kind, data=data, graphs=graphs, lo=lo, hi=hi, heads=heads, d=d, dv=dv, k=k, drop=drop)
    return dict(c, name=name) if name else c


def listed():
    return [
        # One superpixel-sized graph at inference: latency and launches count.
        _case("infer_graph_311", "infer", "normal", 0, 311, 311, 3, 32, 32, 16),
        # The smallest benchmark configuration, served without allocation.
        _case("serve_2048", "serve", "normal", 0, 2048, 2048, 1, 32, 32, 16),
        # A training batch of superpixel graphs (the second benchmark configuration).
        _case("train_128_graphs", "train", "normal", 128, 100, 450, 3, 32, 32, 16),
        # The layer's training step on such a batch: wider values, attention dropout.
        _case("layer_64_graphs", "layer", "normal", 64, 100, 450, 3, 32, 64, 16, 0.2),
        # A training batch of point clouds, a few thousand points each.
        _case("train_16_clouds", "train", "cloud", 16, 1024, 4096, 4, 32, 32, 32),
        # The efficiency study's inputs at N = 10^4 (odd size), one head, k = 10.
        _case("train_normal_10007", "train", "normal", 0, 10007, 10007, 1, 16, 16, 10),
        # A city road network (the third benchmark configuration).
        _case("train_city_100k", "train", "fourier", 0, 100000, 100000, 4, 32, 32, 32),
        # Wide heads.
        _case("train_city_20k_d128", "train", "fourier", 0, 20011, 20011, 4, 128, 128, 32),
        # A large k (the start of a k schedule).
        _case("train_city_30k_k256", "train", "fourier", 0, 30000, 30000, 4, 32, 32, 256),
        # The headline configuration: a point cloud of 500k nodes.
        _case("train_cloud_500k", "train", "cloud", 0, 500000, 500000, 4, 16, 16, 32),
        # Clustered keys with many near ties, k = 128 (the fifth configuration).
        _case("train_mixture_262k", "train", "mixture", 0, 262144, 262144, 1, 64, 64, 128),
        # The efficiency study's inputs at N = 10^6, inference.
        _case("infer_normal_1m", "infer", "normal", 0, 1000000, 1000000, 1, 16, 16, 10),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.randrange(10)
    if kind == 0:
        n = _log_int(rng, 64, 8000)
        d = rng.choice((16, 32, 64))
        return _case("", rng.choice(("infer", "serve")), "normal", 0, n, n, rng.randint(1, 4), d, d,
                     rng.choice((8, 10, 16, 32)))
    if kind == 1:
        lo = rng.randint(10, 150)
        d = rng.choice((16, 32, 64))
        return _case("", rng.choice(("infer", "train")), "normal", _log_int(rng, 4, 128), lo, lo + rng.randint(50, 330),
                     rng.randint(1, 4), d, d, rng.choice((8, 16, 20, 32)))
    if kind == 2:
        lo = rng.randint(10, 150)
        return _case("", "layer", "normal", _log_int(rng, 4, 96), lo, lo + rng.randint(50, 330), rng.randint(1, 4),
                     rng.choice((16, 32)), rng.choice((16, 32, 64)), rng.choice((8, 16, 20)), rng.choice((0.0, 0.1, 0.3)))
    if kind == 3:
        lo = _log_int(rng, 500, 2000)
        d = rng.choice((16, 32, 64))
        return _case("", rng.choice(("infer", "train")), "cloud", rng.randint(2, 16), lo, 2 * lo + rng.randint(0, 96),
                     rng.randint(1, 4), d, d, rng.choice((10, 16, 32)))
    if kind == 4:
        n = _log_int(rng, 8200, 30000)
        d = rng.choice((16, 32))
        return _case("", "train", "normal", 0, n, n, rng.randint(1, 3), d, d, rng.choice((10, 16, 32)))
    if kind == 5:
        n = _log_int(rng, 3000, 100000)
        d = rng.choice((16, 32, 64))
        return _case("", rng.choice(("infer", "train")), "fourier", 0, n, n, rng.randint(1, 4), d, d, rng.choice((16, 24, 32)))
    if kind == 6:
        n = _log_int(rng, 2000, 20000)
        return _case("", rng.choice(("infer", "train")), "fourier", 0, n, n, rng.randint(1, 4), 128, 128,
                     rng.choice((10, 16, 32, 64)))
    if kind == 7:
        n = _log_int(rng, 2000, 24000)
        return _case("", "train", "fourier", 0, n, n, rng.randint(1, 4), 32, 32, rng.randint(129, 300))
    if kind == 8:
        n = _log_int(rng, 9000, 500000)
        return _case("", "train", "cloud", 0, n, n, rng.randint(1, 4), 16, 16, rng.choice((16, 32)))
    n = _log_int(rng, 9000, 260000)
    return _case("", "train", "mixture", 0, n, n, 1, 64, 64, rng.randint(33, 128))


# ---- inputs ----


def _sizes(case):
    """Graph sizes: the case's own, the same for every seed."""
    if not case["graphs"]:
        return [case["lo"]]
    rng = random.Random("%(graphs)d graphs of %(lo)d to %(hi)d" % case)
    return [rng.randint(case["lo"], case["hi"]) for _ in range(case["graphs"])]


def _offsets(sizes):
    o = [0]
    for s in sizes:
        o.append(o[-1] + s)
    return o


def _qkv(data, N, H, d, dv, gen):
    """Q, K [N, H, d] and V [N, H, dv] in bf16, by the named recipe."""

    def normal(*shape, std=1.0):
        return torch.randn(*shape, generator=gen, device=DEVICE) * std

    if data == "normal":
        q, k, v = normal(N, H * d), normal(N, H * d), normal(N, H * dv)
    elif data == "mixture":
        mu = normal(64, H * d)
        q, k = (mu[torch.randint(64, (N,), generator=gen, device=DEVICE)] + normal(N, H * d, std=0.1) for _ in range(2))
        v = normal(N, H * dv)
    else:
        if data == "fourier":
            pos = torch.rand(N, 2, generator=gen, device=DEVICE)
            ang = 2 * math.pi * (pos @ normal(2, 16, std=8.0) + torch.rand(16, generator=gen, device=DEVICE))
            x = torch.cat([ang.cos(), ang.sin()], 1) + normal(N, 32, std=0.1)
        else:
            x = torch.rand(N, 3, generator=gen, device=DEVICE) @ normal(3, 64) + normal(N, 64, std=0.05)
        f = x.shape[1]
        q, k, v = (x @ normal(f, H * w, std=f ** -0.5) for w in (d, d, dv))
    return tuple(t.to(torch.bfloat16).view(N, H, -1).contiguous() for t in (q, k, v))


def _inputs(case, seed):
    """Everything drawn for a case: offsets, then tensors in a fixed order."""
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    sizes = _sizes(case)
    offsets = _offsets(sizes) if case["graphs"] else None
    N, H, d, dv, k = sum(sizes), case["heads"], case["d"], case["dv"], case["k"]
    s = {"case": case, "offsets": offsets, "scale": 1.0 / math.sqrt(d)}
    if case["kind"] == "layer":
        layer = kmip.KMIPAttention(32 * H, H, d, dv, k, attn_dropout=case["drop"], device=DEVICE, generator=gen)
        s["layer"] = layer.train()
        s["x"] = torch.randn(N, 32 * H, generator=gen, device=DEVICE).requires_grad_()
        s["grad"] = torch.randn(N, 32 * H, generator=gen, device=DEVICE)
        s["keep"] = None
        if case["drop"] > 0:
            s["keep"] = (torch.rand(N, H, k, generator=gen, device=DEVICE) >= case["drop"]).to(torch.uint8)
        return s
    s["q"], s["k"], s["v"] = _qkv(case["data"], N, H, d, dv, gen)
    if case["kind"] == "train":
        s["dout"] = torch.randn(N, H, dv, generator=gen, device=DEVICE).to(torch.bfloat16)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    if case["kind"] == "serve":
        N, H, _ = s["q"].shape
        s["out"] = torch.empty(N, H, case["dv"], device=DEVICE)
        s["idx"] = torch.empty(N, H, case["k"], dtype=torch.int32, device=DEVICE)
        s["lse"] = torch.empty(N, H, device=DEVICE)
    elif case["kind"] != "layer":
        s["ws"], s["bws"] = kmip.Workspace(), kmip.Workspace()
    return s


def run(state):
    case = state["case"]
    if case["kind"] == "layer":
        layer, x = state["layer"], state["x"]
        out = layer(x, state["offsets"], keep=state["keep"])
        leaves = (x, layer.w_q, layer.w_k, layer.w_v, layer.w_o)
        gx, gq, gk, gv, go = torch.autograd.grad(out, leaves, state["grad"])
        return {"out": out.detach(), "dx": gx, "dw_q": gq, "dw_k": gk, "dw_v": gv, "dw_o": go}
    q, k, v = state["q"], state["k"], state["v"]
    if case["kind"] == "serve":
        kmip.fwd_noalloc(q, k, v, case["k"], state["scale"], state["out"], state["idx"], state["lse"])
        return {"out": state["out"], "idx": state["idx"], "lse": state["lse"]}
    out, idx, lse = kmip.fwd(q, k, v, case["k"], state["scale"], graph_offsets=state["offsets"], workspace=state["ws"])
    got = {"out": out, "idx": idx, "lse": lse}
    if case["kind"] == "train":
        got["dq"], got["dk"], got["dv"] = kmip.bwd(q, k, v, state["dout"], idx, lse, state["scale"],
                                                   workspace=state["bws"])
    return got


# ---- what a pass cannot do without, and how far it may be off ----


def work(case):
    """Inputs read once, outputs written once; every score of each graph and
    the products over the k kept keys of each query.  (Where the library's
    bounds rule key blocks out exactly, a pass computes fewer scores.)"""
    sizes = _sizes(case)
    N, H, d, dv, k = sum(sizes), case["heads"], case["d"], case["dv"], case["k"]
    rows, pairs = N * H, H * sum(n * min(k, n) for n in sizes)
    flops = 2 * H * d * sum(n * n for n in sizes) + 2 * pairs * dv
    if case["kind"] == "layer":
        m = 32 * H
        weights = m * H * (2 * d + 2 * dv) * 4
        nbytes = 4 * N * m * 4 + 2 * weights + (rows * k if case["drop"] > 0 else 0)
        flops += 3 * 2 * N * m * H * (2 * d + 2 * dv)
    else:
        nbytes = rows * (2 * (2 * d + dv) + 4 * dv + 4 * k + 4)
        if case["kind"] == "train":
            nbytes += rows * (2 * dv + 4 * (2 * d + dv))
    if case["kind"] in ("train", "layer"):
        flops += 2 * pairs * (2 * dv + 2 * d)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Selection compares float32 scores of bf16 rows: another order of their
    sums swaps keys whose scores agree to about 2^-22, and a swapped key brings
    its own value row.  Scores crowd most in the mixture and least among normal
    rows, where most inputs show no swap at all (errors of 3e-7 then).
    Against 64 bits: 7.6e-4 (normal), 3.3e-3 (fourier, cloud, 7e-5 of the
    indices), 3.5e-3 (mixture, 8e-4 of the indices) and 4.6e-3 (the layer,
    which rounds to bf16 in between); about four times that is allowed."""
    if case["kind"] == "layer":
        return {"rel": 1.8e-2, "max": 0.9}
    if case["data"] == "normal":
        return {"rel": 3e-3, "max": 0.9, "differ": 2e-4}
    if case["data"] == "mixture":
        return {"rel": 1.4e-2, "max": 0.9, "differ": 3e-3}
    return {"rel": 1.2e-2, "max": 0.9, "differ": 3e-4}


# ---- the same in 64 bits ----


def _top(s, k):
    """Columns of the k largest entries of each row of s."""
    rows, n = s.shape
    if n < 16384:
        return s.topk(k, dim=1).indices
    # the k largest entries lie in the k blocks of largest maxima
    w = 256
    whole = n // w * w
    best = s[:, :whole].view(rows, -1, w).amax(2).topk(min(k, whole // w), dim=1).indices
    cols = (best[:, :, None] * w + torch.arange(w, device=s.device)).view(rows, -1)
    cols = torch.cat([cols, torch.arange(whole, n, device=s.device).expand(rows, -1)], 1)
    return cols.gather(1, s.gather(1, cols).topk(k, dim=1).indices)


def _attend64(q, k, v, kk, scale, offsets, dout=None, keep=None, rate=0.0):
    """out, lse and, with dout, dq, dk, dv of Eq. 1, all tensors float64."""
    N, H, d = q.shape
    out, lse = torch.empty_like(v), torch.empty(N, H, dtype=q.dtype, device=q.device)
    dq, dk, dv = torch.empty_like(q), torch.zeros_like(k), torch.zeros_like(v)
    bounds = list(zip(offsets, offsets[1:])) if offsets else [(0, N)]
    for h in range(H):
        for a, b in bounds:
            kg, vg, kT = k[a:b, h].contiguous(), v[a:b, h].contiguous(), k[a:b, h].t().contiguous()
            m = min(kk, b - a)
            step = max(32, min(b - a, (1 << 28) // max(1, b - a)))
            for i in range(a, b, step):
                e = min(b, i + step)
                qc = q[i:e, h].contiguous()
                s = qc @ kT
                top = _top(s, m)
                st = s.gather(1, top) * scale
                del s
                lse[i:e, h] = torch.logsumexp(st, 1)
                p = torch.softmax(st, 1)
                f = 1.0
                if keep is not None:
                    # the draws belong to slots in order of decreasing score
                    f = keep[i:e, h, :m].double() / (1.0 - rate)
                part = max(1, (1 << 27) // (m * max(d, v.shape[2])))
                for j in range(0, e - i, part):
                    t = top[j:j + part]
                    pj = p[j:j + part]
                    fj = f if keep is None else f[j:j + part]
                    vt, kt = vg[t], kg[t]
                    out[i + j:i + j + len(t), h] = ((pj * fj)[:, :, None] * vt).sum(1)
                    if dout is None:
                        continue
                    do = dout[i + j:i + j + len(t), h]
                    dp = (vt * do[:, None, :]).sum(2) * fj
                    g = pj * (dp - (pj * dp).sum(1, keepdim=True)) * scale
                    dq[i + j:i + j + len(t), h] = (g[:, :, None] * kt).sum(1)
                    rows = (t + a).reshape(-1)
                    dk[:, h].index_add_(0, rows, (g[:, :, None] * qc[j:j + len(t)][:, None, :]).reshape(len(rows), -1))
                    dv[:, h].index_add_(0, rows, ((pj * fj)[:, :, None] * do[:, None, :]).reshape(len(rows), -1))
    return out, lse, dq, dk, dv


def exact(case, seed):
    s = _inputs(case, seed)
    if case["kind"] == "layer":
        layer, x, H = s["layer"], s["x"].detach().double(), case["heads"]
        w = [p.detach().double() for p in (layer.w_q, layer.w_k, layer.w_v, layer.w_o)]
        # the layer hands its projections, and the gradients it gets back, on in bf16
        q, k, v = ((x @ t).to(torch.bfloat16).double().view(len(x), H, -1) for t in w[:3])
        grad = s["grad"].double()
        dout = (grad @ w[3].t()).to(torch.bfloat16).double().view(len(x), H, -1)
        o, _, dq, dk, dv = _attend64(q, k, v, case["k"], s["scale"], s["offsets"], dout, s["keep"], case["drop"])
        o = o.reshape(len(x), -1)
        dq, dk, dv = (t.to(torch.bfloat16).double().reshape(len(x), -1) for t in (dq, dk, dv))
        return {"out": o @ w[3], "dx": dq @ w[0].t() + dk @ w[1].t() + dv @ w[2].t(), "dw_q": x.t() @ dq,
                "dw_k": x.t() @ dk, "dw_v": x.t() @ dv, "dw_o": o.t() @ grad}
    q, k, v = (s[n].double() for n in ("q", "k", "v"))
    dout = s["dout"].double() if case["kind"] == "train" else None
    out, lse, dq, dk, dv = _attend64(q, k, v, case["k"], s["scale"], s["offsets"], dout)
    got = {"out": out, "idx": None, "lse": lse}
    if dout is not None:
        got.update(dq=dq, dk=dk, dv=dv)
    return got
