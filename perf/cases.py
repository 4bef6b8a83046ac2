"""The calls whose speed is watched: 2-simplicial attention as a program uses it.

Each case is one call (or one training step) through the package's public entry
points, at sizes taken from the repository's workloads, benchmark and tests:

  listed()             the named cases
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  inputs and buffers a program holds before the call
  run(state)           one pass; returns every output
  work(case)           bytes and FLOPs the pass cannot do without
  tolerance(case)      how far another correct implementation may be off
  exact(case, seed)    the outputs in float64, plain torch

Fields of a case: `kind` ("fwd", "bwd", "train", "det", "layer"), sizes B, N, H,
Hkv (K-side heads; H unless grouped-query), D, windows w1, w2, `dtype`, `inputs`
(the workload transform of the inputs) and the K' / V' constants kpb, vpb.
"""

import math

import torch

from paper_2507_02754_amd import (SimplicialAttention, simplicial_attention, simplicial_attn_bwd,
                                  simplicial_attn_bwd_workspace_size, simplicial_attn_det_bwd,
                                  simplicial_attn_det_fwd, simplicial_attn_fwd, simplicial_attn_fwd_gqa)


def _case(name, kind, B, N, H, D, w1, w2, dtype="bf16", Hkv=0, inputs="none", kpb=0.0, vpb=0.0):
    c = dict(kind=kind, B=B, N=N, H=H, Hkv=Hkv or H, D=D, w1=w1, w2=w2, dtype=dtype, inputs=inputs,
             kpb=kpb, vpb=vpb)
    return dict(c, name=name) if name else c


def listed():
    return [
        # A short prompt through one attention call: both windows reach past
        # its start, so launch and latency count more than throughput.
        _case("fwd_short", "fwd", 1, 192, 8, 128, 512, 32),
        # A prompt of 4096 tokens (the forward-only workload).
        _case("fwd_4k", "fwd", 1, 4096, 8, 128, 512, 32),
        # The training step of a short, ragged sequence.
        _case("train_1k", "train", 1, 1021, 8, 128, 256, 32),
        # The training step of the 8k workload.
        _case("train_8k", "train", 2, 8192, 8, 128, 512, 32),
        # Long-context training, forward and backward separately: the shape
        # of the headline benchmark.
        _case("fwd_32k", "fwd", 1, 32768, 16, 128, 512, 32, inputs="l2norm_qk"),
        _case("bwd_32k", "bwd", 1, 32768, 16, 128, 512, 32, inputs="l2norm_qk"),
        # The wide windows of the second benchmark workload.
        _case("train_wide", "train", 1, 8192, 16, 128, 1024, 64, inputs="scale_half"),
        # Grouped-query attention: four query heads per K-side head.
        _case("train_gqa", "train", 1, 6001, 16, 128, 512, 32, Hkv=4),
        # Determinant (rotation-invariant) logits, forward and backward.
        _case("train_det", "det", 1, 4096, 16, 128, 512, 32),
        # The whole layer with its projections, head_dim 64, K' / V' constants.
        _case("layer_64", "layer", 2, 2048, 16, 64, 512, 24, kpb=0.25, vpb=0.5),
        # A training step in float32 (a layer with attn_dtype float32).
        _case("train_fp32", "train", 1, 2000, 4, 64, 256, 16, dtype="fp32"),
        # Square windows (128, 128), one of the paper's window pairs.
        _case("train_square", "train", 1, 1024, 4, 128, 128, 128),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


MOST_FLOPS = 1.3e13  # of a drawn case: the largest listed one's (bwd_32k)


def draw(rng):
    c = _drawn(rng)
    flops = work(c)["flops"]
    return dict(c, N=max(128, int(c["N"] * MOST_FLOPS / flops))) if flops > MOST_FLOPS else c


def _drawn(rng):
    # Kinds in about the shares of the listed cases; "plain": float32, short
    # head dims or w2 > 64.
    kind = rng.choice(["fwd", "fwd", "fwd", "bwd", "train", "train", "train", "gqa", "det", "layer", "plain", "plain"])
    D = rng.choice([64, 128, 128])
    B, H = rng.choice([1, 1, 2]), rng.choice([4, 8, 8, 16])
    N = _log(rng, 128, 16384)
    w1 = rng.choice([128, 256, 512, 512, 1024, rng.randint(100, 1000)])
    w2 = rng.choice([16, 32, 32, 32, rng.randint(5, 32), 64])
    inputs = rng.choice(["none", "l2norm_qk", "scale_half"])
    if kind == "gqa":
        return _case("", "train", B, N, H, D, w1, w2, Hkv=H // rng.choice([2, 4]), inputs=inputs)
    if kind == "det":
        return _case("", "det", 1, min(N, 8192), H, D, w1, min(w2, 32))
    if kind == "layer":
        return _case("", "layer", B, min(N, 4096), H, D, w1, w2, kpb=rng.choice([0.0, 0.25]), vpb=rng.choice([0.0, 0.5]))
    if kind == "plain":
        N = _log(rng, 128, 2048)
        if rng.random() < 0.5:
            return _case("", rng.choice(["fwd", "train"]), 1, N, 4, rng.choice([32, 64, 128]),
                         rng.choice([128, 256, rng.randint(20, 300)]), rng.choice([8, 16, 32]), dtype="fp32")
        D = rng.choice([32, 128])
        w2 = rng.choice([16, 32]) if D == 32 else rng.choice([96, 128])
        return _case("", rng.choice(["fwd", "train"]), 1, N, 4, D, rng.choice([128, rng.randint(100, 200)]), w2)
    return _case("", kind, B, N, H, D, w1, w2, inputs=inputs)


def _dtype(case):
    return torch.float32 if case["dtype"] == "fp32" else torch.bfloat16


def _inputs(case, seed):
    """q, k, kp, v, vp, do on the GPU: standard normals with the workload's transform."""
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    B, N, D = case["B"], case["N"], case["D"]

    def normal(heads):
        return torch.randn((B, N, heads, D), generator=g, device="cuda")

    q = normal(case["H"])
    k, kp, v, vp = (normal(case["Hkv"]) for _ in range(4))
    do = normal(case["H"])
    if case["inputs"] == "l2norm_qk":
        q = q / q.norm(dim=-1, keepdim=True) * D ** 0.5
        k = k / k.norm(dim=-1, keepdim=True) * D ** 0.5
    elif case["inputs"] == "scale_half":
        q, k, kp, v, vp = (x * 0.5 for x in (q, k, kp, v, vp))
    return [x.to(_dtype(case)).contiguous() for x in (q, k, kp, v, vp, do)]


def _layer_inputs(case, seed):
    """A layer of d_model = H * D with seeded weights, its input and upstream gradient."""
    H, D = case["H"], case["D"]
    dm = H * D
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    layer = SimplicialAttention(dm, H, D, case["w1"], case["w2"], kp_bias=case["kpb"], vp_bias=case["vpb"],
                                attn_dtype=_dtype(case), device="cuda", dtype=_dtype(case))
    with torch.no_grad():
        for p in layer.parameters():
            p.copy_(torch.randn(p.shape, generator=g, device="cuda") * dm ** -0.5)
    x, dy = (torch.randn((case["B"], case["N"], dm), generator=g, device="cuda").to(_dtype(case)) for _ in range(2))
    return layer, x, dy


def _scale(case):
    return case["D"] ** -0.5


def prepare(case, seed):
    if case["kind"] == "layer":
        layer, x, dy = _layer_inputs(case, seed)
        return dict(case, layer=layer, x=x.requires_grad_(True), dy=dy)
    t = _inputs(case, seed)
    state = dict(case, t=t)
    if case["kind"] == "train":
        state["leaves"] = [x.requires_grad_(True) for x in t[:5]]
    if case["kind"] == "fwd":
        state["out"] = torch.empty_like(t[0])
        state["lse"] = torch.empty((case["B"], case["H"], case["N"]), dtype=torch.float32, device="cuda")
    if case["kind"] == "bwd":
        w = (case["w1"], case["w2"])
        state["out"], state["lse"] = simplicial_attn_fwd(*t[:5], *w, _scale(case))
        state["grads"] = tuple(torch.empty_like(t[0]) for _ in range(5))
        need = simplicial_attn_bwd_workspace_size(case["B"], case["N"], case["H"], case["D"], *w, t[0].dtype)
        state["workspace"] = torch.empty(max(need, 16), dtype=torch.uint8, device="cuda")
    return state


def run(state):
    w1, w2, kind = state["w1"], state["w2"], state["kind"]
    scale = _scale(state)
    if kind == "layer":
        layer, x = state["layer"], state["x"]
        params = [layer.wq.weight, layer.wk.weight, layer.wkp.weight, layer.wv.weight, layer.wvp.weight, layer.wo.weight]
        y = layer(x)
        return [y, *torch.autograd.grad(y, [x, *params], state["dy"])]
    q, k, kp, v, vp, do = state["t"]
    if kind == "fwd":
        fwd = simplicial_attn_fwd if state["Hkv"] == state["H"] else simplicial_attn_fwd_gqa
        return list(fwd(q, k, kp, v, vp, w1, w2, scale, out=state["out"], lse=state["lse"]))
    if kind == "bwd":
        return list(simplicial_attn_bwd(q, k, kp, v, vp, state["out"], do, state["lse"], w1, w2, scale,
                                        grads=state["grads"], workspace=state["workspace"]))
    if kind == "det":
        out, lse = simplicial_attn_det_fwd(q, k, kp, v, vp, w1, w2, scale)
        return [out, lse, *simplicial_attn_det_bwd(q, k, kp, v, vp, out, do, lse, w1, w2, scale)]
    o = simplicial_attention(*state["leaves"], w1, w2, scale, state["kpb"], state["vpb"])
    return [o, *torch.autograd.grad(o, state["leaves"], do)]


def _pairs(case):
    """(j, k) pairs over all queries of one head, clipped at the start of the sequence."""
    N, w1, w2 = case["N"], min(case["w1"], case["N"]), min(case["w2"], case["N"])
    lo = max(w1, w2)
    return sum(min(w1, i + 1) * min(w2, i + 1) for i in range(lo)) + (N - lo) * w1 * w2


def work(case):
    B, N, H, Hkv, D = (case[x] for x in ("B", "N", "H", "Hkv", "D"))
    el = 4 if case["dtype"] == "fp32" else 2
    qs, ks, stat = B * N * H * D * el, B * N * Hkv * D * el, 4 * B * H * N
    unit = B * H * _pairs(case) * D
    # forward: S and P V; backward: S again, dP, dV, dK and the query side's two
    if case["kind"] == "fwd":
        return {"bytes": 2 * qs + 4 * ks + stat, "flops": 4 * unit}
    if case["kind"] == "bwd":
        return {"bytes": 4 * qs + 8 * ks + stat, "flops": 12 * unit}
    if case["kind"] == "layer":
        rows, dm = B * N, H * D
        return {"bytes": 4 * rows * dm * el + 12 * dm * dm * el, "flops": 16 * unit + 18 * 2 * rows * dm * dm}
    return {"bytes": 4 * qs + 8 * ks + (stat if case["kind"] == "det" else 0), "flops": 16 * unit}


def tolerance(case):
    # Against float64 the forward is 2e-3 .. 3e-3 off in bf16 (operands,
    # probabilities and result rounded to 8 bits) and the gradients 3e-3 ..
    # 1.1e-2; about four times that. float32: 32-bit sums.
    if case["dtype"] == "fp32":
        return {"rel": 1e-5, "max": 1e-3}
    if case["kind"] == "fwd":
        return {"rel": 1e-2, "max": 0.4}
    return {"rel": 0.03, "max": 0.9}


# ---- float64 reference ----


def _cross(a, b):
    """Chunkwise a x b over whole 3-component chunks, trailing components 0."""
    n = a.shape[-1] // 3 * 3
    c = torch.linalg.cross(a[..., :n].unflatten(-1, (-1, 3)), b[..., :n].unflatten(-1, (-1, 3))).flatten(-2)
    return torch.nn.functional.pad(c, (0, a.shape[-1] - n))


def _head_exact(q, k, kp, v, vp, do, w1, w2, scale, det):
    """One head in float64: o, lse and (with do) dq, dk, dkp, dv, dvp, over blocks of queries."""
    N, D = q.shape
    w1, w2 = min(w1, N), min(w2, N)
    QB = 32
    o, lse = torch.zeros_like(q), torch.zeros(N, dtype=q.dtype, device=q.device)
    grads = [torch.zeros_like(q) for _ in range(5)] if do is not None else None
    mul = _cross if det else torch.mul
    dev = q.device
    per = max(1, int(4e7 // (QB * w2 * (QB + w1))))  # blocks of queries at a time
    for i0 in range(0, N, QB * per):
        nblk = min(per, -(-(N - i0) // QB))
        i = i0 + torch.arange(nblk * QB, device=dev).view(nblk, QB)  # queries
        kk = i[:, :, None] - w2 + 1 + torch.arange(w2, device=dev)  # k of the rows
        j = i[:, :1] - w1 + 1 + torch.arange(QB + w1 - 1, device=dev)  # keys of the block
        ic, kc, jc = i.clamp(max=N - 1), kk.clamp(0, N - 1), j.clamp(0, N - 1)
        jok = (j[:, None] >= 0) & (j[:, None] <= i[:, :, None]) & (j[:, None] > i[:, :, None] - w1)
        ok = ((kk >= 0) & (i < N)[..., None])[..., None] & jok[:, :, None]
        qr, kpr = q[ic][:, :, None], kp[kc]
        qt = mul(kpr, qr.expand_as(kpr)).flatten(1, 2)  # rows (query, k)
        kj, vj = k[jc], v[jc]
        s = torch.bmm(qt, kj.transpose(1, 2).contiguous()).view(nblk, QB, w2, -1) * scale
        s = s.masked_fill(~ok, -math.inf)
        ls = torch.logsumexp(s.flatten(2), 2)
        valid = i < N
        ls = torch.where(valid, ls, torch.zeros_like(ls))
        p = torch.exp(s - ls[..., None, None])
        vpr = vp[kc]
        u = torch.bmm(p.flatten(1, 2), vj).view(nblk, QB, w2, D)
        oi = (u * vpr).sum(2)
        iv = i[valid]
        o[iv], lse[iv] = oi[valid], ls[valid]
        if do is None:
            continue
        dor = do[ic][:, :, None]
        dt = (dor * vpr).flatten(1, 2)
        dp = torch.bmm(dt, vj.transpose(1, 2).contiguous()).view_as(s)
        delta = (do[ic] * oi).sum(-1)
        ds = p * (dp - delta[..., None, None]) * scale
        pt, dst = (x.flatten(1, 2).transpose(1, 2).contiguous() for x in (p, ds))
        grads[1].index_add_(0, jc.flatten(), torch.bmm(dst, qt).flatten(0, 1))
        grads[3].index_add_(0, jc.flatten(), torch.bmm(pt, dt).flatten(0, 1))
        dqt = torch.bmm(ds.flatten(1, 2), kj).view(nblk, QB, w2, D)
        if det:  # <dq~, k' x q>
            dqi, dkr = mul(dqt, kpr), mul(qr.expand_as(dqt), dqt)
        else:
            dqi, dkr = dqt * kpr, dqt * qr
        grads[0].index_add_(0, ic.flatten(), dqi.sum(2).flatten(0, 1))
        grads[2].index_add_(0, kc.flatten(), dkr.flatten(0, 2))
        grads[4].index_add_(0, kc.flatten(), (u * dor).flatten(0, 2))
    return o, lse, grads


def _attention_exact(t, case, backward, det=False):
    """[o, lse, dq, dk, dkp, dv, dvp] in float64 of inputs [B, N, heads, D]."""
    q, k, kp, v, vp, do = (None if x is None else x.detach().double() for x in t)
    kp, vp = kp + case["kpb"], vp + case["vpb"]
    B, N, H, D = q.shape
    rep = H // k.shape[2]
    o = torch.zeros_like(q)
    lse = torch.zeros((B, H, N), dtype=q.dtype, device=q.device)
    grads = [torch.zeros_like(x) for x in (q, k, kp, v, vp)]
    for b in range(B):
        for h in range(H):
            g = h // rep
            rows = [x.contiguous() for x in (q[b, :, h], k[b, :, g], kp[b, :, g], v[b, :, g], vp[b, :, g])]
            d = do[b, :, h].contiguous() if backward else None
            o[b, :, h], lse[b, h], gr = _head_exact(*rows, d, case["w1"], case["w2"], _scale(case), det)
            if backward:
                grads[0][b, :, h] = gr[0]
                for x, y in zip(grads[1:], gr[1:]):
                    x[b, :, g] += y
    return [o, lse, *grads]


class _ExactAttention(torch.autograd.Function):
    @staticmethod
    def forward(ctx, q, k, kp, v, vp, case):
        ctx.save_for_backward(q, k, kp, v, vp)
        ctx.case = case
        return _attention_exact([q, k, kp, v, vp, None], case, False)[0]

    @staticmethod
    def backward(ctx, do):
        return (*_attention_exact([*ctx.saved_tensors, do], ctx.case, True)[2:], None)


def exact(case, seed):
    if case["kind"] == "layer":
        layer, x, dy = _layer_inputs(case, seed)
        ws = [getattr(layer, n).weight.detach().double().requires_grad_(True) for n in ("wq", "wk", "wkp", "wv", "wvp", "wo")]
        x = x.double().requires_grad_(True)
        B, N, H, D = (case[n] for n in ("B", "N", "H", "D"))
        qkv = [(x @ w.t()).view(B, N, H, D) for w in ws[:5]]
        o = _ExactAttention.apply(*qkv, case)
        y = o.reshape(B, N, H * D) @ ws[5].t()
        return [y.detach(), *torch.autograd.grad(y, [x, *ws], dy.double())]
    t = _inputs(case, seed)
    full = _attention_exact(t, case, case["kind"] != "fwd", case["kind"] == "det")
    if case["kind"] == "fwd":
        return full[:2]
    if case["kind"] == "bwd":
        return full[2:]
    if case["kind"] == "det":
        return full
    return [full[0], *full[2:]]
