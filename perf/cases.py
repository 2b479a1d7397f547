"""The calls whose speed this repository answers for, as a program makes them.

A reference-cached request is one prefill per layer and 40 denoising steps per
layer; around the attention a layer projects.  The cases go from one tiny
request, where launches and host work are all there is, over 512-pixel images
to the five-reference workload of 1024-pixel images (about 4096 tokens each),
in both cache formats, both head sizes, with whole and ragged segments, one
and two batch entries, and one GPU's share of the heads.

A case names a layout by its segment lengths: st static text anchors, lt live
text tokens, x target tokens, refs the reference lengths (comma separated).
Q, K and V are N(0, std) in bf16, as normalised queries and keys are.
"""
import math

import torch

import paper_2608_21229_amd as rc

DEV = "cuda"


def listed():
    return [
        # one whole request of a toy model (one prefill, one step): launch latency and host work
        dict(name="request_tiny", op="request", mask="perref", st=8, lt=16, x=64, refs="64", B=1, H=2, D=64),
        # one denoising step of a 512-pixel edit with two references: less than one round of query tiles
        dict(name="step_512px", op="step", mask="perref", st=64, lt=512, x=1024, refs="1024,1024", B=1, H=24, D=128),
        # a step at an odd aspect ratio and prompt length, paper mask, 64-wide heads, Q/K/V as views of one
        # fused projection, log-sum-exp wanted
        dict(name="step_ragged_d64", op="step", mask="paper", st=37, lt=203, x=3577, refs="3600,2304,1519", B=1, H=40,
             D=64, fused=True, lse=True),
        # the headline: a step of a 1024-pixel edit with five references
        dict(name="step_5ref", op="step", mask="perref", st=64, lt=512, x=4096, refs="4096,4096,4096,4096,4096", B=1,
             H=24, D=128),
        # the same step on one GPU of eight (3 of the 24 heads), by the entry that allocates nothing
        dict(name="step_5ref_share", op="step_noalloc", mask="perref", st=64, lt=512, x=4096,
             refs="4096,4096,4096,4096,4096", B=1, H=3, D=128),
        # both guidance branches in one call, over references of two resolutions
        dict(name="step_guided_mixed", op="step", mask="perref", st=64, lt=512, x=4096,
             refs="4096,4096,4096,1024,1024,1024", B=2, H=24, D=128),
        # the headline step over the 8-bit cache
        dict(name="step_5ref_fp8", op="step_fp8", mask="perref", st=64, lt=512, x=4096,
             refs="4096,4096,4096,4096,4096", B=1, H=24, D=128),
        # once per request and layer: the headline's reference prefill with its cache store
        dict(name="prefill_5ref", op="prefill", mask="perref", st=64, lt=512, x=4096,
             refs="4096,4096,4096,4096,4096", B=1, H=24, D=128),
        # the same into the 8-bit cache, references of two resolutions
        dict(name="prefill_mixed_fp8", op="prefill_fp8", mask="perref", st=64, lt=512, x=4096,
             refs="4096,4096,4096,1024,1024,1024", B=1, H=24, D=128),
        # the recompute that the cache replaces: dense attention over every row of the headline's sequence
        dict(name="full_5ref", op="full", mask="dense", st=0, lt=512, x=4096, refs="4096,4096,4096,4096,4096", B=1,
             H=24, D=128),
        # the fused QKV projection of the live rows of a 1024-pixel edit
        dict(name="linear_qkv", op="linear", m=4608, n=9216, k=3072, residual=False),
        # a stack of four layers, one step of a 512-pixel edit with one reference (projections, attention,
        # projections with residual): what a program calls once per denoising step
        dict(name="chain_step_512px", op="chain_step", mask="perref", st=64, lt=512, x=1024, refs="1024", B=1, H=24,
             D=128, layers=4),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _image(rng):
    """Tokens of one image: 128 to 1024 pixels a side, any aspect ratio."""
    return _log(rng, 64, 4200)


def draw(rng):
    most = work(next(c for c in listed() if c["name"] == "full_5ref"))["flops"]
    while True:
        op = rng.choice(["request", "step", "step", "step", "step_noalloc", "step_fp8", "prefill", "prefill_fp8", "full",
                         "linear", "linear", "chain_step"])
        if op == "linear":
            # a layer's projections: rows of any prompt and image, hidden sizes of the head counts above
            h = 128 * rng.choice([8, 12, 16, 20, 24, 32])
            c = dict(op=op, m=_log(rng, 16, 24000), n=h * rng.choice([1, 3]), k=h, residual=rng.random() < 0.5)
        else:
            c = dict(op=op, mask=rng.choice(["perref", "perref", "paper", "isolated"]), st=rng.randint(1, 128),
                     lt=rng.choice([512, 256, rng.randint(8, 512)]), x=_image(rng),
                     refs=",".join(str(_image(rng)) for _ in range(rng.choice([1, 1, 2, 3, 4, 5, 6, 10]))),
                     B=rng.choice([1, 1, 2, 3]), H=rng.choice([2, 3, 6, 12, 16, 24, 24, 32, 40]), D=rng.choice([64, 128, 128]))
            if op == "full" and rng.random() < 0.7:
                c["mask"] = "dense"
            if op == "chain_step":
                c.update(H=rng.choice([8, 16, 24]), layers=rng.choice([1, 2, 4]))
            elif op.startswith("step") or op == "full":
                c.update(fused=rng.random() < 0.5, lse=rng.random() < 0.3)
        if work(c)["flops"] <= most:
            return c


# ---------------------------------------------------------------- inputs
KINDS = {"st": 0, "lt": 1, "x": 2}


def _segments(c):
    segs = [(KINDS[k], c[k]) for k in ("st", "lt", "x") if c[k]]
    return segs + [(3, int(n)) for n in c["refs"].split(",")]


def _rows(c):
    segs = _segments(c)
    return {"static": sum(n for k, n in segs if k in (0, 3)), "live": sum(n for k, n in segs if k in (1, 2)),
            "all": sum(n for _, n in segs),
            "cached": sum(n for k, n in segs if k == 3 or (k == 0 and c["mask"] in ("perref", "dense")))}


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _normal(g, shape, std=1.0):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32).mul_(std).to(torch.bfloat16)


def _qkv(c, g, n):
    B, H, D = c["B"], c["H"], c["D"]
    if c.get("fused"):
        t = _normal(g, (B, n, 3, H, D))
        return tuple(t[:, :, i] for i in range(3))
    return tuple(_normal(g, (B, n, H, D)) for _ in range(3))


def _codes(g, shape):
    """An 8-bit cache tensor as the prefill stores it: e4m3 codes and a power-of-two scale per (batch, head)."""
    x = _normal(g, shape)
    s = torch.exp2(torch.ceil(torch.log2(x.float().abs().amax(dim=(2, 3)) / 448.0)))
    codes = (x.float() / s[:, :, None, None]).to(torch.float8_e4m3fn).view(torch.uint8)
    return codes, s


def _inputs(c, seed):
    """Everything a call reads, on the GPU, from the seed alone."""
    g = _gen(seed)
    op = c["op"]
    if op == "linear":
        a = _normal(g, (c["m"], c["k"]))
        w = _normal(g, (c["n"], c["k"]), 1.0 / math.sqrt(c["k"]))
        return {"a": a, "w": w, "r": _normal(g, (c["m"], c["n"])) if c["residual"] else None}
    B, H, D, n = c["B"], c["H"], c["D"], _rows(c)
    cache = (B, H, n["cached"], D)
    if op == "chain_step":
        C = H * D
        return {"h": _normal(g, (B, n["live"], C)),
                "w_qkv": [_normal(g, (3 * C, C), 1.0 / math.sqrt(C)) for _ in range(c["layers"])],
                "w_o": [_normal(g, (C, C), 1.0 / math.sqrt(C)) for _ in range(c["layers"])],
                "caches": [(_normal(g, cache), _normal(g, cache)) for _ in range(c["layers"])]}
    if op == "full":
        return {"all": _qkv(c, g, n["all"])}
    d = {}
    if op in ("prefill", "prefill_fp8", "request"):
        d["static"] = _qkv(c, g, n["static"])
    if op in ("step", "step_noalloc", "step_fp8", "request"):
        d["live"] = _qkv(c, g, n["live"])
    if op in ("step", "step_noalloc"):
        d["cache"] = (_normal(g, cache), _normal(g, cache))
    if op == "step_fp8":
        (k8, sk), (v8, sv) = _codes(g, cache), _codes(g, cache)
        d["cache"] = (k8, v8, torch.stack([sk, sv], dim=2).contiguous())
    return d


def prepare(case, seed):
    """The inputs, and what a serving loop keeps: the layout, the output and cache buffers, the step's workspace."""
    s = dict(_inputs(case, seed), case=case)
    if case["op"] == "linear":
        s["out"] = torch.empty((case["m"], case["n"]), dtype=torch.bfloat16, device=DEV)
        return s
    B, H, D, n = case["B"], case["H"], case["D"], _rows(case)
    L = s["layout"] = rc.Layout(_segments(case), case["mask"])
    if case["op"] == "chain_step":
        s["chain"] = rc.Chain(L, s["w_qkv"], s["w_o"], H, D)
        return s
    bf16 = dict(dtype=torch.bfloat16, device=DEV)
    if "static" in s:
        s["o_static"] = torch.empty((B, n["static"], H, D), **bf16)
        if case["op"] == "prefill_fp8":
            k8, v8, sc = rc.fp8_cache_shapes(L, B, H, D)
            s["new"] = (torch.empty(k8, dtype=torch.uint8, device=DEV), torch.empty(v8, dtype=torch.uint8, device=DEV),
                        torch.empty(sc, dtype=torch.float32, device=DEV))
        else:
            s["new"] = tuple(torch.empty((B, H, n["cached"], D), **bf16) for _ in range(2))
    if "live" in s:
        s["o_live"] = torch.empty((B, n["live"], H, D), **bf16)
        s["lse"] = torch.empty((B, H, n["live"]), dtype=torch.float32, device=DEV) if case.get("lse") else None
        if case["op"] != "step_noalloc":
            need = L.workspace_bytes(B, H, D)
            s["workspace"] = torch.empty(need, dtype=torch.uint8, device=DEV) if need else None
    return s


def run(s):
    op, c = s["case"]["op"], s["case"]
    if op == "linear":
        return rc.linear(s["a"], s["w"], residual=s["r"], out=s["out"])
    if op == "chain_step":
        return s["chain"].step(s["h"], s["caches"])
    L = s["layout"]
    if op == "full":
        return rc.full_attention(L, *s["all"], want_lse=c.get("lse", False))
    out = ()
    cache = s.get("cache")
    if op == "prefill_fp8":
        o, _, k8, v8, sc = rc.ref_kv_prefill_fp8(L, *s["static"], o=s["o_static"], k_cache8=s["new"][0],
                                                 v_cache8=s["new"][1], kv_scale=s["new"][2])
        return o, k8, v8, sc
    if op in ("prefill", "request"):
        o, _, kc, vc = rc.ref_kv_prefill(L, *s["static"], o=s["o_static"], k_cache=s["new"][0], v_cache=s["new"][1])
        out, cache = (o, kc, vc), (kc, vc)
        if op == "prefill":
            return out
    if op == "step_noalloc":
        return rc.step_masked_attention_noalloc(L, *s["live"], *cache, s["o_live"], lse=s["lse"])
    step = rc.step_masked_attention_fp8 if op == "step_fp8" else rc.step_masked_attention
    return (*out, *step(L, *s["live"], *cache, o=s["o_live"], lse=s["lse"], workspace=s["workspace"]))


# ---------------------------------------------------------------- what a call cannot do without
def _visible(c):
    """visible[q][k]: the tokens of segment q read those of segment k (query first)."""
    segs = _segments(c)
    m = c["mask"]

    def v(q, k):
        kq, kk = segs[q][0], segs[k][0]
        if m == "dense":
            return True
        if m == "paper":
            return (kk in (0, 3)) if kq in (0, 3) else kk != 0
        if m == "perref":
            return kk == 0 if kq == 0 else (kk == 0 or k == q) if kq == 3 else True
        return False if kq == 0 else kk == 3 if kq == 3 else kk != 0  # isolated: anchors detached
    return [[v(q, k) for k in range(len(segs))] for q in range(len(segs))]


def _pairs(c, rows):
    segs, vis = _segments(c), _visible(c)
    return sum(n * sum(segs[k][1] for k in range(len(segs)) if vis[q][k])
               for q, (kind, n) in enumerate(segs) if kind in rows)


def _linear_work(m, n, k, residual):
    return 2 * (m * k + n * k + m * n * (2 if residual else 1)), 2 * m * n * k


def work(case):
    c, op = case, case["op"]
    if op == "linear":
        b, f = _linear_work(c["m"], c["n"], c["k"], c["residual"])
        return {"bytes": b, "flops": f}
    B, H, D, n = c["B"], c["H"], c["D"], _rows(c)
    row = 2 * B * H * D  # bytes of one token's Q, K, V or O
    b = f = 0
    if op in ("prefill", "prefill_fp8", "request"):  # Q, K, V read, O and the cached K and V written
        b += row * 4 * n["static"] + (row * 2 if op != "prefill_fp8" else row) * n["cached"]
        f += 4 * B * H * D * _pairs(c, (0, 3))
    if op in ("step", "step_noalloc", "step_fp8", "request"):
        b += row * 4 * n["live"] + (row * 2 if op != "step_fp8" else row) * n["cached"]
        f += 4 * B * H * D * _pairs(c, (1, 2))
    if op == "full":
        b, f = row * 4 * n["all"], 4 * B * H * D * _pairs(c, (0, 1, 2, 3))
    if op == "chain_step":  # hidden states in and out once; weights and caches of every layer once
        C, m = H * D, B * n["live"]
        b = 2 * 2 * m * C + c["layers"] * (2 * 4 * C * C + row * 2 * n["cached"])
        f = c["layers"] * (2 * m * C * 4 * C + 4 * B * H * D * _pairs(c, (1, 2)))
    return {"bytes": b, "flops": f}


def tolerance(case):
    # O is bf16 of an fp32 sum over bf16 weights, about 2.3e-3 from the 64-bit result in the 2-norm; a projection
    # carries its one bf16 rounding (1.7e-3); four chained layers add up theirs.  Largest single differences stay
    # within a few bf16 steps of the result's scale.
    if case["op"] == "linear":
        return {"rel": 7e-3, "max": 0.06}
    return {"rel": 1e-2, "max": 0.1}


# ---------------------------------------------------------------- the same in 64 bits, plain torch
def _bf16(x):
    """Round to bf16 once (round to nearest even), kept in 64 bits: through a float32 that keeps the ties apart."""
    y = x.float()
    exact = y.double() == x
    bits = y.view(torch.int32)
    toward = (x.abs() < y.double().abs()) & ~exact  # float32 rounded away from zero
    bits = torch.where(toward, bits - 1, bits)
    bits = torch.where(exact, bits, bits | 1)       # a sticky bit
    return bits.view(torch.float32).to(torch.bfloat16).double()


def _attend(c, q, k, v, kinds_q, kinds_k):
    """q [B, Nq, H, D] rows of the segments of kinds_q against k, v [B, Nk, H, D] of the segments of kinds_k, each in
    sequence order; 64 bits.  Returns O [B, Nq, H, D] and the log-sum-exp [B, H, Nq]."""
    segs, vis = _segments(c), _visible(c)
    B, Nq, H, D = q.shape
    o = torch.zeros((B, Nq, H, D), dtype=torch.float64, device=q.device)
    lse = torch.full((B, H, Nq), -math.inf, dtype=torch.float64, device=q.device)
    kpos, p = {}, 0
    for i, (kind, n) in enumerate(segs):
        if i in kinds_k:
            kpos[i] = (p, p + n)
            p += n
    for b in range(B):
        for h in range(H):
            kh, vh, qh = k[b, :, h].double(), v[b, :, h].double(), q[b, :, h].double()
            row = 0
            for i, (kind, n) in enumerate(segs):
                if kind not in kinds_q:
                    continue
                keys = [torch.arange(*kpos[j], device=q.device) for j in range(len(segs)) if vis[i][j]]
                if keys:
                    at = torch.cat(keys)
                    ki, vi = kh[at], vh[at]
                    for r in range(row, row + n, 4096):
                        e = min(r + 4096, row + n)
                        s = qh[r:e] @ ki.t().contiguous() / math.sqrt(D)
                        m = s.amax(dim=1, keepdim=True)
                        s = torch.exp(s - m)
                        t = s.sum(dim=1, keepdim=True)
                        o[b, r:e, h] = s @ vi / t
                        lse[b, h, r:e] = (m + torch.log(t))[:, 0]
                row += n
    return o, lse


def _step_keys(c, live, cache):
    """Live and cached K (or V) in sequence order, and the segments they hold."""
    segs = _segments(c)
    parts, held, pl, pc = [], [], 0, 0
    for i, (kind, n) in enumerate(segs):
        if kind in (1, 2):
            parts.append(live[:, pl:pl + n])
            pl += n
        elif kind == 3 or c["mask"] in ("perref", "dense"):
            parts.append(cache[:, :, pc:pc + n].transpose(1, 2))
            pc += n
        else:
            continue
        held.append(i)
    return torch.cat(parts, dim=1), held


def _exact_step(c, q, k, v, kc, vc):
    kk, held = _step_keys(c, k, kc)
    vv, _ = _step_keys(c, v, vc)
    return _attend(c, q, kk, vv, (1, 2), held)


def _exact_prefill(c, static):
    """O of the static rows, and the cached rows of K and V."""
    segs = _segments(c)
    held = [i for i, (kind, _) in enumerate(segs) if kind in (0, 3)]
    o, _ = _attend(c, *static, (0, 3), held)
    first = c["st"] if c["mask"] in ("paper", "isolated") else 0
    kc, vc = (t[:, first:].transpose(1, 2).contiguous() for t in static[1:])
    return o, kc, vc


def exact(case, seed):
    c, op, s = case, case["op"], _inputs(case, seed)
    if op == "linear":
        out = s["a"].double() @ s["w"].double().t().contiguous()
        return out if s["r"] is None else out + s["r"].double()
    if op == "chain_step":
        B, H, D, n = c["B"], c["H"], c["D"], _rows(c)["live"]
        h = s["h"].double()
        for wq, wo, (kc, vc) in zip(s["w_qkv"], s["w_o"], s["caches"]):
            qkv = _bf16(h.reshape(B * n, H * D) @ wq.double().t().contiguous()).view(B, n, 3, H, D)
            o, _ = _exact_step(c, qkv[:, :, 0], qkv[:, :, 1], qkv[:, :, 2], kc.double(), vc.double())
            h = _bf16(_bf16(o).reshape(B * n, H * D) @ wo.double().t().contiguous() + h.reshape(B * n, H * D))
        return h.view(B, n, H * D)
    if op == "full":
        o, lse = _attend(c, *s["all"], (0, 1, 2, 3), list(range(len(_segments(c)))))
        return o, lse if c.get("lse") else None
    if op == "prefill_fp8":
        o, kc, vc = _exact_prefill(c, s["static"])
        amax = torch.stack([t.double().abs().amax(dim=(2, 3)) for t in (kc, vc)], dim=2)
        return o, None, None, torch.exp2(torch.ceil(torch.log2(amax / 448.0)))
    out, cache = (), s.get("cache")
    if op in ("prefill", "request"):
        o, kc, vc = _exact_prefill(c, s["static"])
        out, cache = (o, kc.double(), vc.double()), (kc, vc)
        if op == "prefill":
            return out
    if op == "step_fp8":
        k8, v8, sc = cache
        cache = tuple(t.view(torch.float8_e4m3fn).float() * sc[:, :, i, None, None] for i, t in enumerate((k8, v8)))
    o, lse = _exact_step(c, *s["live"], *cache)
    return (*out, o, lse if c.get("lse") else None)
