"""Performance cases: the calls that a user of this library makes, through the public binding.

A case is a dict of plain values.  Its "kind" says which entry point it goes through:

  attn      dsattn_forward: the fused attention of one U-Net level
  two_stage dsattn_gather_context, then dsattn_forward_ctx on the gathered context
  layer     dsattn_temporal_layer: Q/K/V projections, attention, output projection
  groupnorm dsattn_groupnorm over the whole video
  conv      dsattn_temporal_conv

listed() holds fixed cases, draw() gives more of the same ranges, prepare() makes inputs on the GPU
from a seed, run() makes one pass, work() counts what a pass cannot do without, exact() computes the
same results in 64 bits with plain torch, and tolerance() says how far two correct implementations
may be apart.
"""
import math

import numpy as np
import torch

from paper_2406_16260_amd import binding as B

DEV = "cuda:0"
GROUPS = 32   # channel groups of the group normalisation
EPS = 1e-5

_ATTN = {"clip_len": 16, "w": 2, "G": 16, "dtype": "bf16", "out": "bf16", "window": -1,
         "bias_local": 0.0, "bias_global": 0.0, "dedup": False}


def _attn(name, **kw):
    return {"name": name, "kind": "attn", **_ATTN, **kw}


def listed():
    return [
        # The tiny fp32 configuration (2 clips x 4 frames, 4 x 4 positions, one head of 8): a call
        # whose work is nothing, so that its cost is the host path and one launch.
        _attn("attn_f32_tiny", clip_len=4, n_clips=2, w=1, G=2, P=16, heads=1, D=8, dtype="f32",
              out="f32"),
        # The widest U-Net level (40 x 64 positions, 8 heads of 40) on a short video of 64 frames:
        # the ordinary single generation.
        _attn("attn_64f_l1", n_clips=4, P=2560, heads=8, D=40),
        # The headline configuration: 2,304 frames at the 10 x 16 level, 8 heads of 160.
        _attn("attn_2304f_l3", n_clips=144, P=160, heads=8, D=160),
        # The largest call: 2,304 frames at the widest level with 64 global frames and 4 + 4
        # neighbouring ones (the four-level sweep's first level).
        _attn("attn_2304f_l1_g64", n_clips=144, w=4, G=64, P=2560, heads=8, D=40),
        # The paper's own setting: 8 clips of 288 frames, 8 + 8 neighbouring frames, every query
        # seeing the frames within 8 of its own, and the global scope's weight raised tenfold as
        # during the first denoising steps.
        _attn("attn_288f_window", clip_len=288, n_clips=8, w=8, P=160, heads=8, D=160, window=8,
              bias_global=math.log(10.0)),
        # Clips of a base model that does not generate 16 frames at a time (24 here), an odd number
        # of positions (9 x 15), five heads.
        _attn("attn_24f_clips", clip_len=24, n_clips=12, w=3, G=12, P=135, heads=5, D=64),
        # One layer at the bottom of the U-Net (5 x 8 positions, 1,280 channels) on a short video:
        # three launches that do not fill the chip.
        _attn("layer_64f_l4", kind="layer", n_clips=4, P=40, heads=8, D=160, bias=True),
        # One layer at the headline configuration.
        _attn("layer_2304f_l3", kind="layer", n_clips=144, P=160, heads=8, D=160, bias=False),
        # One layer in fp32, as a check run of the same model makes it.
        _attn("layer_f32", kind="layer", n_clips=4, P=160, heads=8, D=80, dtype="f32", out="f32",
              bias=True),
        # The paper's data flow: the context is gathered first, then attended over.
        _attn("two_stage_l2", kind="two_stage", n_clips=24, P=640, heads=8, D=80),
        # The group normalisation in front of a temporal module, headline level.
        {"name": "groupnorm_2304f_l3", "kind": "groupnorm", "clip_len": 16, "n_clips": 144,
         "P": 160, "C": 1280, "dtype": "bf16"},
        # The temporal convolution (3 taps) of the 20 x 32 level on 384 frames.
        {"name": "conv_384f_l2", "kind": "conv", "clip_len": 16, "n_clips": 24, "P": 640,
         "c_in": 640, "c_out": 640, "reach": 1, "dtype": "bf16"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["attn", "attn", "attn", "layer", "layer", "two_stage", "groupnorm", "conv"])
    f32 = rng.random() < (0.15 if kind == "conv" else 0.25)
    dtype = "f32" if f32 else "bf16"
    P = _log(rng, 16, 2560)
    if kind in ("groupnorm", "conv"):
        # at most as many elements as the headline level's tensor has
        C = rng.choice([320, 640, 960, 1280])
        n_clips = min(_log(rng, 1, 144), max(1, 471859200 // (16 * P * C)))
        if kind == "groupnorm":
            return {"kind": kind, "clip_len": rng.choice([8, 16, 24]) if n_clips <= 96 else 16,
                    "n_clips": n_clips, "P": P, "C": C, "dtype": dtype}
        c_out = rng.choice([320, 640, C])
        reach = rng.choice([1, 1, 1, 2])
        # fp32: at most about 30 GFLOP
        most = 15e9 if f32 else 900e9
        rows = int(most / ((2 * reach + 1) * C * c_out))
        P = min(P, max(1, rows // 16))
        return {"kind": kind, "clip_len": 16, "n_clips": max(1, min(n_clips, rows // (16 * P))),
                "P": P, "c_in": C, "c_out": c_out, "reach": reach, "dtype": dtype}
    D, heads = rng.choice([(40, 8), (80, 8), (160, 8), (64, 5), (64, 10), (128, 8), (96, 6), (32, 4)])
    c = {"kind": kind, **_ATTN, "heads": heads, "D": D, "w": rng.choice([0, 1, 2, 3, 4, 6, 8]),
         "G": rng.choice([0, 4, 8, 12, 16, 16, 16, 32, 64]), "dtype": dtype, "out": dtype}
    c["clip_len"] = rng.choice([16, 16, 16, 16, 8, 14, 24, 25, 32, 48])
    if kind == "attn":
        if c["clip_len"] == 16 and rng.random() < 0.3:
            c["clip_len"] = 16 * rng.choice([2, 4, 6, 12, 18])
            c["window"] = rng.choice([2, 4, 8, 12])
        if rng.random() < 0.25:
            c["bias_global"] = rng.choice([math.log(10.0), -1.5])
        if rng.random() < 0.15:
            c["bias_local"] = math.log(10.0)
        if rng.random() < 0.15:
            c["dedup"] = True
        if rng.random() < 0.2:
            c["out"] = "f32"
    C = heads * D
    # elements of one [F, P, C] tensor: the headline level's at most for the bf16 attention; the
    # two-stage path and fp32 an eighth of that; layers by their flops (900 GFLOP, fp32 60 GFLOP)
    most = 471859200 // (8 if f32 or kind == "two_stage" else 1)
    if kind == "layer":
        most = min(most, int((60e9 if f32 else 900e9) / (8 * C)))
        c["bias"] = rng.random() < 0.5
    c["P"] = min(P, max(1, most // (C * c["clip_len"])))
    c["n_clips"] = max(1, min(_log(rng, 1, 144), most // (C * c["clip_len"] * c["P"])))
    c["G"] = min(c["G"], c["n_clips"] * c["clip_len"])
    return c


# ------------------------------------------------------------------ inputs

def _torch_dtype(name):
    return torch.float32 if name == "f32" else torch.bfloat16


def _frames(gen, F, P, C, dtype, noise=0.1):
    """Slowly varying latents: a base per (position, channel) that all frames share, plus noise."""
    out = torch.empty((F, P, C), dtype=_torch_dtype(dtype), device=DEV)
    base = torch.randn((P, C), generator=gen, device=DEV)
    chunk = max(1, min(F, (1 << 27) // (P * C)))
    for f in range(0, F, chunk):
        n = min(chunk, F - f)
        x = torch.randn((n, P, C), generator=gen, device=DEV)
        out[f:f + n] = x.mul_(noise).add_(base)
    return out


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _global_idx(case, seed):
    """Up to 16 global frames at uniform stride over the video, more at random sorted frames."""
    F, G = case["n_clips"] * case["clip_len"], case["G"]
    if G <= 16:
        return [(j * F) // G for j in range(G)]
    return sorted(np.random.default_rng(seed).choice(F, size=G, replace=False).tolist())


def _code(name):
    return B.DSATTN_F32 if name == "f32" else B.DSATTN_BF16


def _inputs(case, seed):
    """What the case's tensors are, in a fixed order from one generator: run() and exact() see the
    same values."""
    gen = _gen(seed)
    F, P = case["n_clips"] * case["clip_len"], case["P"]
    kind, dt = case["kind"], case["dtype"]
    if kind in ("attn", "two_stage"):
        C = case["heads"] * case["D"]
        return [_frames(gen, F, P, C, dt) for _ in range(3)]
    if kind == "layer":
        C = case["heads"] * case["D"]
        x = _frames(gen, F, P, C, dt)
        W = [(torch.randn((C, C), generator=gen, device=DEV) / C ** 0.5).to(_torch_dtype(dt))
             for _ in range(4)]
        b = [0.1 * torch.randn((C,), generator=gen, device=DEV) for _ in range(4)]
        return [x, W, b if case["bias"] else None]
    if kind == "groupnorm":
        C = case["C"]
        x = _frames(gen, F, P, C, dt, noise=0.5)
        return [x, 1.0 + 0.1 * torch.randn((C,), generator=gen, device=DEV),
                0.1 * torch.randn((C,), generator=gen, device=DEV)]
    ci, co, taps = case["c_in"], case["c_out"], 2 * case["reach"] + 1
    x = _frames(gen, F, P, ci, dt)
    w = (torch.randn((taps, co, ci), generator=gen, device=DEV) / (taps * ci) ** 0.5).to(_torch_dtype(dt))
    return [x, w, 0.1 * torch.randn((co,), generator=gen, device=DEV)]


def prepare(case, seed):
    s = {"case": case, "in": _inputs(case, seed)}
    F, P = case["n_clips"] * case["clip_len"], case["P"]
    kind, dt = case["kind"], case["dtype"]
    if kind in ("attn", "two_stage", "layer"):
        C = case["heads"] * case["D"]
        s["plan"] = B.dsattn_plan(
            case["clip_len"], case["n_clips"], case["w"], P, case["heads"], case["D"],
            _global_idx(case, seed), io_dtype=_code(dt), out_dtype=_code(case["out"]),
            flags=B.DSATTN_FLAG_DEDUP_GLOBAL if case["dedup"] else 0, device=0,
            bias_local=case["bias_local"], bias_global=case["bias_global"],
            window=case["window"] if case["window"] >= 0 else None)
        s["out"] = torch.empty((F, P, C), dtype=_torch_dtype(case["out"]), device=DEV)
        if kind == "two_stage":
            lk = s["plan"].lk_max
            s["ctx"] = [torch.empty((case["n_clips"], lk, P, C), dtype=_torch_dtype(dt), device=DEV)
                        for _ in range(2)]
        if kind == "layer":
            s["space"] = torch.empty(B.dsattn_temporal_layer_workspace(s["plan"]), dtype=torch.uint8,
                                     device=DEV)
    elif kind == "groupnorm":
        n = B.dsattn_groupnorm_workspace(case["clip_len"], case["n_clips"], P, case["C"], GROUPS,
                                         io_dtype=_code(dt), eps=EPS)
        s["space"] = torch.empty(n, dtype=torch.uint8, device=DEV)
        s["out"] = torch.empty_like(s["in"][0])
        s["stats"] = torch.empty(2 * GROUPS, device=DEV)
    else:
        s["out"] = torch.empty((F, P, case["c_out"]), dtype=_torch_dtype(dt), device=DEV)
    return s


def run(state):
    c, t, o = state["case"], state["in"], state["out"]
    kind = c["kind"]
    if kind == "attn":
        B.dsattn_forward(state["plan"], t[0], t[1], t[2], o)
        return o
    if kind == "two_stage":
        kc, vc = state["ctx"]
        B.dsattn_gather_context(state["plan"], t[1], t[2], kc, vc)
        B.dsattn_forward_ctx(state["plan"], t[0], kc, vc, o)
        return [o, kc, vc]
    if kind == "layer":
        B.dsattn_temporal_layer(state["plan"], t[0], t[1], state["space"], o, biases=t[2])
        return o
    if kind == "groupnorm":
        B.dsattn_groupnorm(c["clip_len"], c["n_clips"], c["P"], c["C"], GROUPS, t[0], o,
                           state["space"], state["space"].numel(), gamma=t[1], beta=t[2],
                           stats=state["stats"], io_dtype=_code(c["dtype"]), eps=EPS)
        return [o, state["stats"]]
    B.dsattn_temporal_conv(c["clip_len"], c["n_clips"], c["P"], c["c_in"], c["c_out"], c["reach"],
                           t[0], t[1], o, bias=t[2], io_dtype=_code(c["dtype"]),
                           out_dtype=_code(c["dtype"]))
    return o


# ------------------------------------------------------------------ what a pass cannot do without

def _ctx_ranges(case):
    """Per clip: the local frame range [lo, hi) of its context list."""
    Fc, N, w = case["clip_len"], case["n_clips"], case["w"]
    F = Fc * N
    return [(max(0, i * Fc - w), min(F, (i + 1) * Fc + w)) for i in range(N)]


def work(case):
    F, P = case["n_clips"] * case["clip_len"], case["P"]
    e = 4 if case["dtype"] == "f32" else 2
    kind = case["kind"]
    if kind == "groupnorm":
        n = F * P * case["C"]
        return {"bytes": 2 * n * e + 8 * case["C"] + 8 * GROUPS, "flops": 8 * n}
    if kind == "conv":
        ci, co, n = case["c_in"], case["c_out"], case["reach"]
        pairs = sum(min(F, f + n + 1) - max(0, f - n) for f in range(F))
        return {"bytes": F * P * (ci + co) * e + (2 * n + 1) * ci * co * e + 4 * co,
                "flops": 2 * pairs * P * ci * co}
    C = case["heads"] * case["D"]
    n = F * P * C
    keys = 0  # (query, key) pairs of one position and head
    for i, (lo, hi) in enumerate(_ctx_ranges(case)):
        if case["window"] < 0:
            keys += case["clip_len"] * (hi - lo + case["G"])
        else:
            for a in range(i * case["clip_len"], (i + 1) * case["clip_len"]):
                keys += min(hi, a + case["window"] + 1) - max(lo, a - case["window"]) + case["G"]
    flops = 4 * keys * P * C
    if kind == "layer":
        return {"bytes": 2 * n * e + 4 * C * C * e + (16 * C if case["bias"] else 0),
                "flops": flops + 8 * n * C}
    out = 4 if case["out"] == "f32" else 2
    if kind == "attn":
        return {"bytes": 3 * n * e + n * out, "flops": flops}
    lk = max(hi - lo for lo, hi in _ctx_ranges(case)) + case["G"]
    ctx = case["n_clips"] * lk * P * C
    # K and V read, both contexts written and read again, Q read, O written
    return {"bytes": 3 * n * e + 4 * ctx * e + n * out, "flops": flops}


def tolerance(case):
    # About four times what the entry points are off exact() by (2-norm).  bf16: 1.7e-3, which is the
    # rounding of the outputs alone; 2.4e-3 for a layer, which rounds Q, K, V and the attention's
    # output too.  fp32: 5e-7 in a layer with sums of 640 terms, about 1e-6 for the longest sums.
    if case["dtype"] == "f32":
        return {"rel": 5e-6}
    return {"rel": 1e-2 if case["kind"] == "layer" else 7e-3}


# ------------------------------------------------------------------ the same in 64 bits

def _attention64(case, gidx, q, k, v):
    """[F, P, C] each, any float type; the Dual-scope attention in 64 bits, clip by clip."""
    F, P, C = q.shape
    h, D = case["heads"], case["D"]
    Fc, r = case["clip_len"], case["window"]
    out = torch.empty((F, P, C), dtype=torch.float64, device=q.device)
    pc = max(1, (1 << 27) // ((2 * Fc + 2 * case["w"] + case["G"]) * C))
    for i, (lo, hi) in enumerate(_ctx_ranges(case)):
        frames = list(range(lo, hi)) + list(gidx)
        nl = hi - lo
        ctx = torch.tensor(frames, device=q.device)
        aq = torch.arange(i * Fc, (i + 1) * Fc, device=q.device)
        bias = torch.zeros((Fc, len(frames)), dtype=torch.float64, device=q.device)
        bias[:, :nl] += case["bias_local"]
        bias[:, nl:] += case["bias_global"]
        if r >= 0:
            bias[:, :nl].masked_fill_((ctx[None, :nl] - aq[:, None]).abs() > r, -math.inf)
        if case["dedup"]:
            seen_before = [g in gidx[:j] for j, g in enumerate(gidx)]
            for j, g in enumerate(gidx):
                if seen_before[j]:
                    bias[:, nl + j] = -math.inf
                elif lo <= g < hi:
                    near = (aq - g).abs() <= r if r >= 0 else torch.ones_like(aq, dtype=torch.bool)
                    bias[near, nl + j] = -math.inf
        for p in range(0, P, pc):
            def rows(t, idx):
                x = t[idx, p:p + pc].to(torch.float64).reshape(len(idx), -1, h, D)
                return x.permute(1, 2, 0, 3).contiguous()
            s = torch.matmul(rows(q, aq), rows(k, ctx).transpose(2, 3).contiguous())
            s = torch.softmax(s / math.sqrt(D) + bias, dim=-1)
            o = torch.matmul(s, rows(v, ctx))
            out[i * Fc:(i + 1) * Fc, p:p + pc] = o.permute(2, 0, 1, 3).reshape(Fc, -1, C)
    return out


def _affine64(x, w, b):
    F, P, C = x.shape
    out = torch.empty((F, P, w.shape[0]), dtype=torch.float64, device=x.device)
    wt = w.to(torch.float64).t().contiguous()
    chunk = max(1, (1 << 27) // (P * C))
    for f in range(0, F, chunk):
        y = torch.matmul(x[f:f + chunk].to(torch.float64).reshape(-1, C), wt)
        if b is not None:
            y += b.to(torch.float64)
        out[f:f + chunk] = y.reshape(-1, P, w.shape[0])
    return out


def exact(case, seed):
    t = _inputs(case, seed)
    kind = case["kind"]
    if kind == "attn":
        return _attention64(case, _global_idx(case, seed), *t)
    if kind == "two_stage":
        gidx = _global_idx(case, seed)
        spans = _ctx_ranges(case)
        lk = max(hi - lo for lo, hi in spans) + len(gidx)
        ctx = [torch.zeros((case["n_clips"], lk) + tuple(x.shape[1:]), dtype=x.dtype, device=DEV)
               for x in t[1:]]
        for i, (lo, hi) in enumerate(spans):
            frames = torch.tensor(list(range(lo, hi)) + list(gidx), device=DEV)
            for c, x in zip(ctx, t[1:]):
                c[i, :len(frames)] = x[frames]
        return [_attention64(case, gidx, *t)] + ctx
    if kind == "layer":
        x, W, b = t
        b = b or [None] * 4
        q, k, v = (_affine64(x, W[g], b[g]) for g in range(3))
        a = _attention64(case, _global_idx(case, seed), q, k, v)
        return _affine64(a, W[3], b[3])
    if kind == "groupnorm":
        x, gamma, beta = t
        F, P, C = x.shape
        chunk = max(1, (1 << 27) // (P * C))
        n = F * P * (C // GROUPS)

        def sums(f):
            total = torch.zeros(C, dtype=torch.float64, device=DEV)
            for i in range(0, F, chunk):
                total += f(x[i:i + chunk].to(torch.float64)).sum(dim=(0, 1))
            return total.reshape(GROUPS, -1).sum(dim=1) / n
        mean = sums(lambda z: z)
        mc = mean.repeat_interleave(C // GROUPS)
        rstd = 1.0 / torch.sqrt(sums(lambda z: (z - mc) ** 2) + EPS)
        scale = rstd.repeat_interleave(C // GROUPS) * gamma.to(torch.float64)
        out = torch.empty((F, P, C), dtype=torch.float64, device=DEV)
        for i in range(0, F, chunk):
            out[i:i + chunk] = (x[i:i + chunk].to(torch.float64) - mc) * scale + beta.to(torch.float64)
        return [out, torch.cat([mean, rstd])]
    x, w, b = t
    F = x.shape[0]
    out = None
    for tap in range(w.shape[0]):
        y = _affine64(x, w[tap], b if tap == case["reach"] else None)
        if out is None:
            out = torch.zeros_like(y)
        d = tap - case["reach"]
        lo, hi = max(0, -d), min(F, F - d)
        out[lo:hi] += y[lo + d:hi + d]
    return out
