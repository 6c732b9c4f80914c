"""The matrix-core kernels behind dsattn_forward for what the streaming kernel does not take (fp32
tensors, clips that are not whole 16-frame tiles, wide local scopes, long global lists): parity with
the oracle and agreement with the generic kernel, which the flag still selects.

Bars: nothing is rounded to 16 bits on the way (bf16 inputs are exact, weights keep 24 bits), so fp32
results, from either input type, are held to the fp32 bar of 1e-5; the observed maximum is 1e-6."""
import numpy as np
import pytest
import torch

import parity_util as U
from paper_2406_16260_amd import binding as B
from paper_2406_16260_amd import synth

DEV = "cuda:0"
pytestmark = pytest.mark.gpu


def make(F, P, C, dtype, seed=17, gen="iid"):
    return tuple(synth.make_tensor(F, P, C, seed + t, gen, dtype).to(DEV) for t in range(3))


def assert_tile_kernel(info, clip_len, n_clips, P, h, query_tiles=1):
    """The report of a plan that runs the 16-query tile kernel: no streaming variant, a wavefront per
    query tile (or two of them), position and head, four to a workgroup."""
    assert (info["kernel"], info["variant"], info["block_threads"]) == (0, -1, 256), info
    assert info["n_tasks"] == n_clips * P * h * -(-clip_len // (16 * query_tiles)), info


def assert_generic_kernel(info, n_clips, P, h):
    assert (info["kernel"], info["variant"], info["block_threads"]) == (0, -1, 64), info
    assert info["n_tasks"] == n_clips * P * h, info


CASES = [
    # clip_len, n_clips, w, P, h, D, G, options
    (24, 4, 3, 5, 2, 64, 12, {}),                        # two query tiles, the second half empty
    (1, 9, 1, 4, 2, 112, 3, {}),                         # a single query per tile
    (7, 5, 3, 9, 3, 72, 4, {}),                          # D not a multiple of 16
    (33, 3, 0, 2, 1, 40, 0, {}),                         # no context at all: 33 keys, one in the last tile
    (16, 1, 0, 3, 1, 8, 0, {}),                          # exactly one key tile (bf16: the streaming kernel's job
                                                         # at other head sizes)
    (15, 2, 1, 3, 1, 16, 1, {}),                         # 17 keys
    (48, 2, 20, 2, 2, 160, 200, {}),                     # 68 to 268 keys, the largest head
    (14, 5, 6, 3, 2, 128, 20, {"window": 4}),
    (24, 4, 5, 3, 2, 80, 20, {"window": 0}),             # every local key hidden but one
    (24, 4, 2, 3, 2, 48, 30, {"dedup": True}),
    (24, 4, 2, 3, 2, 144, 30, {"dedup": True, "window": 5}),
    (20, 3, 2, 3, 5, 96, 16, {"bias_global": 2.302585}),
    (20, 3, 2, 3, 3, 32, 16, {"bias_local": 50.0, "bias_global": -50.0}),
    (12, 3, 2, 2, 1, 24, 7, {"bias_global": 3e38, "bias_local": -3e38}),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", CASES)
def test_tile_kernels_match_oracle_and_generic_kernel(case, dtype):
    clip_len, n_clips, w, P, h, D, G, opts = case
    print(f"[case] tile {case} {dtype}", flush=True)
    F = clip_len * n_clips
    g = np.random.default_rng(5).integers(0, F, size=G).tolist()     # unsorted, with repeats
    q, k, v = make(F, P, h * D, dtype)
    opts = dict(opts)
    dedup = opts.pop("dedup", False)
    flags = B.DSATTN_FLAG_DEDUP_GLOBAL if dedup else 0
    ref = U.oracle_forward(q, k, v, clip_len, n_clips, w, h, g, dedup=dedup, **opts)
    for out in (["f32"] if dtype == "f32" else ["f32", "bf16"]):
        o, info = U.library_forward(q, k, v, clip_len, n_clips, w, h, g, out_dtype=out, flags=flags, **opts)
        assert_tile_kernel(info, clip_len, n_clips, P, h)
        U.assert_parity(o, ref, "f32_strict" if out == "f32" else "bf16", what=str(case))
        og, info = U.library_forward(q, k, v, clip_len, n_clips, w, h, g, out_dtype=out,
                                  flags=flags | B.DSATTN_FLAG_FORCE_GENERIC, **opts)
        assert_generic_kernel(info, n_clips, P, h)
        # both within 1e-5 of the same numbers, then at most one rounding apart in bf16
        bar = 2e-5 if out == "f32" else 2e-5 + 2 * U.bf16_half_ulp(ref).max()
        assert float((o.double() - og.double()).abs().max()) <= bar


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("clip_len,w,G", [
    (24, 3, 0), (8, 0, 1), (25, 2, 16),   # 24 to 30, 8 and 27 to 29 local keys; the last bit of a tile
    (8, 4, 62), (24, 4, 63), (13, 1, 63),  # the most entries that one word of bits holds, and padding behind them
    (24, 4, 64), (8, 2, 70),               # more: key by key
])
@pytest.mark.parametrize("biases", [{}, {"bias_global": 1.5}, {"bias_local": 2.0}])
def test_set_union_without_a_window(clip_len, w, G, biases, dtype):
    """Hidden entries are a word of bits a task, from 64 on looked up key by key: the first and last entries, entries
    on both sides of a key tile's edge and of the local keys' end, repeats, and every entry local."""
    n_clips, P, h, D = 6, 2, 2, 40
    F = clip_len * n_clips
    rng = np.random.default_rng(G + clip_len)
    lists = [rng.integers(0, F, size=G).tolist(), [(F // 2 + i) % F for i in range(G)]] if G else [[]]
    for g in lists:
        print(f"[case] union clip_len={clip_len} w={w} G={G} {biases} {dtype}", flush=True)
        q, k, v = make(F, P, h * D, dtype)
        ref = U.oracle_forward(q, k, v, clip_len, n_clips, w, h, g, dedup=True, **biases)
        o, info = U.library_forward(q, k, v, clip_len, n_clips, w, h, g, out_dtype="f32",
                                    flags=B.DSATTN_FLAG_DEDUP_GLOBAL, **biases)
        assert_tile_kernel(info, clip_len, n_clips, P, h)
        U.assert_parity(o, ref, "f32_strict", what=f"union G={G}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D", [8, 24, 32, 64, 72, 80, 96, 112, 128, 144, 160])
def test_set_union_and_biases_at_every_head_size(D, dtype):
    """The kernels for the set union and for biases alone, on the tensors and on a materialised context, in both output
    types: lists on both sides of a key tile's edge, repeats, local entries."""
    clip_len, n_clips, w, P, h, G = 24, 5, 3, 2, 2, 19
    F = clip_len * n_clips
    g = np.random.default_rng(D).integers(0, F, size=G).tolist()
    q, k, v = make(F, P, h * D, dtype)
    for opts in ({"dedup": True}, {"dedup": True, "bias_local": 1.5}, {"bias_global": 1.5}):
        print(f"[case] union D={D} {opts} {dtype}", flush=True)
        ref = U.oracle_forward(q, k, v, clip_len, n_clips, w, h, g, **opts)
        kw = {x: y for x, y in opts.items() if x != "dedup"}
        kw["flags"] = B.DSATTN_FLAG_DEDUP_GLOBAL if "dedup" in opts else 0
        for out in (["f32"] if dtype == "f32" else ["f32", "bf16"]):
            o, info = U.library_forward(q, k, v, clip_len, n_clips, w, h, g, out_dtype=out, **kw)
            assert_tile_kernel(info, clip_len, n_clips, P, h)
            U.assert_parity(o, ref, "f32_strict" if out == "f32" else "bf16", what=f"{opts}")
            plan = B.dsattn_plan(clip_len, n_clips, w, P, h, D, g, io_dtype=U.dt_code(dtype), out_dtype=U.dt_code(out),
                                 **kw)
            ctx = [torch.empty(n_clips, plan.lk_max, P, h * D, dtype=q.dtype, device=DEV) for _ in range(2)]
            o2 = torch.full_like(o, float("nan"))
            B.dsattn_gather_context(plan, k, v, *ctx)
            B.dsattn_forward_ctx(plan, q, *ctx, o2)
            torch.cuda.synchronize()
            plan.close()
            assert torch.equal(o, o2)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("clip_len,w,G,window", [
    (24, 3, 0, 0), (8, 8, 1, 2), (25, 2, 16, 7),     # nothing but itself; across clips; local and global in one tile
    (40, 8, 9, 3), (48, 0, 70, 200),                 # whole key tiles out of a query's sight; wider than the clip
])
@pytest.mark.parametrize("opts", [{}, {"bias_global": 1.5}, {"bias_local": 2.0}, {"dedup": True}])
def test_window_with_and_without_the_set_union(clip_len, w, G, window, opts, dtype):
    n_clips, P, h = 5, 2, 2
    F = clip_len * n_clips
    rng = np.random.default_rng(G + clip_len)
    g = rng.integers(0, F, size=G).tolist()
    for D in (40, 96):
        print(f"[case] window clip_len={clip_len} w={w} G={G} r={window} {opts} {dtype} D={D}", flush=True)
        q, k, v = make(F, P, h * D, dtype)
        ref = U.oracle_forward(q, k, v, clip_len, n_clips, w, h, g, window=window, **opts)
        biases = {x: y for x, y in opts.items() if x != "dedup"}
        o, info = U.library_forward(q, k, v, clip_len, n_clips, w, h, g, out_dtype="f32", window=window,
                                    flags=B.DSATTN_FLAG_DEDUP_GLOBAL if "dedup" in opts else 0, **biases)
        assert_tile_kernel(info, clip_len, n_clips, P, h)
        U.assert_parity(o, ref, "f32_strict", what=f"window {window}, G={G}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_peaked_softmax_with_growing_maximum(dtype):
    """Scores that grow along the list (the running maximum moves at every key tile) and scores that
    shrink (it never moves again), 100 in size: the accumulated sums are rescaled, not lost."""
    clip_len, n_clips, P, D = 40, 2, 3, 64
    F = clip_len * n_clips
    for sign in (1.0, -1.0):
        q, k, v = make(F, P, D, dtype)
        ramp = sign * torch.linspace(0.0, 12.0, F, device=DEV)[:, None, None]
        q = (q * 0.1 + 1.0).to(q.dtype)
        k = (k.float() * 0.1 + ramp).to(k.dtype)
        ref = U.oracle_forward(q, k, v, clip_len, n_clips, 6, 1, [79, 0, 40])
        o, info = U.library_forward(q, k, v, clip_len, n_clips, 6, 1, [79, 0, 40], out_dtype="f32")
        assert_tile_kernel(info, clip_len, n_clips, P, 1)
        # fp32 scores of size 100: an absolute error of up to 64 products' roundings at that size
        # (2^-24 * 100 each, as a random walk) enters the weights relatively
        bar = 1e-5 + 8 * 100 * 2.0 ** -24 * float(v.float().abs().max())
        assert float(np.abs(o.double().cpu().numpy() - ref).max()) <= bar


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_materialised_context_gives_the_same(dtype):
    for (clip_len, n_clips, w, P, h, D, G, kw) in [(24, 3, 5, 3, 2, 40, 10, {}),
                                                   (20, 3, 2, 3, 1, 160, 33, {"window": 3})]:
        F = clip_len * n_clips
        g = np.random.default_rng(6).integers(0, F, size=G).tolist()
        q, k, v = make(F, P, h * D, dtype)
        plan = B.dsattn_plan(clip_len, n_clips, w, P, h, D, g, io_dtype=U.dt_code(dtype), **kw)
        assert_tile_kernel(B.dsattn_plan_launch_info(plan), clip_len, n_clips, P, h)
        o1, o2 = torch.empty_like(q), torch.empty_like(q)
        B.dsattn_forward(plan, q, k, v, o1)
        ctx = [torch.full((n_clips, plan.lk_max, P, h * D), float("nan"), dtype=q.dtype, device=DEV)
               for _ in range(2)]
        B.dsattn_gather_context(plan, k, v, *ctx)
        B.dsattn_forward_ctx(plan, q, *ctx, o2)
        torch.cuda.synchronize()
        assert torch.equal(o1, o2)
        plan.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_non_finite_values_go_where_the_generic_kernel_puts_them(dtype):
    clip_len, n_clips, w, P, h, D, g = 24, 3, 2, 3, 2, 40, [5, 70, 33]
    F = clip_len * n_clips
    for which, frame, bad in [("v", 10, float("inf")), ("v", 71, float("-inf")), ("v", 33, float("nan")),
                              ("k", 10, float("inf")), ("k", 70, float("nan")), ("q", 30, float("inf")),
                              ("q", 30, float("nan")), ("k", 12, float("-inf"))]:
        t = dict(zip("qkv", make(F, P, h * D, dtype)))
        t[which][frame, 1, 45] = bad                 # position 1, head 1, channel 5
        o, info = U.library_forward(t["q"], t["k"], t["v"], clip_len, n_clips, w, h, g, out_dtype="f32")
        assert_tile_kernel(info, clip_len, n_clips, P, h)
        og, info = U.library_forward(t["q"], t["k"], t["v"], clip_len, n_clips, w, h, g, out_dtype="f32",
                                     flags=B.DSATTN_FLAG_FORCE_GENERIC)
        assert_generic_kernel(info, n_clips, P, h)
        finite = torch.isfinite(og)
        assert torch.equal(torch.isfinite(o), finite), (which, frame, bad)
        assert torch.equal(torch.isnan(o), torch.isnan(og)) and torch.equal(o == float("inf"), og == float("inf"))
        assert float((o - og)[finite].abs().max()) <= 2e-5


def test_tile_kernel_in_hip_graph_replays():
    clip_len, n_clips, w, P, h, D, g = 24, 3, 2, 5, 2, 64, [5, 70, 33]
    q, k, v = make(72, P, h * D, "bf16")
    plan = B.dsattn_plan(clip_len, n_clips, w, P, h, D, g)
    assert_tile_kernel(B.dsattn_plan_launch_info(plan), clip_len, n_clips, P, h)
    want, o = torch.empty_like(q), torch.zeros_like(q)
    B.dsattn_forward(plan, q, k, v, want)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.dsattn_forward(plan, q, k, v, o)
    for _ in range(3):
        o.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(o, want)
    plan.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("bias", [(-1e3, 0.0), (-1e4, 0.0), (-1e9, 0.0), (-3e38, 0.0), (0.0, -1e9),
                                  (0.0, 1e9), (1e9, 0.0), (2e9, 1e9), (-3e38, -3e38),
                                  (-2e38, -3e38)])
def test_scopes_far_apart_keep_the_heavier_ones_scores(bias, dtype):
    """A scope damped or switched off by its bias leaves the other scope's scores as they are: the
    difference of the biases is taken from the lighter scope, never added to the heavier one, where
    it would drown the scores.  (The last two: beside a bias of 1e38 the oracle's 64 bits hold no score
    either.)"""
    clip_len, n_clips, w, P, h, D, G = 24, 3, 2, 3, 2, 64, 12
    F = clip_len * n_clips
    g = np.random.default_rng(8).integers(0, F, size=G).tolist()
    q, k, v = make(F, P, h * D, dtype)
    kw = dict(bias_local=float(np.float32(bias[0])), bias_global=float(np.float32(bias[1])))
    ref = U.oracle_forward(q, k, v, clip_len, n_clips, w, h, g, **kw)
    o, info = U.library_forward(q, k, v, clip_len, n_clips, w, h, g, out_dtype="f32", **kw)
    assert_tile_kernel(info, clip_len, n_clips, P, h)
    U.assert_parity(o, ref, "f32_strict", what=f"biases {bias}")
    # no global scope at all, and one that the set union hides from every query of the middle clip
    for g, dedup in (([], False), ([24, 30, 47, 30], True)):
        # (with the heavier scope hidden, the oracle's 64 bits hold the scores beside -1e9, not -3e38)
        ro = dict(kw, bias_local=-1e9) if dedup and bias == (-3e38, 0.0) else kw
        ref = U.oracle_forward(q, k, v, clip_len, n_clips, w, h, g, dedup=dedup, **ro)
        o, info = U.library_forward(q, k, v, clip_len, n_clips, w, h, g, out_dtype="f32",
                                    flags=B.DSATTN_FLAG_DEDUP_GLOBAL if dedup else 0, **kw)
        assert_tile_kernel(info, clip_len, n_clips, P, h)
        U.assert_parity(o, ref, "f32_strict", what=f"biases {bias} G={g}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("clip_len", [3, 40])
def test_an_infinity_in_v_meets_small_weights(clip_len, dtype):
    """The smallest weights are not zero beside an infinity: infinite as in the generic kernel, where
    the weight is subnormal (90 to 102 below the others' scores) or a part of it would be (84).  At 110 the
    generic kernel's weight is zero, and zero times infinity is NaN; the fp32 tile kernel's never is.
    Finite values are off by at most 2^-126 of themselves, the weights below the smallest normal number."""
    n_clips, P, D = 1, 2, 64
    for below in (84.0, 90.0, 96.0, 102.0, 110.0):
        q = torch.ones(clip_len, P, D, device=DEV)
        k = torch.zeros(clip_len, P, D, device=DEV)
        k[-1] = -below / 8.0
        for special in (float("inf"), float("-inf"), 1e38, -2e38):
            v = torch.linspace(-1.0, 1.0, clip_len, device=DEV)[:, None, None].repeat(1, P, D)
            v[-1, 0, 5] = special
            t = [x.to(synth.torch_dtype(dtype)) for x in (q, k, v)]
            o, info = U.library_forward(*t, clip_len, n_clips, 0, 1, [], out_dtype="f32")
            assert_tile_kernel(info, clip_len, n_clips, P, 1)
            og, _ = U.library_forward(*t, clip_len, n_clips, 0, 1, [], out_dtype="f32",
                                      flags=B.DSATTN_FLAG_FORCE_GENERIC)
            if np.isinf(special):
                for x, nan in ((o, below > 104.0 and dtype == "bf16"), (og, below > 104.0)):
                    assert (x[:, 0, 5].isnan() if nan else x[:, 0, 5] == special).all(), (below, special)
                o[:, 0, 5] = og[:, 0, 5] = 0.0
            # (the exponent, of size 120 to 160 in base 2, is rounded to 2^-17 of its unit in both kernels)
            big = 0.0 if np.isinf(special) else abs(special)
            bar = 2e-5 + big * (2.0 ** -126 + 2 * 2.0 ** -17 * np.exp(-below))
            assert float((o.double() - og.double()).abs().max()) <= bar, (below, special)


@pytest.mark.parametrize("D,h", [(40, 2), (160, 1), (72, 3)])
@pytest.mark.parametrize("opts", [{}, {"window": 4, "dedup": True}, {"bias_global": 2.0, "dedup": True},
                                  {"bias_local": 3.0, "window": 0}, {"bias_global": 1e9, "dedup": True}])
def test_tasks_with_infinities_are_done_again_with_every_option(opts, D, h):
    """Infinities of both signs in one channel of V send every bf16 task of their head through the second
    pass: that channel is NaN, all others are the generic kernel's numbers, on the tensors and on a
    materialised context."""
    clip_len, n_clips, w, P = 24, 4, 5, 2
    F = clip_len * n_clips
    g = np.random.default_rng(9).integers(0, F, size=80).tolist()
    opts = dict(opts)
    flags = B.DSATTN_FLAG_DEDUP_GLOBAL if opts.pop("dedup", False) else 0
    q, k, v = make(F, P, h * D, "bf16")
    v[0::2, :, D - 1], v[1::2, :, D - 1] = float("inf"), float("-inf")
    for out in ("f32", "bf16"):
        o, info = U.library_forward(q, k, v, clip_len, n_clips, w, h, g, out_dtype=out, flags=flags, **opts)
        assert_tile_kernel(info, clip_len, n_clips, P, h)
        og, _ = U.library_forward(q, k, v, clip_len, n_clips, w, h, g, out_dtype=out,
                                  flags=flags | B.DSATTN_FLAG_FORCE_GENERIC, **opts)
        assert o[:, :, D - 1].isnan().all() and og[:, :, D - 1].isnan().all()
        keep = [c for c in range(h * D) if c != D - 1]
        a, b = o[:, :, keep].double(), og[:, :, keep].double()
        if opts.get("bias_global") == 1e9:      # (the generic kernel adds the bias to the scores that count)
            vz = v.clone()
            vz[:, :, D - 1] = 0.0
            ref = U.oracle_forward(q, k, vz, clip_len, n_clips, w, h, g, dedup=bool(flags), **opts)
            b = torch.from_numpy(ref).to(DEV)[:, :, keep]
        bar = 2e-5 + (0 if out == "f32" else 2 * U.bf16_half_ulp(b.cpu().numpy()).max())
        assert float((a - b).abs().max()) <= bar
    plan = B.dsattn_plan(clip_len, n_clips, w, P, h, D, g, flags=flags, **opts)
    ctx = [torch.empty(n_clips, plan.lk_max, P, h * D, dtype=q.dtype, device=DEV) for _ in range(2)]
    o2 = torch.empty_like(q)
    B.dsattn_gather_context(plan, k, v, *ctx)
    B.dsattn_forward_ctx(plan, q, *ctx, o2)
    torch.cuda.synchronize()
    plan.close()
    assert torch.equal(o2[:, :, keep], o[:, :, keep])


@pytest.mark.parametrize("D,h", [(40, 2), (160, 1), (96, 2), (32, 2)])
@pytest.mark.parametrize("opts", [{"dedup": True}, {"dedup": True, "bias_local": 2.0}, {"bias_global": 2.0}, {"window": 4}])
def test_tasks_with_infinities_are_done_again_by_the_kernels_of_one_option(opts, D, h):
    """The same with 19 global frames: the kernels for the set union, for biases and for a window alone."""
    clip_len, n_clips, w, P = 24, 4, 5, 2
    F = clip_len * n_clips
    g = np.random.default_rng(9).integers(0, F, size=19).tolist()
    opts = dict(opts)
    flags = B.DSATTN_FLAG_DEDUP_GLOBAL if opts.pop("dedup", False) else 0
    q, k, v = make(F, P, h * D, "bf16")
    v[0::2, :, D - 1], v[1::2, :, D - 1] = float("inf"), float("-inf")
    keep = [c for c in range(h * D) if c != D - 1]
    for out in ("f32", "bf16"):
        print(f"[case] infinities D={D} {opts} flags={flags} out={out}", flush=True)
        o, info = U.library_forward(q, k, v, clip_len, n_clips, w, h, g, out_dtype=out, flags=flags, **opts)
        assert_tile_kernel(info, clip_len, n_clips, P, h)
        og, _ = U.library_forward(q, k, v, clip_len, n_clips, w, h, g, out_dtype=out,
                                  flags=flags | B.DSATTN_FLAG_FORCE_GENERIC, **opts)
        assert o[:, :, D - 1].isnan().all() and og[:, :, D - 1].isnan().all()
        a, b = o[:, :, keep].double(), og[:, :, keep].double()
        bar = 2e-5 + (0 if out == "f32" else 2 * U.bf16_half_ulp(b.cpu().numpy()).max())
        assert float((a - b).abs().max()) <= bar


BRANCHES = [
    # clip_len, n_clips, w, P, h, D, G, options: clips that fill no query tile
    (8, 5, 6, 3, 2, 64, 4, {}),
    (5, 7, 3, 2, 2, 40, 9, {"window": 2, "dedup": True}),
    (3, 11, 9, 2, 1, 96, 5, {"bias_global": 1.5}),
    (2, 3, 1, 2, 1, 16, 0, {"bias_local": 1.0}),
    # more global entries than the table in LDS holds, and exactly as many
    (24, 12, 2, 1, 1, 32, 257, {"dedup": True}),
    (24, 12, 2, 1, 1, 160, 256, {"bias_local": -1.0, "dedup": True}),
    (40, 8, 2, 1, 1, 64, 300, {}),
    # few thousand query tiles: the second one of a clip nearly empty, full; the third, the fifth
    (17, 8, 2, 131, 2, 32, 5, {"two": ["f32"]}),
    (32, 8, 1, 129, 2, 128, 16, {"two": ["f32"]}),
    (48, 5, 0, 139, 2, 64, 3, {}),
    (80, 4, 5, 103, 2, 104, 7, {}),
    # two query tiles per wavefront: the second nearly empty, full, absent from the last wavefront
    (17, 8, 2, 1283, 2, 32, 5, {"two": ["f32", "bf16"]}),
    (32, 8, 1, 389, 2, 128, 16, {"two": ["f32", "bf16"]}),
    (48, 5, 0, 1231, 2, 40, 3, {"two": ["bf16"]}),
    (80, 4, 5, 311, 2, 104, 7, {"two": ["bf16"]}),
    (17, 30, 2, 70, 16, 104, 3, {"two": ["f32", "bf16"]}),
    (24, 12, 2, 515, 2, 64, 20, {"two": ["f32", "bf16"]}),
    (24, 12, 2, 260, 2, 40, 21, {"two": ["f32", "bf16"]}),
    # a window that hides most of a long clip
    (100, 2, 12, 2, 1, 72, 11, {"window": 3, "dedup": True}),
    (100, 2, 12, 2, 1, 136, 0, {"window": 40}),
    # one to five key tiles, the last one full and of one key; odd and even in one launch
    (4, 3, 0, 2, 2, 64, 12, {}),
    (4, 3, 0, 2, 2, 64, 13, {"bias_global": -1.0}),
    (4, 8, 0, 3, 1, 160, 28, {"dedup": True}),
    (4, 8, 0, 3, 1, 160, 29, {}),
    (24, 4, 0, 2, 1, 80, 24, {}),
    (24, 4, 0, 2, 1, 80, 25, {"window": 5}),
    (8, 5, 4, 2, 1, 128, 17, {"bias_local": 1.0}),
    (40, 3, 12, 2, 1, 40, 9, {"window": 7, "dedup": True}),
    (24, 12, 2, 100, 2, 64, 20, {"two": ["f32"]}),
    (24, 12, 2, 100, 2, 40, 21, {"two": ["f32"]}),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", BRANCHES)
def test_tile_kernel_branches_match_oracle_on_both_sources(case, dtype):
    """The forms that the launch chooses between, on the tensors and on a materialised context."""
    clip_len, n_clips, w, P, h, D, G, opts = case
    print(f"[case] tile branch {case} {dtype}", flush=True)
    F = clip_len * n_clips
    g = np.random.default_rng(15).integers(0, F, size=G).tolist()
    q, k, v = make(F, P, h * D, dtype, seed=23)
    opts = dict(opts)
    dedup = opts.pop("dedup", False)
    two = dtype in opts.pop("two", [])
    pos = list(range(P)) if P <= 200 else sorted({*range(0, P, P // 40), P - 1})
    ref = U.oracle_forward(q, k, v, clip_len, n_clips, w, h, g, dedup=dedup, positions=pos, **opts)
    plan = B.dsattn_plan(clip_len, n_clips, w, P, h, D, g, io_dtype=U.dt_code(dtype), out_dtype=B.DSATTN_F32,
                         flags=B.DSATTN_FLAG_DEDUP_GLOBAL if dedup else 0, **opts)
    assert_tile_kernel(B.dsattn_plan_launch_info(plan), clip_len, n_clips, P, h, 2 if two else 1)
    o1 = torch.full((F, P, h * D), float("nan"), device=DEV)
    o2 = o1.clone()
    B.dsattn_forward(plan, q, k, v, o1)
    ctx = [torch.full((n_clips, plan.lk_max, P, h * D), float("nan"), dtype=q.dtype, device=DEV) for _ in range(2)]
    B.dsattn_gather_context(plan, k, v, *ctx)
    B.dsattn_forward_ctx(plan, q, *ctx, o2)
    torch.cuda.synchronize()
    plan.close()
    U.assert_parity(o1, ref, "f32_strict", positions=pos, what=f"{case} on the tensors")
    assert torch.equal(o1, o2)                               # (a NaN is equal to none)


@pytest.mark.parametrize("D", list(range(4, 161, 12)))
def test_every_fp32_row_shape(D):
    """Blocks of 64, 32 and 16 channels, the last one full or not."""
    q, k, v = make(40, 2, 2 * D, "f32", seed=31)
    ref = U.oracle_forward(q, k, v, 20, 2, 3, 2, [39, 3])
    o, info = U.library_forward(q, k, v, 20, 2, 3, 2, [39, 3], out_dtype="f32")
    assert_tile_kernel(info, 20, 2, 2, 2)
    U.assert_parity(o, ref, "f32_strict", what=f"D={D}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_scores_of_minus_infinity_in_the_first_tiles(dtype):
    """Keys whose scores are -inf have no weight, also where they fill the first step."""
    q, k, v = make(40, 2, 64, dtype, seed=37)
    q = (q.abs() + 0.1).to(q.dtype)
    k[:32, 1, 5] = float("-inf")
    o, _ = U.library_forward(q, k, v, 40, 1, 0, 1, [], out_dtype="f32")
    og, _ = U.library_forward(q, k, v, 40, 1, 0, 1, [], out_dtype="f32", flags=B.DSATTN_FLAG_FORCE_GENERIC)
    assert torch.isfinite(og).all() and float((o - og).abs().max()) <= 2e-5
