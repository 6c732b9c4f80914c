"""Clip-parallel group normalisation (Section 4.2): boundary checks on the CPU, parity of the HIP
kernels against the oracle on the GPU."""
import ctypes

import numpy as np
import pytest
import torch

import parity_util as U
from oracle import oracle
from paper_2406_16260_amd import binding as B
from paper_2406_16260_amd import synth

DEV = "cuda:0"


# ---------------------------------------------------------------- CPU: validation only

def raw_desc(**kw):
    d = dict(clip_len=4, n_clips=3, spatial=5, channels=64, groups=4, io_dtype=B.DSATTN_BF16,
             eps=1e-5)
    d.update(kw)
    return B.DsattnGnDesc(**d)


@pytest.mark.parametrize("kw,code", [
    (dict(clip_len=0), B.DSATTN_EINVAL), (dict(n_clips=0), B.DSATTN_EINVAL),
    (dict(spatial=0), B.DSATTN_EINVAL), (dict(channels=0), B.DSATTN_EINVAL),
    (dict(groups=0), B.DSATTN_EINVAL), (dict(groups=5), B.DSATTN_EINVAL),
    (dict(io_dtype=3), B.DSATTN_EINVAL), (dict(eps=-1.0), B.DSATTN_EINVAL),
    (dict(eps=float("nan")), B.DSATTN_EINVAL),
    (dict(channels=16, groups=4), B.DSATTN_EUNSUPPORTED),     # 4 channels per group < one lane
    (dict(channels=36, groups=3), B.DSATTN_EUNSUPPORTED),     # rows are not whole 16-byte lanes
    (dict(channels=16384, groups=1), B.DSATTN_EUNSUPPORTED),  # more than 1024 lanes per row
])
def test_groupnorm_rejects_bad_descriptors(kw, code):
    lib = B.load()
    out = ctypes.c_size_t()
    d = raw_desc(**kw)
    assert lib.dsattn_groupnorm_workspace(ctypes.byref(d), ctypes.byref(out)) == code
    assert lib.dsattn_groupnorm(ctypes.byref(d), 0x1000, None, None, 0x2000, None, 0x3000, 1 << 20,
                                None) == code


def test_groupnorm_argument_checks_before_launch():
    lib = B.load()
    d = raw_desc()
    out = ctypes.c_size_t()
    assert lib.dsattn_groupnorm_workspace(ctypes.byref(d), ctypes.byref(out)) == B.DSATTN_OK
    need = out.value
    assert need >= (3 * 4 + 2 * 4) * 4
    assert lib.dsattn_groupnorm_workspace(None, ctypes.byref(out)) == B.DSATTN_EINVAL
    assert lib.dsattn_groupnorm_workspace(ctypes.byref(d), None) == B.DSATTN_EINVAL
    ok = (0x1000, None, None, 0x2000, None, 0x3000, need, None)
    assert lib.dsattn_groupnorm(ctypes.byref(d), None, *ok[1:]) == B.DSATTN_EINVAL
    assert lib.dsattn_groupnorm(ctypes.byref(d), 0x1004, *ok[1:]) == B.DSATTN_EINVAL   # misaligned
    assert lib.dsattn_groupnorm(ctypes.byref(d), 0x1000, None, None, 0x2000, None, None, need,
                                None) == B.DSATTN_EINVAL                                # no workspace
    assert lib.dsattn_groupnorm(ctypes.byref(d), 0x1000, None, None, 0x2000, None, 0x3000,
                                need - 1, None) == B.DSATTN_EINVAL                      # too small
    assert "workspace" in B.dsattn_last_error()


# ---------------------------------------------------------------- GPU: parity

def run_gn(x, clip_len, n_clips, groups, gamma=None, beta=None, eps=1e-5, in_place=False):
    F, P, C = x.shape
    dt = U.dt_code("f32" if x.dtype == torch.float32 else "bf16")
    nbytes = B.dsattn_groupnorm_workspace(clip_len, n_clips, P, C, groups, io_dtype=dt, eps=eps)
    ws = torch.empty((nbytes + 3) // 4, dtype=torch.float32, device=x.device)
    y = x if in_place else torch.full_like(x, float("nan"))
    stats = torch.full((2 * groups,), float("nan"), dtype=torch.float32, device=x.device)
    B.dsattn_groupnorm(clip_len, n_clips, P, C, groups, x, y, ws, nbytes, gamma=gamma, beta=beta,
                       stats=stats, io_dtype=dt, eps=eps)
    torch.cuda.synchronize()
    return y, stats


GN_SHAPES = [
    # clip_len, n_clips, P, C, groups, dtype
    (4, 3, 5, 64, 4, "bf16"),
    (16, 4, 7, 320, 8, "bf16"),
    (16, 4, 7, 320, 32, "bf16"),      # 10 channels per group: lanes straddle group boundaries
    (4, 6, 5, 640, 32, "bf16"),       # 20 channels per group
    (2, 3, 9, 48, 4, "bf16"),         # 12 channels per group
    (3, 4, 6, 36, 6, "f32"),          # 6 channels per group, 4-channel lanes
    (1, 9, 3, 1280, 32, "bf16"),      # one frame per clip
    (5, 1, 2, 8192, 1, "bf16"),       # 1024 lanes per row, one workgroup row
    (3, 4, 6, 24, 3, "f32"),
    (2, 2, 1, 4, 1, "f32"),           # a single lane per row
    (8, 3, 11, 640, 32, "f32"),
]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", GN_SHAPES)
def test_groupnorm_matches_oracle(shape):
    clip_len, n_clips, P, C, groups, dtype = shape
    print(f"[case] groupnorm {shape}", flush=True)
    F = clip_len * n_clips
    x = synth.make_tensor(F, P, C, 5, "iid", dtype)
    # clips with different means and scales
    x = (x.float() * (1.0 + torch.arange(F)[:, None, None] / F) +
         0.5 * torch.sin(torch.arange(F, dtype=torch.float32))[:, None, None]).to(x.dtype).to(DEV)
    gen = torch.Generator().manual_seed(3)
    gamma = torch.randn(C, generator=gen).to(DEV)
    beta = torch.randn(C, generator=gen).to(DEV)
    xs = x.to("cpu").to(torch.float64).numpy()
    ref, mean, var = oracle.groupnorm(xs, clip_len, n_clips, groups, eps=1e-5,
                                      gamma=gamma.cpu().double().numpy(),
                                      beta=beta.cpu().double().numpy())
    y, stats = run_gn(x, clip_len, n_clips, groups, gamma, beta)
    st = stats.cpu().double().numpy()
    np.testing.assert_allclose(st[:groups], mean, rtol=0, atol=2e-6)
    np.testing.assert_allclose(st[groups:], 1.0 / np.sqrt(var + 1e-5), rtol=3e-6, atol=0)
    U.assert_parity(y, ref, "f32_strict" if dtype == "f32" else "bf16", what=f"groupnorm {shape}")
    # no affine parameters, in place
    ref2, _, _ = oracle.groupnorm(xs, clip_len, n_clips, groups, eps=1e-5)
    y2, _ = run_gn(x.clone(), clip_len, n_clips, groups, in_place=True)
    U.assert_parity(y2, ref2, "f32_strict" if dtype == "f32" else "bf16", what="groupnorm in place")


@pytest.mark.gpu
def test_groupnorm_partition_independent_and_deterministic():
    F, P, C, groups = 48, 9, 320, 8
    x = synth.make_tensor(F, P, C, 7, "correlated", "bf16").to(DEV)
    ys = [run_gn(x, cl, F // cl, groups)[0] for cl in (16, 4, 48, 1)]
    ref, _, _ = oracle.groupnorm(x.cpu().double().numpy(), 16, 3, groups)
    for y in ys:
        U.assert_parity(y, ref, "bf16", what="groupnorm partition")
    again = run_gn(x, 16, 3, groups)[0]
    assert torch.equal(again, ys[0])


@pytest.mark.gpu
def test_groupnorm_full_size_level():
    # the headline level's tensor: 2,304 frames x 160 positions x 1,280 channels, 32 groups
    wl = synth.WORKLOADS["C3"]
    lv = wl.levels[0]
    x = synth.make_tensor(wl.F, lv.P, lv.C, 11, "correlated", "bf16", device=DEV)
    y, stats = run_gn(x, wl.clip_len, wl.n_clips, 32)
    # statistics against a library reduction on the device (fp64), outputs on sampled positions
    xg = x.view(wl.F, lv.P, 32, lv.C // 32).double()
    mean = xg.mean(dim=(0, 1, 3))
    var = xg.var(dim=(0, 1, 3), unbiased=False)
    assert (stats[:32].double() - mean).abs().max().item() < 2e-6
    assert ((stats[32:].double() * torch.sqrt(var + 1e-5)) - 1).abs().max().item() < 3e-6
    pos = [0, 53, 159]
    ref = ((xg[:, pos] - mean[None, None, :, None]) / torch.sqrt(var + 1e-5)[None, None, :, None])
    ref = ref.reshape(wl.F, len(pos), lv.C).cpu().numpy()
    U.assert_parity(y, ref, "bf16", positions=pos, what="groupnorm full size")


@pytest.mark.gpu
def test_groupnorm_level_sized_tensor_against_the_oracle():
    # a whole level-sized tensor (the 64-frame workload's level: 64 x 2,560 x 320, 32 groups)
    # checked element by element against the oracle itself, statistics included
    wl = synth.WORKLOADS["C1"]
    lv = wl.levels[0]
    print(f"[case] groupnorm {wl.F} x {lv.P} x {lv.C} vs oracle", flush=True)
    x = synth.make_tensor(wl.F, lv.P, lv.C, 13, "correlated", "bf16", device=DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(14)
    gamma = 1.0 + 0.1 * torch.randn(lv.C, generator=gen, device=DEV)
    beta = 0.1 * torch.randn(lv.C, generator=gen, device=DEV)
    y, stats = run_gn(x, wl.clip_len, wl.n_clips, 32, gamma=gamma, beta=beta)
    ref, mean, var = oracle.groupnorm(x.cpu().double().numpy(), wl.clip_len, wl.n_clips, 32,
                                      gamma=gamma.cpu().double().numpy(),
                                      beta=beta.cpu().double().numpy())
    st = stats.cpu().double().numpy()
    np.testing.assert_allclose(st[:32], mean, rtol=0, atol=2e-6)
    np.testing.assert_allclose(st[32:], 1.0 / np.sqrt(var + 1e-5), rtol=3e-6, atol=0)
    U.assert_parity(y, ref, "bf16", what="groupnorm level-sized vs oracle")


@pytest.mark.gpu
@pytest.mark.parametrize("offset", [100.0, -3000.0])
def test_groupnorm_large_means_do_not_cancel(offset):
    """Means far larger than the deviations (fp32 tensors, |mean| / std up to 3,000): the one-pass
    statistics keep their accuracy because every partial sum is taken about a nearby pilot."""
    clip_len, n_clips, P, C, groups = 4, 5, 33, 64, 8
    F = clip_len * n_clips
    gen = torch.Generator().manual_seed(4)
    x = (torch.randn(F, P, C, generator=gen) + offset +
         0.25 * torch.arange(F, dtype=torch.float32)[:, None, None]).to(DEV)
    ref, mean, var = oracle.groupnorm(x.cpu().double().numpy(), clip_len, n_clips, groups, eps=1e-5)
    y, stats = run_gn(x, clip_len, n_clips, groups)
    st = stats.cpu().double().numpy()
    # the mean is held to fp32 resolution at its own size, the variance to a few 1e-6 relative
    np.testing.assert_allclose(st[:groups], mean, rtol=2e-7, atol=0)
    np.testing.assert_allclose(st[groups:], 1.0 / np.sqrt(var + 1e-5), rtol=1e-5, atol=0)
    # y = (x - mean) * rstd: the subtraction of two fp32 numbers of size |offset| costs up to
    # one ulp of them, relative to a spread of order one
    err = np.abs(y.cpu().double().numpy() - ref).max()
    assert err <= 4 * abs(offset) * 2.0 ** -24 + 1e-5, err


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [
    # clip_len, n_clips, P, C, groups, dtype
    (1, 50, 1, 64, 4, "bf16"),        # fewer bites of rows than clips: one workgroup reads, not fifty
    (1, 300, 7, 512, 8, "f32"),       # more bites than the statistics pass has workgroups, last one partial
    (16, 5, 401, 320, 32, "bf16"),    # 20.5 MB: plain loads and stores, last bite partial
    (16, 8, 401, 328, 41, "bf16"),    # 33.7 MB: streaming loads and stores, a lane is a group
    (7, 9, 211, 640, 32, "f32"),      # 34.0 MB
])
def test_groupnorm_walks_cover_every_row(shape):
    """The passes walk the whole video in interleaved bites of rows (the second one backwards):
    sizes around the changes of their launch shape, with affine parameters, held to the bars of
    test_groupnorm_matches_oracle."""
    clip_len, n_clips, P, C, groups, dtype = shape
    print(f"[case] groupnorm walk {shape}", flush=True)
    F = clip_len * n_clips
    x = synth.make_tensor(F, P, C, 15, "iid", dtype)
    x = (x.float() + 0.01 * torch.arange(F, dtype=torch.float32)[:, None, None]).to(x.dtype).to(DEV)
    gen = torch.Generator().manual_seed(16)
    gamma, beta = torch.randn(C, generator=gen).to(DEV), torch.randn(C, generator=gen).to(DEV)
    ref, mean, var = oracle.groupnorm(x.cpu().double().numpy(), clip_len, n_clips, groups, eps=1e-5,
                                      gamma=gamma.cpu().double().numpy(),
                                      beta=beta.cpu().double().numpy())
    for in_place in (False, True):
        y, stats = run_gn(x.clone(), clip_len, n_clips, groups, gamma, beta, in_place=in_place)
        st = stats.cpu().double().numpy()
        np.testing.assert_allclose(st[:groups], mean, rtol=0, atol=2e-6)
        np.testing.assert_allclose(st[groups:], 1.0 / np.sqrt(var + 1e-5), rtol=3e-6, atol=0)
        U.assert_parity(y, ref, "f32_strict" if dtype == "f32" else "bf16", what=f"walk {shape}")


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_groupnorm_non_finite_values_stay_in_their_group(dtype):
    clip_len, n_clips, P, C, groups = 4, 3, 11, 80, 4   # 20 channels per group: lanes straddle
    x = synth.make_tensor(12, P, C, 21, "iid", dtype).to(DEV)
    clean, _ = run_gn(x.clone(), clip_len, n_clips, groups)
    for bad in (float("nan"), float("inf")):
        z = x.clone()
        z[5, 3, 27] = bad                               # group 1
        y, stats = run_gn(z, clip_len, n_clips, groups)
        assert torch.isnan(stats[groups + 1]) and not torch.isnan(stats[groups + 0])
        assert torch.isnan(y[:, :, 20:40]).all()
        keep = [c for c in range(C) if not 20 <= c < 40]
        assert torch.equal(y[:, :, keep], clean[:, :, keep])
    # a constant group: variance exactly zero
    y, stats = run_gn(torch.full_like(x, 3.5), clip_len, n_clips, groups, eps=0.25)
    assert torch.equal(stats, torch.tensor([3.5] * groups + [2.0] * groups, device=DEV))
    assert not y.any()


@pytest.mark.gpu
def test_groupnorm_long_sums_keep_fp32_statistics():
    """576,000 rows, some 100 to 500 a thread: 1 / sigma within four roundings of an fp32 number (a single
    fp32 sum per thread was off by 4.3e-7 here, sums of 32 rows by 0.9e-7)."""
    F_clip, N, P, C = 24, 80, 300, 320
    torch.manual_seed(0)
    x = (torch.randn(1, P, C, device="cuda")
         + 0.1 * torch.randn(F_clip * N, P, C, device="cuda")).to(torch.bfloat16)
    y, stats = torch.empty_like(x), torch.empty(2, 32, device="cuda")
    n = B.dsattn_groupnorm_workspace(F_clip, N, P, C, 32)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    B.dsattn_groupnorm(F_clip, N, P, C, 32, x, y, ws, n, stats=stats)
    for g in range(0, 32, 8):
        xd = x[:, :, g * 10:g * 10 + 10].double()
        want = 1.0 / torch.sqrt(((xd - xd.mean()) ** 2).mean() + 1e-5)
        assert abs(stats[1, g].item() / want.item() - 1.0) <= 4 * 2.0 ** -24


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("sigma", [3e17, 1e-21])
def test_groupnorm_spreads_at_the_ends_of_the_range(sigma, dtype):
    """Sums of squared deviations beyond fp32's range, and below it, in one workgroup: no single
    square leaves the range, so the statistics are right.  8,192 elements a workgroup and group, about
    7e38 and 8e-39 in sum.  Bound at the lower end: 64 squares of 1e-42 are each rounded to a multiple of
    2^-149, 0.14 % of one; their average is off by less."""
    clip_len, n_clips, P, C, groups = 16, 16, 64, 512, 4
    x = synth.make_tensor(clip_len * n_clips, P, C, 33, "iid", "f32")
    x = (x * sigma).to(synth.torch_dtype(dtype)).to(DEV)
    eps = 0.0
    ref, mean, var = oracle.groupnorm(x.cpu().double().numpy(), clip_len, n_clips, groups, eps=eps)
    y, stats = run_gn(x, clip_len, n_clips, groups, eps=eps)
    st = stats.cpu().double().numpy()
    rtol = 3e-6 if sigma > 1 else 1.4e-3
    np.testing.assert_allclose(st[groups:], 1.0 / np.sqrt(var), rtol=rtol, atol=0)
    np.testing.assert_allclose(st[:groups], mean, rtol=0, atol=2e-6 * sigma)
    err = np.abs(y.cpu().double().numpy() - ref)
    assert (err <= 1e-5 + rtol * np.abs(ref) + (0 if dtype == "f32" else U.bf16_half_ulp(ref))).all()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_groupnorm_affine_factors_meet_the_normalised_value(dtype):
    """gamma multiplies the normalised value: 1 / sigma times gamma alone may leave fp32's range where
    the result does not (a constant tensor with a large gamma, large values with a small one)."""
    clip_len, n_clips, P, C, groups = 4, 3, 11, 64, 4
    gamma = torch.full((C,), 1e37, device=DEV)
    beta = torch.linspace(-1.0, 1.0, C, device=DEV)
    x = torch.full((12, P, C), 3.5, dtype=synth.torch_dtype(dtype), device=DEV)
    y, _ = run_gn(x, clip_len, n_clips, groups, gamma, beta)
    assert torch.equal(y, beta.to(y.dtype).expand_as(y))
    x = (synth.make_tensor(12, P, C, 34, "iid", "f32") * 1e17).to(x.dtype).to(DEV)
    gamma.fill_(3e-26)
    ref, _, _ = oracle.groupnorm(x.cpu().double().numpy(), clip_len, n_clips, groups, eps=1e-5,
                                 gamma=gamma.cpu().double().numpy())
    y, _ = run_gn(x, clip_len, n_clips, groups, gamma)
    # a few roundings of fp32 (the mean's by its own size), and that of a bf16 result
    np.testing.assert_allclose(y.cpu().double().numpy(), ref, atol=8 * 2.0 ** -24 * 3e-26,
                               rtol=8 * 2.0 ** -24 + (2.0 ** -8 if dtype == "bf16" else 0))


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,C,groups", [
    (1, 128, 8),          # one row: a few pairs for 1,024 threads
    (1023, 128, 8),       # the last size of eight pairs a thread less a row
    (1024, 128, 8),       # exactly that size
    (1025, 128, 8),       # the next one
    (2048, 128, 8),       # the last size that one launch takes, and one row more
    (2049, 128, 8),
    (2560, 96, 12),       # the row limits of the two types
    (2561, 96, 12),
    (4096, 64, 8),
    (4097, 64, 8),
    (97, 2048, 8),        # 256 channels per group: the most that one launch takes
    (97, 2064, 8),
    (1228, 2560, 320),    # the most pieces of rows that one launch takes, and a row more
    (1229, 2560, 320),
])
def test_groupnorm_small_tensors_in_one_launch(rows, C, groups, dtype):
    """Sizes around the limits of the single-launch kernel, held to the bars of test_groupnorm_matches_oracle;
    half of the tensor is shifted, so that no part has the whole's mean."""
    check_small(rows, C, groups, dtype)


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [512, 513, 768])
def test_groupnorm_small_groups_of_four_channels(rows):
    """fp32 only: the most pieces of rows that one launch takes of groups of less than eight channels, and more."""
    check_small(rows, 2048, 512, "f32")


def check_small(rows, C, groups, dtype):
    print(f"[case] groupnorm small {rows} {C} {groups} {dtype}", flush=True)
    x = synth.make_tensor(rows, 1, C, 41, "iid", dtype)
    x = (x.float() + (torch.arange(rows) % 2 * 3.0)[:, None, None]).to(x.dtype).to(DEV)
    gen = torch.Generator().manual_seed(4)
    gamma, beta = torch.randn(C, generator=gen).to(DEV), torch.randn(C, generator=gen).to(DEV)
    ref, mean, var = oracle.groupnorm(x.cpu().double().numpy(), rows, 1, groups, eps=1e-5,
                                      gamma=gamma.cpu().double().numpy(), beta=beta.cpu().double().numpy())
    for in_place in (False, True):
        y, stats = run_gn(x.clone(), rows, 1, groups, gamma, beta, in_place=in_place)
        st = stats.cpu().double().numpy()
        np.testing.assert_allclose(st[:groups], mean, rtol=0, atol=2e-6)
        np.testing.assert_allclose(st[groups:], 1.0 / np.sqrt(var + 1e-5), rtol=3e-6, atol=0)
        U.assert_parity(y, ref, "f32_strict" if dtype == "f32" else "bf16", what=f"small {rows} {C}")


@pytest.mark.gpu
@pytest.mark.parametrize("rows,C,groups,dtype", [(4097, 8192, 1024, "bf16"), (2561, 4096, 1024, "f32"),
                                                 (4099, 7936, 992, "bf16")])
def test_groupnorm_as_many_groups_as_lanes(rows, C, groups, dtype):
    """A group per lane at the widest rows, in three launches: the statistics pass's LDS is at its largest.  Held to
    the bars of test_groupnorm_matches_oracle."""
    print(f"[case] groupnorm many groups {rows} {C} {groups} {dtype}", flush=True)
    x = synth.make_tensor(rows, 1, C, 43, "iid", dtype)
    ref, mean, var = oracle.groupnorm(x.double().numpy(), rows, 1, groups, eps=1e-5)
    y, stats = run_gn(x.to(DEV), rows, 1, groups)
    st = stats.cpu().double().numpy()
    np.testing.assert_allclose(st[:groups], mean, rtol=0, atol=2e-6)
    np.testing.assert_allclose(st[groups:], 1.0 / np.sqrt(var + 1e-5), rtol=3e-6, atol=0)
    U.assert_parity(y, ref, "f32_strict" if dtype == "f32" else "bf16", what=f"many groups {rows} {C}")


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("outlier", [1e5, -3e12])
@pytest.mark.parametrize("rows,C,groups", [(1024, 256, 8), (300, 320, 32), (5000, 256, 8)])
def test_groupnorm_one_outlier_rounds_few_sums(rows, C, groups, outlier, dtype):
    """An element far from all others, first or in the middle of its group.  Only the fp32 sums of the one thread that
    takes it as its pilot, or adds it, are rounded at its size.  In one launch they are 16 elements: deviations off by
    2^-24 of it and sums of up to 16 of them by 2^-24 of 1 to 16 times it, 152 times 2^-24 at the most; in three launches
    32 rows of 8, as a random walk sqrt(256) times about 10.  (About one pilot for all elements: off by 2^-24 of it in
    each, 2.8e-4 of the mean's 3 with 1e5 among 32,768; the bar is 5e-5 there.)"""
    for at in (0, rows * C // groups // 2):
        print(f"[case] groupnorm outlier {rows} {C} {groups} {outlier} {at} {dtype}", flush=True)
        cg = C // groups
        x = synth.make_tensor(rows, 1, C, 44, "iid", dtype)
        for g in range(groups):
            x[at // cg, 0, g * cg + at % cg] = outlier
        _, mean, var = oracle.groupnorm(x.double().numpy(), rows, 1, groups, eps=1e-5)
        _, stats = run_gn(x.to(DEV), rows, 1, groups)
        st = stats.cpu().double().numpy()
        n = rows * cg
        np.testing.assert_allclose(st[:groups], mean, rtol=2.0 ** -23, atol=256 * abs(outlier) * 2.0 ** -24 / n)
        np.testing.assert_allclose(st[groups:], 1.0 / np.sqrt(var + 1e-5), rtol=3e-6, atol=0)
