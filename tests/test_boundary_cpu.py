"""CPU-side tests of the C-ABI boundary: exported symbols, argument validation,
host-only plans and bit-exact context tables against the oracle.  No kernel is launched."""
import ctypes
import os
import re
import struct

import numpy as np
import pytest

from conftest import ROOT, read_golden_ctx_lists
from oracle import oracle
from paper_2406_16260_amd import binding as B
from paper_2406_16260_amd import synth


def declared_functions():
    text = open(os.path.join(ROOT, "include", "dsattn.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(dsattn_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = B.load()
    names = declared_functions()
    assert set(names) == set(B.EXPORTS)
    for n in names:
        assert getattr(lib, n) is not None


def raw_plan(desc_kwargs, gidx, device=-1):
    lib = B.load()
    d = dict(clip_len=4, n_clips=2, local_ctx=1, spatial=16, heads=1, head_dim=8,
             io_dtype=B.DSATTN_F32, out_dtype=B.DSATTN_F32, scale=0.0, flags=0, bias_local=0.0,
             bias_global=0.0, window=0)
    d.update(desc_kwargs)
    desc = B.DsattnDesc(**d)
    g = np.asarray(gidx, dtype=np.int32)
    h = ctypes.c_void_p()
    rc = lib.dsattn_plan(ctypes.byref(desc), g.ctypes.data if g.size else None, g.size, device,
                         ctypes.byref(h))
    return rc, h


@pytest.mark.parametrize("kw,g", [
    (dict(clip_len=0), [0]), (dict(n_clips=0), [0]), (dict(local_ctx=-1), [0]),
    (dict(spatial=0), [0]), (dict(heads=0), [0]), (dict(head_dim=0), [0]),
    (dict(io_dtype=7), [0]), (dict(out_dtype=-1), [0]),
    (dict(io_dtype=B.DSATTN_F32, out_dtype=B.DSATTN_BF16), [0]),
    (dict(scale=float("nan")), [0]), (dict(scale=float("inf")), [0]),
    (dict(bias_local=float("nan")), [0]), (dict(bias_global=float("-inf")), [0]),
    (dict(flags=B.DSATTN_FLAG_SLIDING_WINDOW, window=-1), [0]),
    (dict(), [8]), (dict(), [-1]), (dict(), [0, 3, 99]),
])
def test_plan_rejects_bad_arguments(kw, g):
    rc, h = raw_plan(kw, g)
    assert rc == B.DSATTN_EINVAL
    assert not h.value
    assert B.dsattn_last_error() != ""


def test_plan_null_pointers_and_bad_device():
    lib = B.load()
    h = ctypes.c_void_p()
    assert lib.dsattn_plan(None, None, 0, -1, ctypes.byref(h)) == B.DSATTN_EINVAL
    desc = B.DsattnDesc(4, 2, 1, 16, 1, 8, 0, 0, 0.0, 0)
    assert lib.dsattn_plan(ctypes.byref(desc), None, 0, -1, None) == B.DSATTN_EINVAL
    assert lib.dsattn_plan(ctypes.byref(desc), None, 2, -1, ctypes.byref(h)) == B.DSATTN_EINVAL
    assert lib.dsattn_plan(ctypes.byref(desc), None, -1, -1, ctypes.byref(h)) == B.DSATTN_EINVAL
    assert lib.dsattn_plan(ctypes.byref(desc), None, 0, -2, ctypes.byref(h)) == B.DSATTN_EINVAL
    lib.dsattn_plan_destroy(None)  # must be a no-op
    out = ctypes.c_int32()
    assert lib.dsattn_plan_ctx_max(None, ctypes.byref(out)) == B.DSATTN_EINVAL
    assert lib.dsattn_plan_ctx_indices(None, None, None) == B.DSATTN_EINVAL
    assert lib.dsattn_plan_launch_info(None, None) == B.DSATTN_EINVAL


def test_host_only_plan_refuses_device_work():
    lib = B.load()
    rc, h = raw_plan({}, [0, 4])
    assert rc == B.DSATTN_OK and h.value
    fake = 0x1000  # never dereferenced: validation stops first
    assert lib.dsattn_forward(h, fake, fake, fake, fake, None) == B.DSATTN_ENODEVICE
    assert lib.dsattn_forward_ctx(h, fake, fake, fake, fake, None) == B.DSATTN_ENODEVICE
    assert lib.dsattn_gather_context(h, fake, fake, fake, fake, None) == B.DSATTN_ENODEVICE
    assert lib.dsattn_forward(h, None, fake, fake, fake, None) == B.DSATTN_EINVAL
    assert lib.dsattn_forward(None, fake, fake, fake, fake, None) == B.DSATTN_EINVAL
    lib.dsattn_plan_destroy(h)


def test_copy_probe_validates_before_launch():
    lib = B.load()
    assert lib.dsattn_copy_probe(None, 0x1000, 64, None) == B.DSATTN_EINVAL
    assert lib.dsattn_copy_probe(0x1000, 0x2000, 0, None) == B.DSATTN_EINVAL
    assert lib.dsattn_copy_probe(0x1000, 0x2000, 24, None) == B.DSATTN_EINVAL   # not x16
    assert lib.dsattn_copy_probe(0x1004, 0x2000, 64, None) == B.DSATTN_EINVAL   # misaligned
    assert lib.dsattn_copy_probe(0x1000, 0x1010, 64, None) == B.DSATTN_EINVAL   # overlap


def test_strerror_is_total():
    for code in (0, -1, -2, -3, -4, -5, -77, 5):
        s = B.dsattn_strerror(code)
        assert isinstance(s, str) and s
    assert B.dsattn_strerror(0) == "ok"


@pytest.mark.parametrize("case", read_golden_ctx_lists())
def test_plan_ctx_table_matches_hand_derived(case):
    clip_len, n_clips, w, g, clip, expected = case
    plan = B.dsattn_plan(clip_len, n_clips, w, 1, 1, 8, g, io_dtype=B.DSATTN_F32, device=-1)
    idx, ln = B.dsattn_plan_ctx_indices(plan)
    assert idx[clip, :ln[clip]].tolist() == expected
    plan.close()


@pytest.mark.parametrize("name", ["C0", "C1", "C2", "C3", "C4"])
def test_plan_ctx_table_bit_exact_vs_oracle_on_workloads(name):
    wl = synth.WORKLOADS[name]
    g = synth.global_idx_for(wl)
    assert len(g) == wl.n_global
    lv = wl.levels[0]
    dt = B.DSATTN_F32 if wl.dtype == "f32" else B.DSATTN_BF16
    plan = B.dsattn_plan(wl.clip_len, wl.n_clips, wl.local_ctx, lv.P, lv.heads, lv.head_dim, g,
                         io_dtype=dt, device=-1)
    idx, ln = B.dsattn_plan_ctx_indices(plan)
    ridx, rln = oracle.ctx_indices(wl.clip_len, wl.n_clips, wl.local_ctx, g)
    assert B.dsattn_plan_ctx_max(plan) == ridx.shape[1]
    assert np.array_equal(idx, ridx) and np.array_equal(ln, rln)
    info = B.dsattn_plan_launch_info(plan)
    esz = 4 if wl.dtype == "f32" else 2
    assert info["algorithmic_bytes"] == 4 * wl.F * lv.P * lv.C * esz
    plan.close()


def test_plan_ctx_table_random_shapes_vs_oracle():
    rng = np.random.default_rng(0)
    for _ in range(200):
        clip_len = int(rng.integers(1, 20))
        n_clips = int(rng.integers(1, 12))
        w = int(rng.integers(0, 3 * clip_len + 2))
        F = clip_len * n_clips
        g = rng.integers(0, F, size=int(rng.integers(0, 9))).astype(np.int32)
        plan = B.dsattn_plan(clip_len, n_clips, w, 2, 2, 4, g, io_dtype=B.DSATTN_F32, device=-1)
        idx, ln = B.dsattn_plan_ctx_indices(plan)
        ridx, rln = oracle.ctx_indices(clip_len, n_clips, w, g)
        assert np.array_equal(idx, ridx) and np.array_equal(ln, rln)
        plan.close()


def test_workload_recipes():
    assert synth.stride_global_idx(8, 2).tolist() == [0, 4]
    assert synth.stride_global_idx(64, 16).tolist() == list(range(0, 64, 4))
    assert synth.stride_global_idx(2304, 16).tolist() == list(range(0, 2304, 144))
    g = synth.global_idx_for(synth.WORKLOADS["C4"])
    assert len(g) == 64 and len(set(g.tolist())) == 64 and (np.diff(g) > 0).all()
    assert g.min() >= 0 and g.max() < 2304
    q1 = synth.make_tensor(8, 4, 16, 5, "correlated", "bf16")
    q2 = synth.make_tensor(8, 4, 16, 5, "correlated", "bf16")
    assert (q1 == q2).all()
    # frames are strongly correlated, positions are not
    x = q1.float()
    assert (x[0] - x[7]).abs().mean() < 0.3 and (x[:, 0] - x[:, 1]).abs().mean() > 0.5


# ---------------------------------------------------------------- launch planner (host logic)

def plan_info(wl, lv, **kw):
    g = synth.global_idx_for(wl)
    plan = B.dsattn_plan(wl.clip_len, wl.n_clips, wl.local_ctx, lv.P, lv.heads, lv.head_dim, g,
                         io_dtype=B.DSATTN_F32 if wl.dtype == "f32" else B.DSATTN_BF16, device=-1,
                         **kw)
    info = B.dsattn_plan_launch_info(plan)
    plan.close()
    return info


def test_planner_choices_per_level():
    W = synth.WORKLOADS
    c0 = plan_info(W["C0"], W["C0"].levels[0])            # fp32: the 16-query tile kernel
    assert (c0["kernel"], c0["variant"], c0["block_threads"]) == (0, -1, 256)
    c3 = plan_info(W["C3"], W["C3"].levels[0])
    assert (c3["kernel"], c3["heads_per_wave"], c3["local_tiles"], c3["global_tiles"]) == (1, 1, 2, 1)
    assert c3["block_threads"] == 512 and c3["lds_bytes"] <= 160 * 1024
    assert plan_info(W["C2"], W["C2"].levels[0])["heads_per_wave"] == 2   # 2 x 80 channels per row
    assert plan_info(W["C1"], W["C1"].levels[0])["heads_per_wave"] == 4   # 4 x 40
    for lv in W["C4"].levels:                                             # 64 global frames
        i = plan_info(W["C4"], lv)
        assert i["kernel"] == 1 and i["global_tiles"] == 4 and i["local_tiles"] == 2
        assert i["heads_per_wave"] * lv.head_dim <= 160
    for name in ("C1", "C2", "C3", "C4"):
        for lv in W[name].levels:
            i = plan_info(W[name], lv)
            waves = i["block_threads"] // 64
            row_groups = lv.P * lv.heads // i["heads_per_wave"]
            chunks = -(-W[name].n_clips // i["clips_per_task"])
            assert row_groups % waves == 0
            assert i["n_tasks"] == row_groups * chunks
            assert 1 <= i["clips_per_task"] <= W[name].n_clips


def test_planner_fallbacks_and_overrides(monkeypatch):
    W = synth.WORKLOADS
    lv = W["C3"].levels[0]
    i = plan_info(W["C3"], lv, flags=B.DSATTN_FLAG_FORCE_GENERIC)
    assert (i["kernel"], i["block_threads"]) == (0, 64)
    monkeypatch.setenv("DSATTN_FORCE_GENERIC", "1")
    i = plan_info(W["C3"], lv)
    assert (i["kernel"], i["block_threads"]) == (0, 64)
    monkeypatch.delenv("DSATTN_FORCE_GENERIC")
    monkeypatch.setenv("DSATTN_CLIPS_PER_TASK", "7")
    monkeypatch.setenv("DSATTN_WAVES_PER_BLOCK", "2")
    i = plan_info(W["C3"], lv)
    assert i["clips_per_task"] == 7 and i["block_threads"] == 128
    assert i["n_tasks"] == 1280 * 21
    monkeypatch.delenv("DSATTN_CLIPS_PER_TASK")
    monkeypatch.delenv("DSATTN_WAVES_PER_BLOCK")
    # shapes without a streaming variant run the 16-query tile kernel
    for kw in (dict(clip_len=8), dict(head_dim=48), dict(local_ctx=17), dict(n_global=65)):
        clip_len = kw.get("clip_len", 16)
        g = list(range(kw.get("n_global", 4)))
        plan = B.dsattn_plan(clip_len, 8, kw.get("local_ctx", 2), 4, 2, kw.get("head_dim", 160), g,
                             device=-1)
        i = B.dsattn_plan_launch_info(plan)
        assert (i["kernel"], i["variant"], i["block_threads"]) == (0, -1, 256), kw
        plan.close()
    # and rows that are not whole 16-byte pieces, or heads above 160 channels, the generic kernel
    for D in (36, 168):
        plan = B.dsattn_plan(16, 8, 2, 4, 2, D, [0], device=-1)
        i = B.dsattn_plan_launch_info(plan)
        assert (i["kernel"], i["variant"], i["block_threads"]) == (0, -1, 64), D
        plan.close()


@pytest.mark.parametrize("io,D,positions,tasks,lds", [
    # 24 frames, 12 clips, 5 heads: two query tiles a clip, a wavefront each or, where there are enough, one for both
    (B.DSATTN_BF16, 64, 204, 2, 4 * 32 * (128 + 16) + 1024),
    (B.DSATTN_BF16, 64, 205, 1, 4 * 32 * (128 + 16) + 1024),
    (B.DSATTN_BF16, 40, 103, 1, 4 * 32 * (128 + 16) + 1024),
    (B.DSATTN_BF16, 80, 500, 2, 4 * 32 * (192 + 16) + 1024),
    (B.DSATTN_F32, 64, 34, 2, 4 * 16 * (256 + 16) + 1024),
    (B.DSATTN_F32, 64, 35, 1, 4 * 16 * (256 + 16) + 1024),
    (B.DSATTN_F32, 112, 500, 2, 4 * 16 * (448 + 16) + 1024),
    (B.DSATTN_F32, 160, 500, 2, 4 * 16 * (640 + 16) + 1024),
])
def test_tile_kernel_reports_its_tasks_and_lds(io, D, positions, tasks, lds):
    plan = B.dsattn_plan(24, 12, 3, positions, 5, D, [0, 5], io_dtype=io, device=-1)
    i = B.dsattn_plan_launch_info(plan)
    plan.close()
    assert (i["block_threads"], i["n_tasks"], i["lds_bytes"]) == (256, 12 * positions * 5 * tasks, lds)


def test_tile_kernel_leaves_launches_of_2_to_the_32_threads_to_the_generic_kernel():
    # a clip of 80 frames is five query tiles a position: with 64 threads each 67,108,832 are 32 short of 2^26, whose
    # launch would have 2^32 threads.  (Two to a wavefront they are three tasks.)
    for P, threads in ((13421766, 256), (13421767, 64)):
        plan = B.dsattn_plan(80, 1, 0, P, 1, 8, [], device=-1)
        i = B.dsattn_plan_launch_info(plan)
        plan.close()
        assert (i["kernel"], i["block_threads"], i["n_tasks"]) == (0, threads, P * (3 if threads == 256 else 1))


def test_flags_are_validated_and_dedup_limits_the_planner():
    lib = B.load()
    d = B.DsattnDesc(16, 4, 2, 4, 2, 160, B.DSATTN_BF16, B.DSATTN_BF16, 0.0, 8, 0.0, 0.0, 0)
    out = ctypes.c_void_p()
    assert lib.dsattn_plan(ctypes.byref(d), None, 0, -1, ctypes.byref(out)) == B.DSATTN_EINVAL
    assert "flag" in B.dsattn_last_error()
    # the set-union option runs on the matrix-core kernel with up to 16 global frames, and with
    # up to 64 where the variant has a whole SIMD's registers (head_dim 160 and 128)
    for D, G, kernel in ((160, 16, 1), (160, 17, 1), (160, 64, 1), (160, 0, 1), (128, 40, 1),
                         (80, 16, 1), (80, 17, 0), (40, 64, 0), (96, 33, 0)):
        plan = B.dsattn_plan(16, 8, 2, 4, 2, D, list(range(G)), flags=B.DSATTN_FLAG_DEDUP_GLOBAL,
                             device=-1)
        assert B.dsattn_plan_launch_info(plan)["kernel"] == kernel, (D, G)
        plan.close()


@pytest.mark.parametrize("D,h,G,hpw", [
    (128, 8, 16, 1), (96, 8, 16, 2), (96, 5, 16, 1), (64, 8, 16, 2), (64, 3, 0, 1), (32, 8, 16, 4),
    (32, 6, 16, 2), (32, 7, 3, 1), (40, 6, 16, 2), (40, 5, 16, 1), (80, 3, 16, 1),
    # 17..64 global frames: fewer heads per wavefront so that the global context fits in registers
    (128, 4, 64, 1), (96, 4, 33, 1), (64, 4, 64, 1), (32, 8, 64, 2), (32, 3, 64, 1), (40, 7, 17, 1),
])
def test_planner_head_dims_and_heads_per_wave(D, h, G, hpw):
    """Every supported head_dim has an MFMA variant for any head count: the planner takes the
    widest rows (most heads per wavefront) that divide the head count."""
    plan = B.dsattn_plan(16, 8, 4, 6, h, D, list(range(0, 2 * G, 2)), device=-1)
    i = B.dsattn_plan_launch_info(plan)
    plan.close()
    assert i["kernel"] == 1 and i["heads_per_wave"] == hpw, i
    assert i["global_tiles"] == (0 if G == 0 else 1 if G <= 16 else 4)
    assert i["n_tasks"] % (i["block_threads"] // 64) == 0
    assert i["lds_bytes"] <= 160 * 1024


@pytest.mark.parametrize("n_clips,P,h,D,w,G,hpw,waves", [
    (39, 48, 8, 80, 0, 32, 1, 4),    # 1,920 of 2,048 wavefronts, rows of 160 bytes; wide rows had eight to a workgroup
    (118, 20, 5, 40, 3, 64, 1, 4),   # rows of 80 bytes
    (12, 32, 8, 80, 2, 16, 1, 4),    # exactly three quarters of them
    (12, 28, 8, 80, 2, 16, 1, 2),    # 1,344
    (40, 64, 8, 40, 2, 16, 2, 4),    # two heads of 80 bytes
    (24, 60, 8, 128, 2, 16, 1, 4),   # whole 64 bytes, 180 MB of tensors
    (24, 40, 8, 128, 2, 16, 1, 2),   # 120 MB
    (8, 192, 8, 128, 2, 16, 1, 2),   # 192 MB, but eight query tiles
])
def test_streaming_launches_that_fill_the_chip_keep_half_a_compute_unit_together(n_clips, P, h, D, w, G, hpw, waves):
    plan = B.dsattn_plan(16, n_clips, w, P, h, D, list(range(G)), device=-1)
    i = B.dsattn_plan_launch_info(plan)
    plan.close()
    assert (i["kernel"], i["heads_per_wave"], i["block_threads"]) == (1, hpw, 64 * waves), i


@pytest.mark.parametrize("n_clips,P,h,D,w,out,hpw,waves", [
    (3, 15, 8, 40, 2, B.DSATTN_BF16, 4, 2),      # fewer than 16 positions: the widest rows
    (3, 16, 8, 40, 2, B.DSATTN_BF16, 1, 1),
    (16, 16, 8, 40, 2, B.DSATTN_BF16, 2, 2),     # 1,024 query tiles of two heads
    (15, 17, 8, 40, 2, B.DSATTN_BF16, 1, 4),     # 1,020
    (16, 48, 4, 32, 2, B.DSATTN_BF16, 2, 2),     # head_dim 32: tensors of exactly 12 MB
    (16, 49, 4, 32, 2, B.DSATTN_BF16, 4, 1),
    (16, 38, 4, 32, 2, B.DSATTN_F32, 2, 2),      # fp32 output: 10 bytes an element
    (16, 39, 4, 32, 2, B.DSATTN_F32, 4, 1),
    (16, 256, 8, 64, 2, B.DSATTN_BF16, 1, 4),    # exactly 256 MB
    (16, 257, 8, 64, 2, B.DSATTN_BF16, 2, 4),
    (16, 204, 8, 64, 2, B.DSATTN_F32, 1, 4),
    (16, 205, 8, 64, 2, B.DSATTN_F32, 2, 2),
    (16, 257, 8, 64, 12, B.DSATTN_BF16, 1, 4),   # three local key tiles: above it too,
    (16, 520, 8, 32, 12, B.DSATTN_BF16, 4, 2),   # but not at head_dim 32
    (16, 140, 8, 128, 12, B.DSATTN_BF16, 1, 4),  # nor from 128 on
    (16, 120, 8, 128, 12, B.DSATTN_BF16, 1, 2),
    (1, 256, 8, 64, 2, B.DSATTN_BF16, 1, 4),     # 640 bytes of a frame and 512 workgroups
    (1, 255, 8, 64, 2, B.DSATTN_BF16, 1, 2),
    (1, 128, 8, 128, 2, B.DSATTN_BF16, 1, 2),
    (1, 127, 8, 128, 2, B.DSATTN_BF16, 1, 1),
])
def test_bounds_of_narrow_streaming_launches(n_clips, P, h, D, w, out, hpw, waves):
    plan = B.dsattn_plan(16, n_clips, w, P, h, D, list(range(16)), out_dtype=out, device=-1)
    i = B.dsattn_plan_launch_info(plan)
    plan.close()
    assert (i["kernel"], i["heads_per_wave"], i["block_threads"]) == (1, hpw, 64 * waves), i


def test_header_is_plain_c_and_usable_from_c(tmp_path):
    """include/dsattn.h compiles as C99 with warnings as errors, and a C program linked against
    libdsattn.so drives the host-side entry points."""
    import subprocess
    exe = tmp_path / "host_only_plan"
    src = os.path.join(ROOT, "tests", "c_abi", "host_only_plan.c")
    libdir = os.path.dirname(B.LIB_PATH)
    subprocess.run(["gcc", "-std=c99", "-Wall", "-Wextra", "-Werror", "-pedantic",
                    "-I", os.path.join(ROOT, "include"), src, "-o", str(exe),
                    "-L", libdir, "-l:libdsattn.so", f"-Wl,-rpath,{libdir}"], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    assert out.startswith("ok lk_max=7")


# ---------------------------------------------------------------- binding: tensor checks
# The C ABI takes bare pointers, so the Python wrappers refuse tensors whose size, element type or
# device does not fit the plan or descriptor before anything reaches a kernel.  Driven here with
# host-only plans (device = -1) and CPU tensors: no GPU is needed to reach the checks.

def _host_plan(**kw):
    args = dict(clip_len=4, n_clips=3, local_ctx=1, spatial=5, heads=2, head_dim=8,
                global_idx=[0, 7], io_dtype=B.DSATTN_BF16, device=-1)
    args.update(kw)
    return B.dsattn_plan(**args)


def test_binding_refuses_wrong_sized_or_typed_tensors_for_a_plan():
    import torch
    plan = _host_plan()
    n = 12 * 5 * 16
    good = lambda: torch.zeros(12, 5, 16, dtype=torch.bfloat16)
    with pytest.raises(ValueError, match="elements"):
        B.dsattn_forward(plan, torch.zeros(n - 16, dtype=torch.bfloat16), good(), good(), good())
    with pytest.raises(ValueError, match="elements"):
        B.dsattn_forward(plan, good(), good(), good(), torch.zeros(n + 1, dtype=torch.bfloat16))
    with pytest.raises(ValueError, match="dtype"):
        B.dsattn_forward(plan, good(), torch.zeros(12, 5, 16, dtype=torch.float32), good(), good())
    with pytest.raises(ValueError, match="dtype"):   # O follows out_dtype (bf16 here)
        B.dsattn_forward(plan, good(), good(), good(), torch.zeros(12, 5, 16, dtype=torch.float32))
    with pytest.raises(ValueError, match="contiguous"):
        B.dsattn_forward(plan, torch.zeros(12, 16, 5, dtype=torch.bfloat16).transpose(1, 2), good(),
                         good(), good())
    # well-formed tensors pass the wrapper; the library then refuses the host-only plan
    with pytest.raises(B.DsattnError) as ei:
        B.dsattn_forward(plan, good(), good(), good(), good(), stream=0)
    assert ei.value.code == B.DSATTN_ENODEVICE
    # materialised contexts are [N, lk_max, P, C]
    lk = B.dsattn_plan_ctx_max(plan)
    assert lk == 4 + 2 + 2
    ctx = lambda k=lk: torch.zeros(3, k, 5, 16, dtype=torch.bfloat16)
    with pytest.raises(ValueError, match="Kctx"):
        B.dsattn_gather_context(plan, good(), good(), ctx(lk - 1), ctx(), stream=0)
    with pytest.raises(ValueError, match="Vctx"):
        B.dsattn_forward_ctx(plan, good(), ctx(), ctx(lk + 1), good(), stream=0)
    with pytest.raises(B.DsattnError):
        B.dsattn_forward_ctx(plan, good(), ctx(), ctx(), good(), stream=0)
    plan.close()
    # fp32 output of a bf16 plan
    plan = _host_plan(out_dtype=B.DSATTN_F32)
    with pytest.raises(ValueError, match="dtype"):
        B.dsattn_forward(plan, good(), good(), good(), good(), stream=0)
    plan.close()


def test_binding_refuses_tensors_on_the_wrong_device():
    import torch
    plan = B.Plan(None, B.DsattnDesc(4, 3, 1, 5, 2, 8, B.DSATTN_BF16, B.DSATTN_BF16, 0.0, 0, 0.0,
                                     0.0, 0), 0, device=0)   # a device plan's bookkeeping only
    t = torch.zeros(12, 5, 16, dtype=torch.bfloat16)
    with pytest.raises(ValueError, match="device memory expected"):
        plan.check("dsattn_forward", [plan.frames(t, "Q")])
    with pytest.raises(ValueError, match="device memory expected"):
        B.dsattn_copy_probe(t, t.clone(), t.numel() * 2, stream=0)
    with pytest.raises(ValueError, match="at least"):
        B.dsattn_copy_probe(t, t.clone(), t.numel() * 2 + 16, stream=0)


def test_binding_checks_groupnorm_conv_and_linear_tensors():
    import torch
    bf = lambda *s: torch.zeros(*s, dtype=torch.bfloat16)
    f32 = lambda *s: torch.zeros(*s, dtype=torch.float32)
    # group normalisation: X, Y [F, P, C]; gamma, beta [C] fp32; stats [2 groups] fp32
    gn = dict(clip_len=4, n_clips=3, spatial=5, channels=64, groups=4)
    with pytest.raises(ValueError, match="X"):
        B.dsattn_groupnorm(**gn, X=bf(12, 5, 32), Y=bf(12, 5, 64), workspace=f32(1024),
                           workspace_bytes=4096, stream=0)
    with pytest.raises(ValueError, match="gamma"):
        B.dsattn_groupnorm(**gn, X=bf(12, 5, 64), Y=bf(12, 5, 64), workspace=f32(1024),
                           workspace_bytes=4096, gamma=bf(64), stream=0)
    with pytest.raises(ValueError, match="stats"):
        B.dsattn_groupnorm_static(**gn, X=bf(12, 5, 64), Y=bf(12, 5, 64), stats=f32(4), stream=0)
    with pytest.raises(ValueError, match="device memory expected"):
        B.dsattn_groupnorm_static(**gn, X=bf(12, 5, 64), Y=bf(12, 5, 64), stream=0)
    # temporal convolution: W [2n + 1, c_out, c_in], Y [F, P, c_out]
    cv = dict(clip_len=4, n_clips=3, spatial=5, c_in=16, c_out=24, reach=1)
    with pytest.raises(ValueError, match="W"):
        B.dsattn_temporal_conv(**cv, X=bf(12, 5, 16), W=bf(1, 24, 16), Y=bf(12, 5, 24), stream=0)
    with pytest.raises(ValueError, match="Y"):
        B.dsattn_temporal_conv(**cv, X=bf(12, 5, 16), W=bf(3, 24, 16), Y=bf(12, 5, 16), stream=0)
    with pytest.raises(ValueError, match="bias"):
        B.dsattn_temporal_conv(**cv, X=bf(12, 5, 16), W=bf(3, 24, 16), Y=bf(12, 5, 24),
                               bias=bf(24), stream=0)
    # projections: every W [c_out, c_in], every Y [rows, c_out]
    with pytest.raises(ValueError, match=r"W\[1\]"):
        B.dsattn_linear(60, 16, 24, bf(60, 16), [bf(24, 16), bf(16, 16)], [bf(60, 24), bf(60, 24)],
                        stream=0)
    with pytest.raises(ValueError, match=r"Y\[0\]"):
        B.dsattn_linear(60, 16, 24, bf(60, 16), [bf(24, 16)], [bf(59, 24)], stream=0)
    with pytest.raises(ValueError, match="dtype"):
        B.dsattn_linear(60, 16, 24, bf(60, 16), [bf(24, 16)], [f32(60, 24)], stream=0)


# ---------------------------------------------------------------- planner: long clips, resolved variant

@pytest.mark.parametrize("D,h", [(160, 8), (80, 8), (40, 8)])
@pytest.mark.parametrize("clip_len,n_clips", [(32, 72), (48, 48), (288, 8)])
def test_long_clips_with_a_window_run_the_matrix_core_kernel(D, h, clip_len, n_clips):
    for w, r, G, reach in ((8, 8, 16, 8), (8, 3, 0, 3), (2, 8, 64, 8), (4, 0, 16, 0), (8, 16, 16, 16)):
        plan = B.dsattn_plan(clip_len, n_clips, w, 160, h, D, list(range(0, 4 * G, 4)), device=-1,
                             window=r)
        i = B.dsattn_plan_launch_info(plan)
        plan.close()
        assert i["kernel"] == 1 and i["ring_reach"] == reach, (w, r, G, i)
        assert i["local_tiles"] == (16 + 2 * reach + 15) // 16
        # chunks are counted in 16-frame query tiles and cover the video exactly
        tiles = clip_len * n_clips // 16
        row_groups = 160 * h // i["heads_per_wave"]
        assert i["n_tasks"] == row_groups * -(-tiles // i["clips_per_task"])
    # the window radius (or, with none, the rest of the clip) must fit the on-chip ring
    for kw in (dict(window=17), dict(window=None), dict(window=9, n_global=129)):
        g = list(range(kw.get("n_global", 4)))
        plan = B.dsattn_plan(clip_len, n_clips, 8, 160, h, D, g, device=-1, window=kw["window"])
        i = B.dsattn_plan_launch_info(plan)
        assert (i["kernel"], i["block_threads"]) == (0, 256), kw     # the 16-query tile kernel
        plan.close()


def test_launch_info_carries_the_resolved_variant():
    # the kernel variant is looked up once, by dsattn_plan; dsattn_forward launches what the plan
    # holds.  Distinct shapes resolve to distinct variants, equal shapes to the same one.
    seen = {}
    for D, h, w, G, od in ((160, 8, 2, 16, B.DSATTN_BF16), (160, 8, 2, 16, B.DSATTN_F32),
                           (160, 8, 4, 64, B.DSATTN_BF16), (80, 8, 2, 16, B.DSATTN_BF16),
                           (40, 8, 2, 16, B.DSATTN_BF16), (40, 8, 4, 64, B.DSATTN_BF16)):
        ids = []
        for n_clips in (8, 144):
            plan = B.dsattn_plan(16, n_clips, w, 12, h, D, list(range(G)), out_dtype=od, device=-1)
            i = B.dsattn_plan_launch_info(plan)
            plan.close()
            assert i["kernel"] == 1 and i["variant"] >= 0
            ids.append(i["variant"])
        assert ids[0] == ids[1]
        assert ids[0] not in seen.values()
        seen[(D, h, w, G, od)] = ids[0]
    plan = B.dsattn_plan(16, 8, 2, 12, 8, 48, [0], device=-1)     # no variant for head_dim 48
    assert B.dsattn_plan_launch_info(plan)["variant"] == -1
    plan.close()


def test_planning_a_very_long_video_is_quick():
    import time
    t0 = time.perf_counter()
    plan = B.dsattn_plan(16, 1 << 20, 2, 1, 8, 160, [0, 5, 9], device=-1)   # 16.8 M frames
    i = B.dsattn_plan_launch_info(plan)
    plan.close()
    assert i["kernel"] == 1 and time.perf_counter() - t0 < 2.0


def test_wide_contexts_reach_the_matrix_core_kernel():
    # 16 context frames per side together with up to 64 global frames; 65 to 128 global frames
    # where eight global key tiles fit a wavefront's registers (not at head_dim 160 and 128)
    for D, h, w, G, kernel, tiles in (
            (160, 8, 16, 64, 1, (3, 4)), (80, 8, 16, 17, 1, (3, 4)), (40, 8, 9, 64, 1, (3, 4)),
            (80, 8, 4, 128, 1, (2, 8)), (40, 8, 16, 65, 1, (3, 8)), (40, 5, 4, 128, 1, (2, 8)),
            (96, 4, 16, 128, 1, (3, 8)), (64, 4, 8, 100, 1, (2, 8)), (32, 4, 16, 128, 1, (3, 8)),
            (128, 4, 0, 128, 0, None), (128, 4, 2, 64, 1, (2, 4)), (160, 8, 4, 65, 0, None),
            (40, 5, 16, 128, 0, None), (80, 8, 4, 129, 0, None)):
        plan = B.dsattn_plan(16, 12, w, 6, h, D, [j % 192 for j in range(G)], device=-1)
        i = B.dsattn_plan_launch_info(plan)
        plan.close()
        assert i["kernel"] == kernel, (D, h, w, G, i)
        if tiles:
            assert (i["local_tiles"], i["global_tiles"]) == tiles, (D, h, w, G, i)


def test_layer_entry_point_checks_its_arguments_on_the_host():
    lib = B.load()
    plan = B.dsattn_plan(16, 4, 2, 5, 8, 40, [0, 9], device=-1)
    need = B.dsattn_temporal_layer_workspace(plan)
    one = 64 * 5 * 320 * 2                                  # one [F, P, C] bf16 tensor
    assert need == 4 * ((one + 255) // 256 * 256)
    n = ctypes.c_size_t(0)
    assert lib.dsattn_temporal_layer_workspace(None, ctypes.byref(n)) == B.DSATTN_EINVAL
    assert lib.dsattn_temporal_layer_workspace(plan.handle, None) == B.DSATTN_EINVAL
    w = (ctypes.c_void_p * 4)(0x100000, 0x200000, 0x300000, 0x400000)
    args = lambda **kw: [kw.get("plan", plan.handle), kw.get("x", 0x1000000), kw.get("w", w), None,
                         kw.get("ws", 0x8000000), kw.get("n", need), kw.get("y", 0x4000000), None]
    assert lib.dsattn_temporal_layer(*args(plan=None)) == B.DSATTN_EINVAL
    assert lib.dsattn_temporal_layer(*args(x=None)) == B.DSATTN_EINVAL
    assert lib.dsattn_temporal_layer(*args(w=None)) == B.DSATTN_EINVAL
    assert lib.dsattn_temporal_layer(*args(ws=None)) == B.DSATTN_EINVAL
    assert lib.dsattn_temporal_layer(*args(y=None)) == B.DSATTN_EINVAL
    assert lib.dsattn_temporal_layer(*args()) == B.DSATTN_ENODEVICE      # host-only plan
    plan.close()
    # fp32 output of bf16 attention cannot feed the output projection
    plan = B.dsattn_plan(16, 4, 2, 5, 8, 40, [0, 9], out_dtype=B.DSATTN_F32, device=-1)
    assert lib.dsattn_temporal_layer(*args(plan=plan.handle)) == B.DSATTN_ENODEVICE
    plan.close()


def _device_kernels():
    """Every kernel of the built library with what its code object says of it (registers, scratch memory)."""
    msgpack = pytest.importorskip("msgpack")
    blob = open(B.LIB_PATH, "rb").read()
    kernels, at = {}, 0
    while (at := blob.find(b"\x7fELF\x02\x01\x01\x40", at)) >= 0:  # an AMDGPU code object
        sections, = struct.unpack_from("<Q", blob, at + 40)
        size, count = struct.unpack_from("<HH", blob, at + 58)
        for i in range(count):
            _, kind, _, _, off, length = struct.unpack_from("<IIQQQQ", blob, at + sections + i * size)
            p, end = at + off, at + off + length
            while kind == 7 and p < end:  # notes
                name, desc, note = struct.unpack_from("<III", blob, p)
                p += 12 + (name + 3) // 4 * 4
                if note == 32:  # metadata
                    for k in msgpack.unpackb(blob[p:p + desc])["amdhsa.kernels"]:
                        kernels[k[".name"]] = k
                p += (desc + 3) // 4 * 4
        at += 8
    return kernels


def test_no_kernel_uses_scratch_memory_and_option_kernels_keep_their_wavefronts():
    """512 registers a SIMD, in steps of 8 a wavefront.  The fp32 tile kernels for the set union and for any option:
    wavefronts by head_dim / 16, whole multiples of 16 and the rest."""
    kernels = _device_kernels()
    spills = [n for n, k in kernels.items() if k[".private_segment_fixed_size"]]
    assert kernels and not spills, spills[:5]
    least = {1: (8, 8), 2: (6, 6), 3: (5, 4), 4: (4, 4), 5: (4, 4), 6: (3, 3), 7: (3, 3), 8: (2, 2), 9: (2, 2), 10: (2, 2)}
    seen = 0
    for name, k in kernels.items():
        m = re.search(r"tile_attn_f32_kernelILi(\d+)ELb([01])ELi1ELi([34])E", name)
        if not m:
            continue
        seen += 1
        waves = min(8, 512 // (-(-k[".vgpr_count"] // 8) * 8))
        assert waves >= least[int(m[1])][m[2] == "0"], (name, k[".vgpr_count"])
    assert seen == 40
