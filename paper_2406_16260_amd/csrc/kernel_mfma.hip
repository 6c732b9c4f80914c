// Host side of the bf16 MFMA streaming kernel: variant lookup, the launch planner's choices
// for it (heads per wavefront, wavefronts per workgroup, clips per chunk) and the launcher.
#include <algorithm>
#include <cmath>
#include <cstdlib>

#include "mfma_kernel.h"
#include "plan.h"

namespace dsattn {

namespace {

constexpr int kLdsPerCu = 160 * 1024;  // gfx950 LDS per compute unit, also the per-workgroup cap
constexpr int kCus = 256;

typedef const MfmaVariant *(*VariantTable)(int *);
const VariantTable kTables[] = {mfma_variants_d160, mfma_variants_d128, mfma_variants_d96,
                                mfma_variants_d80,  mfma_variants_d64,  mfma_variants_d40,
                                mfma_variants_d32};

// Position of a variant in the concatenation of the per-head_dim tables: the id that
// dsattn_launch_info reports.
const MfmaVariant *find_variant(int D, int HPW, int NLT, int NGT, bool out_f32, int *id = nullptr)
{
    int base = 0;
    for (VariantTable tab : kTables) {
        int n = 0;
        const MfmaVariant *v = tab(&n);
        for (int i = 0; i < n; ++i)
            if (v[i].D == D && v[i].HPW == HPW && v[i].NLT == NLT && v[i].NGT == NGT &&
                v[i].out_f32 == out_f32) {
                if (id) *id = base + i;
                return &v[i];
            }
        base += n;
    }
    return nullptr;
}

int env_int(const char *name, int dflt)
{
    const char *e = getenv(name);
    return e && *e ? atoi(e) : dflt;
}

// What a launch is made of: the variant, wavefronts per workgroup, query tiles per chunk.
struct Geometry {
    const MfmaVariant *var = nullptr;
    int id = -1, hpw = 0, wpb = 1, m = 1, lds = 0;
    int64_t tasks = 0;  // wavefronts
};

// A plan's shape as the kernel sees it.
struct Shape {
    int n_tiles, wr, R, NLT, NGT, G;
    bool out_f32;
    int64_t bytes;  // of Q, K, V and O
};

// spread: narrower rows and smaller workgroups, see mfma_plan().
bool mfma_geometry(const dsattn_plan_t &pl, const Shape &sh, bool spread, Geometry &geo)
{
    const dsattn_desc &d = pl.desc;
    const int n_tiles = sh.n_tiles, wr = sh.wr, R = sh.R, NLT = sh.NLT, NGT = sh.NGT, G = sh.G;
    const bool out_f32 = sh.out_f32;
    // heads per wavefront: prefer the variant that keeps two wavefronts per SIMD (more loads in
    // flight, compute of one wavefront hidden behind the other), then the widest rows; a
    // wavefront never straddles two positions
    // The set-union option is built into the variants with one global key tile, and into the
    // four-tile variants that run one wavefront per SIMD (head_dim 160 and 128): with that option
    // and four tiles only those are candidates.
    // With eight tiles it is not built in (the 16-query tile kernel takes those).
    if ((d.flags & DSATTN_FLAG_DEDUP_GLOBAL) && NGT == 8) return false;
    const bool need_wpe1 = (d.flags & DSATTN_FLAG_DEDUP_GLOBAL) && NGT == 4;
    const MfmaVariant *var = nullptr;
    int var_id = -1;
    const int force_hpw = env_int("DSATTN_HEADS_PER_WAVE", 0);
    for (int wpe : {2, 1}) {
        if (need_wpe1 && wpe != 1) continue;
        for (int cand : {4, 2, 1}) {
            if (force_hpw && cand != force_hpw) continue;
            if (d.heads % cand != 0) continue;
            int id = -1;
            const MfmaVariant *v = find_variant(d.head_dim, cand, NLT, NGT, out_f32, &id);
            if (v && v->WPE == wpe) {
                var = v;
                var_id = id;
                break;
            }
        }
        if (var) break;
    }
    if (!var) return false;
    // Narrower rows: up to 96 channels (one head, or two of 40 and of 32), and one head where there are fewer than
    // 1,024 query tiles of those.
    const int wide = var->HPW;
    if (spread && !force_hpw) {
        for (int cand : {2, 1}) {
            if (cand >= var->HPW || d.heads % cand != 0) continue;
            if (var->HPW * d.head_dim <= 96 && (int64_t)d.spatial * (d.heads / var->HPW) * n_tiles >= 1024) break;
            int id = -1;
            const MfmaVariant *v = find_variant(d.head_dim, cand, NLT, NGT, out_f32, &id);
            if (v && v->WPE == var->WPE) {
                var = v;
                var_id = id;
            }
        }
    }
    const int hpw = var->HPW;
    const int lds_wave = (2 * R + 16) * row_stride_bytes(d.head_dim * hpw);
    if (lds_wave > kLdsPerCu) return false;
    const int RG = d.spatial * (d.heads / hpw);

    // wavefronts per workgroup.  The wavefronts of a workgroup fetch neighbouring rows together
    // (one barrier per clip), so a workgroup should span at least one whole position (all its
    // heads: a contiguous, line-aligned run per frame).  Beyond that, two workgroups per compute
    // unit are better than one: while one starts or drains a chunk the other keeps streaming.
    const int max_waves_cu = std::min(4 * var->WPE, kLdsPerCu / lds_wave);
    const int waves_per_pos = d.heads / hpw;
    // Where the rows are spread: about 640 bytes of a frame (1 clip of 1,398 positions, 8 x 128, 50.6 us with eight
    // wavefronts, 41.4 with two; 9 of 271 71.9 and 62.4), and 512 workgroups if there are as many wavefronts.
    const int want = spread ? std::min(max_waves_cu, std::max(1, 640 / (2 * hpw * d.head_dim)))
                            : std::min(max_waves_cu, std::max(waves_per_pos, max_waves_cu / 2));
    int wpb = 1;
    for (int cand : {8, 4, 2, 1})
        if (cand <= want && RG % cand == 0) {
            wpb = cand;
            break;
        }
    {
        const int e = env_int("DSATTN_WAVES_PER_BLOCK", wpb);
        if (e >= 1 && e <= 8 && e <= max_waves_cu && RG % e == 0) wpb = e;
    }
    const int blocks_cu = std::max(1, max_waves_cu / wpb);
    const int bpc = RG / wpb;

    // chunks per row group: fewer chunks re-read less context (2w boundary frames + G global
    // frames of K and V per chunk); more chunks fill the machine.  Model: time ~ traffic x fill,
    // where the workgroups run in rounds of `slots`.  With few rounds the workgroups stay in
    // step and a last round less than 85 % full costs a whole round; after about six rounds they have
    // drifted apart and the tail costs little more than its share.  Fewer workgroups than slots
    // leave compute units idle.  Every chunk also pays for its start, which decides short videos
    // (four clips: one chunk per row group beats two).
    const double slots = (double)kCus * blocks_cu;
    int best_nc = 1;
    double best_cost = 1e300;
    // (past a few dozen rounds the fill term is 1 and more chunks only add traffic)
    const int nc_cap = (int)std::min<double>(n_tiles, std::max(4096.0, 64.0 * slots / bpc));
    for (int nc = 1; nc <= nc_cap; ++nc) {
        const int m = (n_tiles + nc - 1) / nc;
        if ((n_tiles + m - 1) / m != nc) continue;  // same chunking as a smaller nc
        const double rounds = (double)bpc * nc / slots;
        const double whole = std::floor(rounds);
        const double rem = rounds - whole;
        const double rounds_eff =
            rounds <= 1.0 ? 1.0
                          : whole + (rem > 1e-9 ? (whole < 6.0 && rem < 0.85 ? 1.0
                                                                              : std::max(rem, 0.6))
                                                : 0.0);
        const double fill = rounds_eff / rounds;
        const double kv = (16.0 * m + (nc > 1 ? 2.0 * wr : 0.0) + G) / (16.0 * m);
        // a chunk's start (two memory round trips before its first tile) costs about one tile, less where
        // narrower wavefronts than the widest leave more of them to fill it
        const double cost = (2.0 + 2.0 * kv) / 4.0 * fill * (1.0 + (hpw < wide ? 0.5 : 1.0) / m);
        if (cost < best_cost - 1e-12) {
            best_cost = cost;
            best_nc = nc;
        }
    }
    int m = (n_tiles + best_nc - 1) / best_nc;
    m = std::max(1, std::min(n_tiles, env_int("DSATTN_CLIPS_PER_TASK", m)));
    const int NC = (n_tiles + m - 1) / m;
    if ((int64_t)RG * NC > 0x7fffffffLL) return false;
    // A short video whose wavefronts all run at once has nothing to pace: two wavefronts per workgroup spread
    // over more compute units and start independently.  Measured, one position's heads per workgroup / two
    // wavefronts: 1 clip, 40 positions, 8 heads of 160 9.1 / 6.6 us; 4 clips, 40 x 8 x 160 10.6 / 9.7, 160 x
    // 8 x 160 28.7 / 24.4, 640 x 8 x 40 31.9 / 29.8; 16 clips, 40 x 8 x 160 24.9 / 23.7.  From 24 clips on
    // (35.5 / 36.1), and with four wavefronts and a single clip (8.0 / 8.3), the shared lines of neighbouring
    // rows count for more.  (Launches that are spread decide by the two rules before it; this one is left to
    // fewer than 16 positions, materialised contexts, and head_dim 32 above 12 MB.)
    if (env_int("DSATTN_WAVES_PER_BLOCK", 0)) {
    } else if (spread && (int64_t)RG * NC * 4 >= (int64_t)kCus * max_waves_cu * 3 &&
               (hpw * d.head_dim % 32 != 0 || (n_tiles > 8 && sh.bytes >= (int64_t)128 << 20))) {
        // From three quarters of the chip's wavefronts on there is little left to spread over, and what a frame's
        // neighbouring rows share counts: rows of 80 and 160 bytes share 128-byte lines, tensors that leave the cache
        // are read in order.  Half a compute unit's wavefronts then stay together.  Time with them over time with one or two:
        //   rows of 80 and 160 bytes (head_dim 40 and 80), by the share of the chip: 0.5 to 0.65 1.04, 0.7 1.01, 0.75 0.96, 0.8
        //   and up 0.945; by query tiles, 1 to 4 0.96, 33 and more 0.94
        //   others, tensors of 128 MB and more, from HBM and from the caches: up to 8 tiles 1.00 and 1.01 (head_dim 128 1.02 and 1.04),
        //   more 0.97 and 0.99; less than 64 MB 1.01 and 1.03, 64 to 128 MB 0.98 and 1.01
        // us from HBM, two and four: 39 clips of 48 positions, 8 x 80, 32 global frames, 41.2 and 37.1, 93 of 24, 8 x 80, 48.6 and 42.8, 24
        // of 60, 8 x 128, 40.8 and 39.0, 24 of 40, 8 x 160, 36.5 and 35.0 (35.6 with eight).
        for (int cand : {4, 2, 1})
            if (cand <= std::max(1, max_waves_cu / 2) && RG % cand == 0) {
                wpb = cand;
                break;
            }
    } else if (spread) {
        while (wpb > 1 && (int64_t)(RG / wpb) * NC < 512) wpb /= 2;
    } else if ((int64_t)RG * NC <= (int64_t)kCus * max_waves_cu && n_tiles <= 16 && wpb > (n_tiles == 1 ? 4 : 2) &&
               RG % 2 == 0) {
        wpb = 2;
    }
    geo.var = var;
    geo.id = var_id;
    geo.hpw = hpw;
    geo.wpb = wpb;
    geo.m = m;
    geo.lds = lds_wave * wpb;
    geo.tasks = (int64_t)RG * NC;
    return true;
}

}  // namespace

bool mfma_plan(dsattn_plan_t &pl)
{
    const dsattn_desc &d = pl.desc;
    // The kernel works on query tiles of 16 frames; a clip is a whole number of them.
    if (d.io_dtype != DSATTN_BF16 || d.clip_len % 16 != 0) return false;
    if (pl.C % 8 != 0) return false;
    // the kernel addresses the 16 frame rows of a tile with 32-bit byte offsets
    if ((int64_t)d.spatial * pl.C * 2 * 16 >= ((int64_t)1 << 32)) return false;
    const int G = (int)pl.global_idx.size();
    // global key tiles: variants exist for 0, 1, 4 and (where a wavefront's registers hold
    // them) 8 tiles; a partly used tile is masked
    if (G > 128) return false;
    const int NGT = G == 0 ? 0 : (G <= 16 ? 1 : (G <= 64 ? 4 : 8));
    // Frames a tile's local scope can reach beyond the tile on each side: up to the end of the
    // clip's local range (the rest of the clip plus the neighbour's context frames), or the
    // sliding window's radius when that is shorter.  With 16-frame clips and no window this is
    // the clip's local context width.
    const int64_t reach = (int64_t)d.clip_len - 16 + d.local_ctx;
    const int64_t wr64 = pl.window >= 0 ? std::min<int64_t>(pl.window, reach) : reach;
    if (wr64 > 16) return false;  // local key tiles: variants exist for 1 to 3
    const int wr = (int)wr64;
    const int n_tiles = pl.F / 16;
    const int R = 16 + 2 * wr;
    const int NLT = (R + 15) / 16;
    const bool out_f32 = d.out_dtype == DSATTN_F32;

    const int64_t bytes = (int64_t)pl.F * d.spatial * pl.C * (out_f32 ? 10 : 8);
    const Shape sh = {n_tiles, wr, R, NLT, NGT, G, out_f32, bytes};
    Geometry geo, ctx;
    if (!mfma_geometry(pl, sh, false, ctx)) return false;
    // More and narrower wavefronts, each with less to do between its loads, in smaller workgroups: where the tensors
    // are no larger than the 256 MB cache, so that how the rows lie in HBM does not decide, and with three local key
    // tiles, whose ring leaves a compute unit less than a full set of wide wavefronts.  us, wide and narrow: 1 clip of
    // 600 positions, 8 x 80, 22.9 and 15.7; 3 clips of 168, 8 x 40, 12.7 and 9.2; 8 clips of 111, 8 x 40, 16.0 and
    // 12.5; three key tiles: 64 frames x 728, 10 x 64, 90 and 65, 2,112 x 696, 8 x 40, 1,054 and 817, 2,432 x 93, 6 x
    // 96, 263 and 219 (from head_dim 128 on there is nothing narrower).  Larger tensors: 2,304 frames of 160 positions,
    // 20 x 64, 728 and 752, under a window, 640, 8 x 80, 1,489 and 1,574.  Time of the launches below over that of the
    // wide ones, two and three key tiles, from HBM and from the caches: 800 drawn shapes up to 256 MB 0.95 and 0.945
    // (1.17 at most), 870 with three key tiles above 0.93 (0.55 to 1.18).
    // Two lines are drawn short of where narrow rows end to be faster, and not moved yet.  Fewer than 16 positions keep
    // the widest rows: 566 drawn shapes of 1 to 15 positions would take 0.90 of the time (0.52 to 1.10; 3 clips of 15,
    // 8 x 40, 10.2 and 5.5 us, of 16 10.2 and 5.4; 40 clips of 15, 8 x 80, 15.8 and 13.2, 144 31.4 and 34.3).  Head_dim
    // 32 has them up to 12 MB only: above, 0.93 to 64 MB and 0.96 to 256 (0.74 to 1.12; 128 frames x 80, 4 heads, 8.3
    // and 6.5, 128 x 160 8.7 and 8.4, 32 x 599 8.9 and 9.4, 1,152 x 160 34.4 and 34.0), with three key tiles above 256
    // MB 0.925 (0.68 to 1.09; 5,184 x 97 123 and 131).
    // A materialised context, whose chunks are clips, keeps the widest rows: 9 clips of 52, 8 x 80, with the gather 26.5
    // and 28.3.
    const bool spread = d.spatial >= 16 && (bytes <= (int64_t)(d.head_dim == 32 ? 12 : 256) << 20 ||
                                            (NLT == 3 && d.head_dim != 32 && d.head_dim < 128));
    // (a launch has less than 2^32 threads)
    if (!spread || !mfma_geometry(pl, sh, true, geo) || geo.tasks > ((int64_t)1 << 32) / 64 - 8) geo = ctx;
    const MfmaVariant *var = geo.var;
    const int m = geo.m;

    dsattn_launch_info &li = pl.launch;
    li.kernel = 1;
    li.heads_per_wave = geo.hpw;
    li.local_tiles = NLT;
    li.global_tiles = NGT;
    li.clips_per_task = m;
    li.n_tasks = (int32_t)geo.tasks;
    li.block_threads = 64 * geo.wpb;
    li.lds_bytes = geo.lds;
    li.variant = geo.id;
    li.ring_reach = wr;
    pl.ctx_hpw = ctx.hpw;
    pl.ctx_wpb = ctx.wpb;
    pl.ctx_lds = ctx.lds;

    // everything a launch needs that does not depend on the tensors
    // (24 tiles: the shortest chunk of the long videos; a clip of a materialised context is a chunk)
    pl.mfma_fn = m >= 24 && var->fn_sel ? var->fn_sel : var->fn;
    pl.mfma_ctx_fn = d.clip_len / 16 >= 24 && ctx.var->fn_sel ? ctx.var->fn_sel : ctx.var->fn;
    pl.gdup = 0;  // entries that repeat an earlier one (the kernel takes at most 64 entries)
    for (size_t j = 0; j < pl.global_idx.size() && j < 64; ++j)
        for (size_t jj = 0; jj < j; ++jj)
            if (pl.global_idx[jj] == pl.global_idx[j]) {
                pl.gdup |= (uint64_t)1 << j;
                break;
            }
    return true;
}

// Raises the kernel's dynamic-LDS cap on the current device to the whole 160 KB (the default
// cap is 64 KB).  Done once per plan, outside the launch path, so that dsattn_forward makes no
// call other than the launch itself (it can be captured into a HIP graph).  The cap is always
// the maximum: plans that share a variant must not lower each other's limit.
hipError_t mfma_prepare(const dsattn_plan_t &pl)
{
    if (!pl.mfma_fn || !pl.mfma_ctx_fn) return hipErrorInvalidValue;
    const hipError_t e =
        hipFuncSetAttribute(pl.mfma_fn, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsPerCu);
    if (e != hipSuccess || pl.mfma_ctx_fn == pl.mfma_fn) return e;
    return hipFuncSetAttribute(pl.mfma_ctx_fn, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsPerCu);
}

hipError_t launch_mfma(const dsattn_plan_t &pl, const void *Q, const void *K, const void *V,
                       void *O, bool ctx_mode, hipStream_t st)
{
    // the variant and the duplicate mask were resolved by mfma_plan: nothing is searched here
    const dsattn_desc &d = pl.desc;
    const dsattn_launch_info &li = pl.launch;
    const void *fn = ctx_mode ? pl.mfma_ctx_fn : pl.mfma_fn;
    if (!fn) return hipErrorInvalidValue;
    const int wpb = ctx_mode ? pl.ctx_wpb : li.block_threads / 64;

    MfmaArgs a;
    a.Q = (const __bf16 *)Q;
    a.K = (const __bf16 *)K;
    a.V = (const __bf16 *)V;
    a.O = O;
    a.gidx = pl.d_global_idx;
    const int n_tiles = pl.F / 16;
    a.N = n_tiles;
    a.F = pl.F;
    a.h = d.heads;
    a.w = li.ring_reach;
    a.G = (int32_t)pl.global_idx.size();
    a.R = 16 + 2 * li.ring_reach;
    a.clip_len = d.clip_len;
    a.wl = d.local_ctx;
    a.window = pl.window;
    a.M = ctx_mode ? d.clip_len / 16 : li.clips_per_task;
    a.cstride = ctx_mode ? (int64_t)pl.lk_max * d.spatial * pl.C : 0;
    a.RG = d.spatial * (d.heads / (ctx_mode ? pl.ctx_hpw : li.heads_per_wave));
    a.BPC = a.RG / wpb;
    a.C = pl.C;
    a.FS = (int64_t)d.spatial * pl.C;
    a.sc = pl.scale * 1.4426950408889634f;
    // (in 64 bits: the difference may be more than a float holds; 3e38 already hides a scope)
    const double diff = a.G ? ((double)d.bias_global - d.bias_local) / pl.scale : 0.0;
    a.lshift = (float)std::max(std::min(-diff, 0.0), -3e38);
    a.gshift = (float)std::max(std::min(diff, 0.0), -3e38);
    a.dedup = (d.flags & DSATTN_FLAG_DEDUP_GLOBAL) ? 1 : 0;
    a.gdup = pl.gdup;

    // the grid must be exactly chunks x workgroups-per-chunk, each workgroup wpb whole row groups
    const int NC = (n_tiles + a.M - 1) / a.M;
    if (a.RG % wpb != 0 || (!ctx_mode && (int64_t)a.BPC * NC * wpb != (int64_t)li.n_tasks) ||
        (int64_t)a.BPC * NC > 0x7fffffffLL)
        return hipErrorInvalidValue;

    void *params[] = {&a};
    return hipLaunchKernel(fn, dim3((unsigned)(a.BPC * NC)), dim3((unsigned)(64 * wpb)),
                           params, (size_t)(ctx_mode ? pl.ctx_lds : li.lds_bytes), st);
}

}  // namespace dsattn
