// Dual-scope attention on the matrix cores for what the streaming kernel does not take: fp32
// tensors, clips that are not whole 16-frame tiles, local scopes that reach further than its ring,
// longer global lists.  Precision is that of the vector kernel: fp32 softmax, weights kept at 24
// bits.
//
// One wavefront owns 16 query frames of one clip, position and head, and walks the clip's context
// list in tiles of 16 keys with a running maximum.  With clips of a few dozen frames a key row is
// used by one to a few wavefronts only, so nothing is shared in LDS and rows are loaded from global
// memory straight into the operand layout of the matrix instructions.
//   S^T = K Q^T   keys on M, queries on N.  The lane's 16 bytes are chunk 4 j + lane / 16 of row
//                 lane % 16, in both operands, so any order of the channels contracts the same:
//                 one operand of v_mfma_f32_16x16x32_bf16, or four of v_mfma_f32_16x16x4_f32.
//   O^T = V^T P^T fp32: v_mfma_f32_16x16x4_f32; lane (m, k) loads W consecutive channels 64 b + W m of
//                 key 4 k + s, the operands of W products, and the weight it holds of that key is the
//                 other operand as it stands.
//                 bf16: v_mfma_f32_16x16x32_bf16 over a pair of key tiles; V passes through a few KB
//                 of wavefront-private LDS for the transposing read, and a weight enters as the sum
//                 of three bf16 numbers (8 bits each: all 24), whose products are exact.
//
// What bounds it: at short context lists HBM and the softmax's vector instructions, about half
// each.  Tasks are numbered so that one XCD works through consecutive clips of one position: the
// global frames and the boundary frames that neighbouring clips share are then in its L2, and measured
// HBM reads are the tensors' own size (1.38 GB of Q, K, V at 90 clips of 25 frames x 160 positions x 640
// channels; 3.0 TB/s with the vector ALUs busy for 48 % of the time).  Positions fastest instead: up to 7 % slower.
// Measured (generic kernel before): 12 clips of 24 frames x 135 positions, 5 heads of 64, bf16 35 us
// (191); 90 clips of 25 x 160, 10 heads of 64, bf16 583 us (3,409; a 5.2 TB/s stream of the four
// tensors: 355); 384 frames x 640, 8 heads of 80, fp32 677 us (2,644; 484); 2 clips of 288 frames,
// 320 keys a clip, bf16 2.4 ms (602).
// Variants: V transposed by a 0/1 selector product instead of through LDS, the same time, but an
// infinity in V reaches the 31 channels beside it; bf16 weights times V on the fp32
// instructions, 30 % slower; weights split by rounding instead of cutting, 10 % slower.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "plan.h"

namespace dsattn {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct TileArgs {
    const void *Q, *K, *V;
    void *O;
    const int32_t *gidx;
    int32_t N, F, P, h, D, clip_len, lk_max;
    int32_t wl;        // local context width of a clip
    int32_t nqt;       // query tiles per clip
    int32_t ctx_mode;  // K and V are materialised contexts [N, lk_max, P, C]
    int32_t G, window, dedup;
    uint32_t per_xcd;  // workgroups per XCD
    uint32_t tasks;
    float sc;          // scale * log2(e)
    float lb, gb;      // shifts of the local and the global keys' raw scores, see launch_tile_attn
};

// The clip's context list: frames [lo, lo + nl), then the global entries; L keys in all.  (Worked
// out here and not read from the plan's table: the first key rows are then asked for at once.)
// Keys j < run are consecutive rows of K and V, from row0 on.
struct Context {
    int lo, nl, L, run;
    int64_t row0;
};
__device__ __forceinline__ Context context_of(const TileArgs &a, int clip)
{
    Context c;
    c.lo = max(0, clip * a.clip_len - a.wl);
    c.nl = min(a.F, (clip + 1) * a.clip_len + a.wl) - c.lo;
    c.L = c.nl + a.G;
    c.run = a.ctx_mode ? c.L : c.nl;
    c.row0 = a.ctx_mode ? (int64_t)clip * a.lk_max : (int64_t)c.lo;
    return c;
}

// row of key j in K and V (keys past the list: the last one's, their weights are zero)
__device__ __forceinline__ int64_t key_row(const TileArgs &a, const Context &c, int j)
{
    j = min(j, c.L - 1);
    return j < c.run ? c.row0 + j : (int64_t)a.gidx[j - c.run];
}
// what the masks need to know about key j: its frame and, with the set union, whether it repeats an
// earlier global entry
__device__ __forceinline__ int key_info(const TileArgs &a, const Context &c, int j)
{
    j = min(j, c.L - 1);
    if (j < c.nl) return c.lo + j;
    const int frame = a.gidx[j - c.nl];
    bool dup = false;
    if (a.dedup)
        for (int u = 0; u + 1 < a.G; ++u) dup = dup || (u < j - c.nl && a.gidx[u] == frame);
    return frame | (dup ? 1 << 30 : 0);
}

// Orders LDS accesses of the wavefront's lanes: they execute in issue order, only the compiler has to
// be kept from moving them.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// maximum / sum over the lanes l, l ^ 16, l ^ 32, l ^ 48
__device__ __forceinline__ float swap16(float x, bool max)
{
    const unsigned a = __builtin_bit_cast(unsigned, x);
    const auto r = __builtin_amdgcn_permlane16_swap(a, a, false, false);
    const unsigned r0 = r[0], r1 = r[1];
    const float y0 = __builtin_bit_cast(float, r0), y1 = __builtin_bit_cast(float, r1);
    return max ? fmaxf(y0, y1) : y0 + y1;
}
__device__ __forceinline__ float swap32(float x, bool max)
{
    const unsigned a = __builtin_bit_cast(unsigned, x);
    const auto r = __builtin_amdgcn_permlane32_swap(a, a, false, false);
    const unsigned r0 = r[0], r1 = r[1];
    const float y0 = __builtin_bit_cast(float, r0), y1 = __builtin_bit_cast(float, r1);
    return max ? fmaxf(y0, y1) : y0 + y1;
}

// 2^x, and not zero for a finite x (the instruction alone returns zero below -126; 2^100 and more below it
// is as good as -inf): a weight of zero would make NaN of an infinity in V, which any weight leaves infinite.
__device__ __forceinline__ float exp2_positive(float x)
{
    return __builtin_amdgcn_exp2f(fmaxf(x, fmaf(x, 0x1p-100f, -126.f)));
}

// The part of the kernel that both types share: masks, running softmax.  KT key tiles per step.
template <int KT, bool POSITIVE>
struct Softmax {
    float m = -INFINITY, l = 0.f;  // running maximum of the query's column; this lane's part of the sum
    // A shift of the local scores holds from the query's first visible global key on: the set union may
    // hide them all, and then it is the local scores that count.
    bool shifted;

    __device__ __forceinline__ explicit Softmax(const TileArgs &a) : shifted(!a.dedup) {}

    // scores of key tiles t0 .. t0 + nt - 1 -> weights (unnormalised; those of a tile that is not
    // there are zero); returns the factor for what has been accumulated so far
    __device__ __forceinline__ float step(const TileArgs &a, const Context &c, f32x4 (&s)[KT], int t0,
                                          int nt, int clip, int qt, int lane)
    {
        const int l16 = lane & 15, lg = lane >> 4, j0 = 16 * t0 + 4 * lg;
        const bool opts = a.window >= 0 || a.dedup;
        if (opts || 16 * (t0 + nt) > c.L) {  // else every key counts
            const int aq = clip * a.clip_len + 16 * qt + l16;
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                if (t >= nt) continue;
                int info = 0;
                if (opts) info = key_info(a, c, 16 * (t0 + t) + l16);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool local = j0 + 16 * t + e < c.nl;
                    bool hidden = j0 + 16 * t + e >= c.L;
                    if (opts) {
                        const int ki = __shfl(info, 4 * lg + e);  // from the key's own lane
                        const int f = ki & 0x3fffffff;
                        const bool far = a.window >= 0 && abs(f - aq) > a.window;
                        const bool seen = (ki >> 30 & 1) || (f >= c.lo && f < c.lo + c.nl && !far);
                        hidden = hidden || (local ? far : a.dedup && seen);
                    }
                    s[t][e] = hidden ? -INFINITY : s[t][e];
                }
            }
        }
        if (a.lb != 0.f || a.gb != 0.f) {
            if (a.dedup && a.lb != 0.f) {
                float mg = -INFINITY;
#pragma unroll
                for (int t = 0; t < KT; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (t < nt && j0 + 16 * t + e >= c.nl) mg = fmaxf(mg, s[t][e]);
                const bool first = !shifted && swap32(swap16(mg, true), true) > -INFINITY;
                m += first ? a.lb * a.sc : 0.f;
                shifted = shifted || first;
            }
            const float ls = shifted ? a.lb : 0.f;
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) s[t][e] += j0 + 16 * t + e < c.nl ? ls : a.gb;
        }
        float mx = -INFINITY;
#pragma unroll
        for (int t = 0; t < KT; ++t)
            if (t < nt)
#pragma unroll
                for (int e = 0; e < 4; ++e) mx = fmaxf(mx, s[t][e]);
        mx *= a.sc;
        mx = fmaxf(m, swap32(swap16(mx, true), true));
        float alpha = 1.f;
        if (__any(mx > m)) {
            // (no visible key so far: weights of zero, not of exp2(-inf + inf))
            alpha = mx == -INFINITY ? 1.f : POSITIVE ? exp2_positive(m - mx) : __builtin_amdgcn_exp2f(m - mx);
            m = mx;
            l *= alpha;
        }
        const float nm = m == -INFINITY ? 0.f : -m;
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            if (t < nt) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float x = fmaf(s[t][e], a.sc, nm);
                    s[t][e] = POSITIVE ? exp2_positive(x) : __builtin_amdgcn_exp2f(x);
                    l += s[t][e];
                }
            } else {
                s[t] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
        return alpha;
    }
    __device__ __forceinline__ float inverse_sum() const
    {
        return 1.0f / swap32(swap16(l, false), false);
    }
};

// (clips of one position are neighbours: numbered the other way round, positions fastest, it
// measured up to 7 % slower)
struct Task {
    int clip, p, g, qt;
    bool exists;
};
__device__ __forceinline__ Task task_of(const TileArgs &a)
{
    // XCD x (= workgroup % 8) takes a contiguous run of tasks
    const uint32_t wg = (blockIdx.x % 8u) * a.per_xcd + blockIdx.x / 8u;
    // (less than 2^31 tasks: 32-bit divisions, a 64-bit one is some hundred scalar instructions)
    uint32_t id = wg * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Task k;
    k.exists = id < a.tasks;
    uint32_t rest = id / (uint32_t)a.nqt;
    k.qt = (int)(id - rest * a.nqt);
    id = rest;
    rest = id / (uint32_t)a.h;
    k.g = (int)(id - rest * a.h);
    k.p = (int)(rest / (uint32_t)a.N);
    k.clip = (int)(rest - (uint32_t)k.p * a.N);
    return k;
}

// A bf16 task whose result has a NaN and whose V rows have an infinity is done again, one query at a time
// on the vector ALUs: zero times an infinity in V is NaN, a small weight times it is not, and the matrix
// products have zeros where there is a weight (below 2^-126, and parts of larger ones).  Here a weight is zero only below 2^-149, as on the
// vector kernel.  (Beside finite values such weights add less than 2^-126 |V|.  Looked for in every step,
// by the smallest score, they were 1 to 6 % of the kernel; a second pass of its loop with positive parts
// cost 3 to 5 % by the registers that the two share.  12 clips of 24 frames x 135 positions, 5 heads of 64: 45 us
// a single call, 53 with a NaN and no infinity in every head, 870 with infinities in every head; the vector
// kernel 200.)
__device__ __forceinline__ bool infinity_in_v(const TileArgs &a, const Task &tk, const Context &cx)
{
    const int64_t C = (int64_t)a.h * a.D, FS = (int64_t)a.P * C;
    const __bf16 *V = (const __bf16 *)a.V + (int64_t)tk.p * C + (int64_t)tk.g * a.D;
    bool inf = false;
    for (int j = threadIdx.x & 63; j < cx.L; j += 64) {
        const __bf16 *v = V + key_row(a, cx, j) * FS;
        for (int d = 0; d < a.D; d += 8) {
            const bf16x8 x = *(const bf16x8 *)(v + d);
#pragma unroll
            for (int e = 0; e < 8; ++e) inf = inf || __builtin_fabsf((float)x[e]) == INFINITY;
        }
    }
    return __any(inf);
}
template <typename TO>
__device__ __forceinline__ void vector_task(const TileArgs &a, const Task &tk, const Context &cx)
{
    const int lane = threadIdx.x & 63, D = a.D;
    const int64_t C = (int64_t)a.h * D, FS = (int64_t)a.P * C;
    const int64_t rowoff = (int64_t)tk.p * C + (int64_t)tk.g * D;
    const __bf16 *K = (const __bf16 *)a.K + rowoff, *V = (const __bf16 *)a.V + rowoff;
    for (int i = 16 * tk.qt; i < min(16 * tk.qt + 16, a.clip_len); ++i) {
        const int aq = tk.clip * a.clip_len + i;
        const __bf16 *q = (const __bf16 *)a.Q + (int64_t)aq * FS + rowoff;
        // raw score of key j, -inf if it does not exist or is hidden
        auto score = [&](int j) -> float {
            const __bf16 *k = K + key_row(a, cx, j) * FS;
            float x = 0.f;
            for (int d = 0; d < D; d += 8) {
                const bf16x8 y = *(const bf16x8 *)(q + d), z = *(const bf16x8 *)(k + d);
#pragma unroll
                for (int e = 0; e < 8; ++e) x = fmaf((float)y[e], (float)z[e], x);
            }
            const int ki = key_info(a, cx, j), f = ki & 0x3fffffff;
            const bool far = a.window >= 0 && abs(f - aq) > a.window;
            const bool seen = (ki >> 30 & 1) || (f >= cx.lo && f < cx.lo + cx.nl && !far);
            return j >= cx.L || (j < cx.nl ? far : a.dedup && seen) ? -INFINITY : x;
        };
        float ml = -INFINITY, mg = -INFINITY;
        for (int j = lane; j < cx.L; j += 64) {
            const float x = score(j);
            ml = j < cx.nl ? fmaxf(ml, x) : ml;
            mg = j < cx.nl ? mg : fmaxf(mg, x);
        }
        for (int w = 32; w > 0; w >>= 1) {
            ml = fmaxf(ml, __shfl_xor(ml, w));
            mg = fmaxf(mg, __shfl_xor(mg, w));
        }
        const float ls = a.dedup && mg == -INFINITY ? 0.f : a.lb;
        const float m = fmaxf(ml + ls, mg + a.gb) * a.sc;
        float l = 0.f, o[3] = {0.f, 0.f, 0.f};  // channels lane, lane + 64, lane + 128
        for (int j0 = 0; j0 < cx.L; j0 += 64) {
            const int j = j0 + lane;
            const float w = exp2f(fmaf(score(j) + (j < cx.nl ? ls : a.gb), a.sc, -m));
            l += w;
            for (int u = 0; u < min(64, cx.L - j0); ++u) {
                const float wu = __shfl(w, u);
                const __bf16 *v = V + key_row(a, cx, j0 + u) * FS;
                for (int r = 0; r < 3; ++r)
                    if (lane + 64 * r < D) o[r] = fmaf(wu, (float)v[lane + 64 * r], o[r]);
            }
        }
        for (int w = 32; w > 0; w >>= 1) l += __shfl_xor(l, w);
        TO *out = (TO *)a.O + (int64_t)aq * FS + rowoff;
        for (int r = 0; r < 3; ++r)
            if (lane + 64 * r < D) out[lane + 64 * r] = (TO)(o[r] * (1.0f / l));
    }
}

// ---------------------------------------------------------------- bf16

// LDS of one wavefront: the V rows of two key tiles, padded so that the rows spread over the banks
constexpr int vrow_bytes(int NKB) { return 64 * NKB + 16; }
constexpr int kBf16Tiles = 2;  // key tiles per step

// NKB = ceil(D / 32)
template <int NKB, bool OUT_F32>
__global__ __launch_bounds__(256, NKB == 1 ? 6 : 2) void tile_attn_bf16_kernel(const TileArgs a)
{
    constexpr int KT = kBf16Tiles;
    constexpr int RS = vrow_bytes(NKB);
    __shared__ __attribute__((aligned(16))) unsigned char smem[4 * KT * 16 * RS];
    const Task tk = task_of(a);
    if (!tk.exists) return;
    const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
    unsigned char *vs = smem + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * (KT * 16 * RS);
    const int D = a.D;
    const int64_t C = (int64_t)a.h * D, FS = (int64_t)a.P * C;
    const int64_t rowoff = (int64_t)tk.p * C + (int64_t)tk.g * D;
    const int q0 = tk.qt * 16 + l16;
    const bool qok = q0 < a.clip_len;
    const int aq = tk.clip * a.clip_len + min(q0, a.clip_len - 1);
    const Context cx = context_of(a, tk.clip);

    // chunks 4 kb + lg of a row (zeros past the head; the others' lanes all exist)
    const bool last_ok = 32 * (NKB - 1) + 8 * lg < D;
    auto load_chunks = [&](const __bf16 *p, bool ok, bf16x8(&r)[NKB]) __attribute__((always_inline)) {
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
            r[kb] = bf16x8{};
            if (ok && (kb + 1 < NKB || last_ok)) r[kb] = *(const bf16x8 *)(p + 32 * kb);
        }
    };
    const int64_t laneoff = rowoff + 8 * lg;
    bf16x8 q[NKB];
    load_chunks((const __bf16 *)a.Q + (int64_t)aq * FS + laneoff, true, q);

    f32x4 o[NKB][2];
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) o[kb][0] = o[kb][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    Softmax<KT, false> sm(a);

    const int tiles = (cx.L + 15) / 16;
    bf16x8 kr[KT][NKB], vr[KT][NKB];
    // this lane's row of the first tile of consecutive rows
    const int64_t run0 = (cx.row0 + l16) * FS + laneoff;
    // (rows of V past the list are zeros: their weights are, and zero times an infinity is not)
    auto load_tiles = [&](int t0) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            const int j = 16 * (t0 + t) + l16;
            if (16 * (t0 + t) + 16 <= cx.run) {
                const int64_t at = run0 + (int64_t)(16 * (t0 + t)) * FS;
                load_chunks((const __bf16 *)a.K + at, true, kr[t]);
                load_chunks((const __bf16 *)a.V + at, true, vr[t]);
            } else if (t0 + t < tiles) {
                const int64_t at = key_row(a, cx, j) * FS + laneoff;
                load_chunks((const __bf16 *)a.K + at, true, kr[t]);
                load_chunks((const __bf16 *)a.V + at, j < cx.L, vr[t]);
            } else {
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb) vr[t][kb] = bf16x8{};
            }
        }
    };
    load_tiles(0);
    for (int t0 = 0; t0 < tiles; t0 += KT) {
        const int nt = min(KT, tiles - t0);
        f32x4 s[KT];
#pragma unroll
        for (int t = 0; t < KT; ++t) {
            s[t] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (t >= nt) continue;
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb)
                s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kr[t][kb], q[kb], s[t], 0, 0, 0);
        }
        // V through LDS, for the transposing read below; the next rows are asked for in the registers
        // that this frees
        wave_lds_sync();
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb)
                *(bf16x8 *)(vs + (16 * t + l16) * RS + 64 * kb + 16 * lg) = vr[t][kb];
        wave_lds_sync();
        load_tiles(t0 + KT);

        const float alpha = sm.step(a, cx, s, t0, nt, tk.clip, tk.qt, lane);
        if (__any(alpha != 1.f)) {
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                for (int u = 0; u < 2; ++u) o[kb][u] *= alpha;
        }
        // The weights as three bf16 numbers each: 8 bits, the next 8, and the 8 that are left.
        u32x4 w[3];
#pragma unroll
        for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int e = 0; e < 4; e += 2) {
                float x0 = s[t][e], x1 = s[t][e + 1];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const uint32_t b0 = __builtin_bit_cast(uint32_t, x0), b1 = __builtin_bit_cast(uint32_t, x1);
                    w[k][2 * t + e / 2] = __builtin_amdgcn_perm(b1, b0, 0x07060302);  // both high halves
                    x0 -= __builtin_bit_cast(float, b0 & 0xffff0000u);
                    x1 -= __builtin_bit_cast(float, b1 & 0xffff0000u);
                }
            }
        // V^T: within a group of 16 lanes the transposing read hands lane i element i % 4 of the 8
        // bytes that lanes i / 4, 4 + i / 4, 8 + i / 4 and 12 + i / 4 point at.  Lane i points at key
        // 4 lg + i / 4, channels 8 (i % 4) + 4 u .. of the block, and so gets keys 4 lg .. 4 lg + 3 of
        // channel 8 (i / 4) + 4 u + i % 4: the operand's layout, with the channels permuted so that a
        // lane ends up with eight neighbouring channels of its query.
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                s16x4 x[KT];
#pragma unroll
                for (int t = 0; t < KT; ++t)
                    x[t] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                        (__attribute__((address_space(3))) s16x4 *)(vs + (16 * t + 4 * lg + (l16 >> 2)) * RS +
                                                                    64 * kb + 16 * (l16 & 3) + 8 * u));
                const bf16x8 v = __builtin_bit_cast(bf16x8, __builtin_shufflevector(x[0], x[1], 0, 1, 2, 3, 4, 5,
                                                                                   6, 7));
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    o[kb][u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(v, __builtin_bit_cast(bf16x8, w[k]),
                                                                      o[kb][u], 0, 0, 0);
            }
    }

    bool nan = false;
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
        for (int u = 0; u < 2; ++u)
            nan = nan || __builtin_isunordered(o[kb][u][0], o[kb][u][1]) ||
                  __builtin_isunordered(o[kb][u][2], o[kb][u][3]);
    if (__any(nan) && infinity_in_v(a, tk, cx)) {
        vector_task<std::conditional_t<OUT_F32, float, __bf16>>(a, tk, cx);
        return;
    }
    const float inv = sm.inverse_sum();
    if (!qok) return;
#pragma unroll
    for (int kb = 0; kb < NKB; ++kb) {
        if (kb == NKB - 1 && !last_ok) break;
        const int64_t at = (int64_t)aq * FS + rowoff + 32 * kb + 8 * lg;
        if constexpr (OUT_F32) {
            *(f32x4 *)((float *)a.O + at) = o[kb][0] * inv;
            *(f32x4 *)((float *)a.O + at + 4) = o[kb][1] * inv;
        } else {
            bf16x8 y;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                y[e] = (__bf16)(o[kb][0][e] * inv);
                y[4 + e] = (__bf16)(o[kb][1][e] * inv);
            }
            *(bf16x8 *)((__bf16 *)a.O + at) = y;
        }
    }
}

// ---------------------------------------------------------------- fp32

template <int W>
struct Floats {
    typedef float type __attribute__((ext_vector_type(W)));
    static __device__ __forceinline__ float get(const type &x, int t) { return x[t]; }
};
template <>
struct Floats<1> {
    typedef float type;
    static __device__ __forceinline__ float get(const type &x, int) { return x; }
};

// NF blocks of 64 channels and, with WL = 1, 2 or 4, one of 16 WL channels: 64 NF < D <= 64 NF + 16 WL
template <int NF, int WL>
__global__ __launch_bounds__(256, NF == 0 && WL == 2 ? 7 : 2) void tile_attn_f32_kernel(const TileArgs a)
{
    constexpr int NC = 4 * NF + WL;  // 16-byte chunks per lane of a Q or K row; 16-channel tiles of O^T
    using Last = Floats<WL>;

    const Task tk = task_of(a);
    if (!tk.exists) return;
    const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
    const int D = a.D;
    const int64_t C = (int64_t)a.h * D, FS = (int64_t)a.P * C;
    const int64_t rowoff = (int64_t)tk.p * C + (int64_t)tk.g * D;
    const int q0 = tk.qt * 16 + l16;
    const bool qok = q0 < a.clip_len;
    const int aq = tk.clip * a.clip_len + min(q0, a.clip_len - 1);
    const Context cx = context_of(a, tk.clip);

    // chunks 4 j + lg of a row of Q or K (zeros past the head)
    auto load_chunks = [&](const float *p, f32x4(&r)[NC]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            if (j < 4 * NF) {  // (every lane's chunk exists)
                r[j] = *(const f32x4 *)(p + 16 * j);
            } else {
                r[j] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (16 * j + 4 * lg < D) r[j] = *(const f32x4 *)(p + 16 * j);
            }
        }
    };
    const int64_t laneoff = rowoff + 4 * lg;
    f32x4 q[NC];
    load_chunks((const float *)a.Q + (int64_t)aq * FS + laneoff, q);

    f32x4 o[NC];  // o[4 b + t]: channel 64 b + W m + t of row m, in block b of width W
#pragma unroll
    for (int j = 0; j < NC; ++j) o[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    Softmax<1, true> sm(a);

    const int tiles = (cx.L + 15) / 16;
    f32x4 kr[NC];
    f32x4 vf[4][NF ? NF : 1];    // [s: key 4 lg + s][block]
    typename Last::type vl[4];
    auto load_k = [&](int t) __attribute__((always_inline)) {
        const int j = 16 * t + l16;
        const int64_t row = 16 * t + 16 <= cx.run ? cx.row0 + j : key_row(a, cx, j);
        load_chunks((const float *)a.K + row * FS + laneoff, kr);
    };
    // (rows past the list are zeros: their weights are, and zero times an infinity is not)
    auto load_v = [&](int t) __attribute__((always_inline)) {
        const bool run = 16 * t + 16 <= cx.run;
        const int c = 64 * NF + WL * l16;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int j = 16 * t + 4 * lg + s;
            const bool ok = run || j < cx.L;
            const float *p = (const float *)a.V + (run ? cx.row0 + j : key_row(a, cx, j)) * FS + rowoff;
#pragma unroll
            for (int b = 0; b < NF; ++b) {
                vf[s][b] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (ok) vf[s][b] = *(const f32x4 *)(p + 64 * b + 4 * l16);
            }
            vl[s] = typename Last::type{};
            if (ok && c < D) vl[s] = *(const typename Last::type *)(p + c);
        }
    };
    load_k(0);
    load_v(0);
    for (int t = 0; t < tiles; ++t) {
        // (two chains: an instruction of one covers the latency of the other's)
        f32x4 s2[2] = {};
#pragma unroll
        for (int j = 0; j < NC; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                s2[e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(kr[j][e], q[j][e], s2[e & 1], 0, 0, 0);
        f32x4 s[1] = {s2[0] + s2[1]};
        if (t + 1 < tiles) load_k(t + 1);  // (K's registers are free again)

        const float alpha = sm.step(a, cx, s, t, 1, tk.clip, tk.qt, lane);
        if (__any(alpha != 1.f)) {
#pragma unroll
            for (int j = 0; j < NC; ++j) o[j] *= alpha;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
#pragma unroll
            for (int b = 0; b < NF; ++b)
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    o[4 * b + u] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[e][b][u], s[0][e], o[4 * b + u], 0, 0, 0);
#pragma unroll
            for (int u = 0; u < WL; ++u)
                o[4 * NF + u] =
                    __builtin_amdgcn_mfma_f32_16x16x4f32(Last::get(vl[e], u), s[0][e], o[4 * NF + u], 0, 0, 0);
        }
        if (t + 1 < tiles) load_v(t + 1);
    }

    const float inv = sm.inverse_sum();
    if (!qok) return;
    float *op = (float *)a.O + (int64_t)aq * FS + rowoff;
#pragma unroll
    for (int b = 0; b <= NF; ++b) {
        const int W = b < NF ? 4 : WL;
        // the lane's 4 W channels 64 b + W (4 lg + e) + t are contiguous, D a multiple of four
#pragma unroll
        for (int u = 0; u < W; ++u) {
            const int c = 64 * b + 4 * W * lg + 4 * u;
            f32x4 y;
#pragma unroll
            for (int x = 0; x < 4; ++x) y[x] = o[4 * b + (4 * u + x) % W][(4 * u + x) / W] * inv;
            if (c < D) *(f32x4 *)(op + c) = y;
        }
    }
}

const void *bf16_fn(int D, bool out_f32)
{
#define DSATTN_TILE_BF16(NKB)                                              \
    case NKB:                                                              \
        return out_f32 ? (const void *)&tile_attn_bf16_kernel<NKB, true>   \
                       : (const void *)&tile_attn_bf16_kernel<NKB, false>;
    switch ((D + 31) / 32) {
        DSATTN_TILE_BF16(1)
        DSATTN_TILE_BF16(2)
        DSATTN_TILE_BF16(3)
        DSATTN_TILE_BF16(4)
        DSATTN_TILE_BF16(5)
    default: return nullptr;
    }
#undef DSATTN_TILE_BF16
}

const void *f32_fn(int D)
{
    const struct {
        int max;
        const void *fn;
    } table[] = {
        {16, (const void *)&tile_attn_f32_kernel<0, 1>},  {32, (const void *)&tile_attn_f32_kernel<0, 2>},
        {64, (const void *)&tile_attn_f32_kernel<0, 4>},  {80, (const void *)&tile_attn_f32_kernel<1, 1>},
        {96, (const void *)&tile_attn_f32_kernel<1, 2>},  {128, (const void *)&tile_attn_f32_kernel<1, 4>},
        {144, (const void *)&tile_attn_f32_kernel<2, 1>}, {160, (const void *)&tile_attn_f32_kernel<2, 2>},
    };
    for (const auto &t : table)
        if (D <= t.max) return t.fn;
    return nullptr;
}

}  // namespace

// The kernel for a plan's type and head size, if there is one.
void tile_attn_plan(dsattn_plan_t &pl)
{
    const dsattn_desc &d = pl.desc;
    // A launch has less than 2^32 threads (64 a task, whole workgroups on every XCD); above, the vector
    // kernel takes what it can.  (Tasks are numbered in 31 bits; a plan's frame numbers have 24: room for
    // the flag beside them.)
    const int64_t nqt = (d.clip_len + 15) / 16, units = (int64_t)d.n_clips * d.spatial * d.heads;
    constexpr int64_t kMaxTasks = (((int64_t)1 << 32) / (8 * 256) - 1) * 32;
    if (units > kMaxTasks / nqt) return;
    // rows are whole 16-byte chunks
    const bool f32 = d.io_dtype == DSATTN_F32;
    if (d.head_dim % (f32 ? 4 : 8) != 0) return;
    pl.tile_fn = f32 ? f32_fn(d.head_dim) : bf16_fn(d.head_dim, d.out_dtype == DSATTN_F32);
    if (!pl.tile_fn) return;
    pl.launch.n_tasks = (int32_t)(units * nqt);
    pl.launch.block_threads = 256;
    pl.launch.lds_bytes = f32 ? 0 : 4 * kBf16Tiles * 16 * vrow_bytes((d.head_dim + 31) / 32);
}

hipError_t launch_tile_attn(const dsattn_plan_t &pl, const void *Q, const void *K, const void *V, void *O,
                            bool ctx_mode, hipStream_t st)
{
    const dsattn_desc &d = pl.desc;
    TileArgs a;
    a.Q = Q;
    a.K = K;
    a.V = V;
    a.O = O;
    a.gidx = pl.d_global_idx;
    a.N = d.n_clips;
    a.F = pl.F;
    a.wl = d.local_ctx;
    a.P = d.spatial;
    a.h = d.heads;
    a.D = d.head_dim;
    a.clip_len = d.clip_len;
    a.lk_max = pl.lk_max;
    a.nqt = (d.clip_len + 15) / 16;
    a.ctx_mode = ctx_mode ? 1 : 0;
    a.G = (int32_t)pl.global_idx.size();
    a.window = pl.window;
    a.dedup = (d.flags & DSATTN_FLAG_DEDUP_GLOBAL) ? 1 : 0;
    a.tasks = (uint32_t)d.n_clips * d.spatial * d.heads * a.nqt;
    a.per_xcd = (a.tasks + 4 * 8 - 1) / (4 * 8);
    // A softmax sees only the difference of the two biases.  It is taken from the lighter scope's scores:
    // added to the heavier one's, which are the ones that count, it would take their low bits (a local
    // bias of -1e4 cost 1e-4 of the result, one of -1e9 all of the scores).  A heavier bias of 2^64 and
    // more swallows the scores beside it in 64 bits too: every key of that scope weighs the same, as on
    // the vector kernel.
    const bool swallows = std::fabs(a.G ? std::max(d.bias_local, d.bias_global) : d.bias_local) >= 0x1p64f;
    a.sc = swallows ? 1e-30f : pl.scale * 1.4426950408889634f;
    const double diff = a.G ? ((double)d.bias_global - d.bias_local) * 1.4426950408889634 / a.sc : 0.0;
    const double hides = 3e38 / std::max(a.sc, 1.f);  // (any scope; times sc it is still finite)
    a.lb = (float)std::max(std::min(-diff, 0.0), -hides);
    a.gb = (float)std::max(std::min(diff, 0.0), -hides);
    void *params[] = {&a};
    return hipLaunchKernel(pl.tile_fn, dim3(a.per_xcd * 8), dim3(256), params, 0, st);
}

}  // namespace dsattn
