// Dual-scope attention on the matrix cores for what the streaming kernel does not take: fp32
// tensors, clips that are not whole 16-frame tiles, local scopes that reach further than its ring,
// longer global lists.  Precision is that of the vector kernel: fp32 softmax, weights kept at 24
// bits.
//
// One wavefront owns 16 or 32 query frames of one clip, position and head and walks the clip's context list
// in tiles of 16 keys with a running maximum.  Rows are fetched with four neighbouring lanes on 64
// neighbouring bytes and pass through a few KB of wavefront-private LDS into the operand layout.  (Fetched in
// the operand layout itself, 16 rows to 16 neighbouring lanes, every lane was an access of its own to the
// first-level cache, which was then busy for the whole of the kernel: 49 to 54 accesses an instruction instead of 15,
// fp32 28 instead of 13, and 12 clips of 24 frames of 64 global ones, 370 positions, 8 x 160: 590 -> 402 us.)
//   S^T = K Q^T   keys on M, queries on N.  The lane's 16 bytes are chunk 4 j + lane / 16 of row
//                 lane % 16, in both operands, so any order of the channels contracts the same:
//                 one operand of v_mfma_f32_16x16x32_bf16, or four of v_mfma_f32_16x16x4_f32.
//   O^T = V^T P^T fp32: v_mfma_f32_16x16x4_f32; lane (m, k) loads W consecutive channels 64 b + W m of
//                 key 4 k + s, the operands of W products, and the weight it holds of that key is the
//                 other operand as it stands.
//                 bf16: v_mfma_f32_16x16x32_bf16 over a pair of key tiles (an odd one: 16x16x16); a weight
//                 enters as the sum of three bf16 numbers (8 bits each: all 24), whose products are exact.
//
// What bounds it: at short context lists HBM and the vector instructions of softmax and splitting (which keep the
// vector ALUs busy for half of the time).  Tasks are numbered so that one XCD works through consecutive clips of one position: the
// global frames and the boundary frames that neighbouring clips share are then in its L2, and measured
// HBM reads are the tensors' own size.  Tensors from HBM: 12 clips of 24 frames x 135 positions, 5 x 64, bf16: 25.2 us
// (35.6 with operand-order loads; 19.4 at the card's copy rate); 2,304 positions x 2 clips of 25, 8 x 80: 162 (213);
// 3 clips of 24 x 925 positions, 8 x 80, fp32: 195 (230).
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
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

struct TileArgs {
    const void *Q, *K, *V;
    void *O;
    const int32_t *ginfo;  // global entries: frame, bit 30 where an earlier entry has the same frame
    int32_t N, F, P, h, D, clip_len, lk_max;
    int32_t wl;        // local context width of a clip
    int32_t nqg;       // tasks (groups of query tiles) per clip
    int32_t ctx_mode;  // K and V are materialised contexts [N, lk_max, P, C]
    int32_t G, window, dedup;
    uint32_t per_xcd;  // workgroups per XCD
    uint32_t tasks;
    uint32_t fsb;      // from a frame to the next one, in units of 16 bytes
    float sc;          // scale * log2(e)
    float lb, gb;      // shifts of the local and the global keys' raw scores, see launch_tile_attn
};

// One wavefront's share: queries [q0, q0 + nq) of one clip, position and head.
struct Task {
    int clip, p, g, q0, nq;
    bool exists;
};
// (clips of one position are neighbours: numbered the other way round, positions fastest, it
// measured up to 7 % slower)
template <int QT>
__device__ __forceinline__ Task task_of(const TileArgs &a)
{
    // XCD x (= workgroup % 8) takes a contiguous run of tasks
    const uint32_t wg = (blockIdx.x % 8u) * a.per_xcd + blockIdx.x / 8u;
    // (less than 2^31 tasks: 32-bit divisions, a 64-bit one is some hundred scalar instructions)
    uint32_t id = wg * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Task k;
    k.exists = id < a.tasks;
    id = min(id, a.tasks - 1);
    uint32_t rest = id / (uint32_t)a.nqg;
    const int qg = (int)(id - rest * a.nqg);
    id = rest;
    rest = id / (uint32_t)a.h;
    k.g = (int)(id - rest * a.h);
    k.p = (int)(rest / (uint32_t)a.N);
    k.clip = (int)(rest - (uint32_t)k.p * a.N);
    k.q0 = k.clip * a.clip_len + 16 * QT * qg;
    k.nq = min(16 * QT, a.clip_len - 16 * QT * qg);
    return k;
}

// The task's context list: the local frames [lo, lo + nl) that any of its queries sees, then the global
// entries; L keys in all.  (Worked out here and not read from the plan's table: the first key rows are
// then asked for at once.)  Rows of K and V are counted from row `base`: local key j is row lrow + j, and
// global entry i of a materialised context row grow + i.
struct Context {
    int lo, nl, L, lrow, grow;
    int64_t base;
};
__device__ __forceinline__ Context context_of(const TileArgs &a, const Task &k)
{
    Context c;
    const int lo = max(0, k.clip * a.clip_len - a.wl), hi = min(a.F, (k.clip + 1) * a.clip_len + a.wl);
    // under a window, what the task's first and last query see: 383 positions of a clip of 192 frames, 10 x 64,
    // fp32, with a window of 8 (3 or 4 key tiles instead of 13): 572 -> 177 us
    c.lo = a.window < 0 ? lo : max(lo, k.q0 - a.window);
    c.nl = (a.window < 0 ? hi : min(hi, k.q0 + k.nq + a.window)) - c.lo;
    c.L = c.nl + a.G;
    c.base = a.ctx_mode ? (int64_t)k.clip * a.lk_max : 0;
    c.lrow = a.ctx_mode ? c.lo - lo : c.lo;
    c.grow = hi - lo;
    return c;
}

// The local frames [lo, lo + span) that a query sees.
struct Visible {
    int lo;
    uint32_t span;
    __device__ __forceinline__ bool sees(int frame) const { return (uint32_t)(frame - lo) < span; }
};
__device__ __forceinline__ Visible visible_to(const TileArgs &a, const Context &c, int aq)
{
    int lo = c.lo, hi = c.lo + c.nl;
    if (a.window >= 0) {
        lo = max(lo, aq - a.window);
        hi = min(hi, aq + a.window + 1);
    }
    return {lo, (uint32_t)(hi - lo)};
}

// The plan's table of global entries, in LDS as far as it fits (read from memory in the loop, an entry
// would be waited for behind the rows that are on their way).
constexpr int kLdsGlobals = 256;
typedef __attribute__((address_space(3))) const int lds_int;
struct Globals {
    const TileArgs &a;
    lds_int *lds;
    __device__ __forceinline__ int operator[](int i) const
    {
        i = min(max(i, 0), a.G - 1);
        if (a.G <= kLdsGlobals) return lds[i];
        return a.ginfo[i];
    }
};

// The table's way into LDS: a thread's entry on its way, and all of them there.
__device__ __forceinline__ bool needs_globals(const TileArgs &a)
{
    return a.G > 0 && a.G <= kLdsGlobals && (!a.ctx_mode || a.dedup);
}
__device__ __forceinline__ int my_global(const TileArgs &a)
{
    return needs_globals(a) ? a.ginfo[min((int)threadIdx.x, a.G - 1)] : 0;
}
__device__ __forceinline__ void put_globals(const TileArgs &a, int *lds, int mine)
{
    if (!needs_globals(a)) return;
    lds[threadIdx.x] = mine;
    __syncthreads();
}

// row of key j, one of tile t's, in K and V, from the context's base on (keys past the list: the last one's,
// their weights are zero)
__device__ __forceinline__ uint32_t key_row(const TileArgs &a, const Context &c, const Globals &g, int t, int j)
{
    j = min(j, c.L - 1);
    uint32_t row = (uint32_t)(c.lrow + j);
    if (16 * t + 16 > c.nl && a.G > 0) {
        const int i = max(j - c.nl, 0);
        const uint32_t gr = a.ctx_mode ? (uint32_t)(c.grow + i) : (uint32_t)g[i] & 0x3fffffffu;
        row = j < c.nl ? row : gr;
    }
    return row;
}
// The wavefront's position and head of a row: rows are 16 fsb bytes apart.
template <typename T>
__device__ __forceinline__ const T *row_ptr(const T *p, uint32_t row, uint32_t fsb)
{
    return (const T *)((const unsigned char *)p + ((uint64_t)row * fsb << 4));
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

// What a kernel is compiled for: no option; biases of the scopes; a window (and biases); the set union without a
// window over up to 63 global frames (and biases); any.  Apart, because the conditions alone, kept in scalar registers and spilled from
// there, were a third of the plain loop's instructions (12 clips of 24 frames x 135 positions, 5 x 64, tensors in the
// caches: 28.3 -> 25.5 us without them).  What an option costs is instructions per score and registers: in the kernel
// for all of them a bias alone takes the union's and the window's conditions along, and the union looks every global
// key up in LDS and compares its frame for every query tile and key tile, though the answer is a task's, not a query's.
// Against that kernel, 16 global frames, us, bias of the global scope; union; both; window of 8 (no option):
//   91 clips of 24 frames x 246 positions, 4 x 32   188.3 -> 174.9  196.7 -> 174.2  208.9 -> 177.1  (as before)      (162)
//   40 clips of 24 frames x 100 positions, 10 x 64  123.8 -> 115.0  129.3 -> 121.5  132.4 -> 124.3  127.7 -> 127.4  (113)
//   40 clips of 25 frames x 100 positions, 8 x 160  265.6 -> 260.4  274.9 -> 260.4  277.3 -> 264.4  256.1 -> 252.5  (257)
//   90 clips of 8 frames x 135 positions, 6 x 96    135.8 -> 118.1  148.2 -> 118.0  152.7 -> 118.8  139.0 -> 119.0  (117)
//   40 clips of 24 frames x 100 positions, 5 x 64, fp32  133.0 -> 132.0  136.2 -> 132.2  137.3 -> 133.9  146 -> 146  (126)
// fp32 under a window of 8, 40 clips of 24 frames, the kernel for any option and its own: head_dim 16 215.5 and 214.3,
// 32 157.4 and 156.4, 48 137.0 and 136.0, 80 281.9 and 281.6, 96 207.3 and 206.6, 128 297 and 260, 144 235.4 and 228.8,
// 160 322.7 and 313.2; 10 clips of 96 frames, 32 132.1 and 127.7, 64 129.9 and 128.5, 80 251.8 and 250.0, 96 183.5 and
// 179.6, 128 271 and 228.
// With the set union a window makes what is hidden a query's own, and more than 63 global frames do not fit one word:
// these stay with the kernel for any option.
enum { kPlain, kBiases, kWindow, kUnion, kAll };
constexpr int kUnionGlobals = 63;

// The global entries, bit i the i-th, that the set union hides from every query of a task: the ones whose frame is a
// local one or an earlier entry's; and those past the list.  (Up to 63: bit 63 says so of what lies beyond.)
__device__ __forceinline__ uint64_t hidden_entries(const TileArgs &a, const Context &c, const Globals &g)
{
    const int i = threadIdx.x & 63;
    bool hidden = i >= a.G;
    if (a.dedup && a.G > 0) {
        const int ki = g[i], frame = ki & 0x3fffffff;
        hidden = hidden || (ki >> 30 & 1) || (frame >= c.lo && frame < c.lo + c.nl);
    }
    return __ballot(hidden);
}

// The part of the kernel that both types share: masks, running softmax.
template <bool POSITIVE, int OPTS>
struct Softmax {
    float m = -INFINITY, l = 0.f;  // running maximum of the query's column; this lane's part of the sum
    // A shift of the local scores holds from the query's first visible global key on: the set union may
    // hide them all, and then it is the local scores that count.
    bool shifted = false;

    // scores of key tiles t0 .. t0 + KT - 1 -> weights (unnormalised; those of keys past the list are zero);
    // returns the factor for what has been accumulated so far
    template <int KT>
    __device__ __forceinline__ float step(const TileArgs &a, const Context &c, const Globals &g, uint64_t hide, int aq,
                                          f32x4 (&s)[KT], int t0, int lane)
    {
        const int lg = lane >> 4, j0 = 16 * t0 + 4 * lg;
        if (OPTS == kUnion) {
            // (a lane's four keys are four bits in a row; local ones are never hidden)
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                if (16 * (t0 + t) + 16 <= c.nl) continue;
                const int at = j0 + 16 * t - c.nl;  // -15 and up
                const uint32_t bits = (uint32_t)(at < 0 ? hide << -at : (uint64_t)((int64_t)hide >> min(at, 63)));
#pragma unroll
                for (int e = 0; e < 4; ++e) s[t][e] = bits >> e & 1 ? -INFINITY : s[t][e];
            }
        } else if (OPTS == kWindow) {
            const Visible vis = visible_to(a, c, aq);
            const int from = j0 + c.lo - vis.lo;
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                const int first = 16 * (t0 + t);
                if (first >= c.nl && first + 16 <= c.L) continue;  // global keys only, and no padding
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int j = j0 + 16 * t + e;
                    bool hidden = (uint32_t)(from + 16 * t + e) >= vis.span;
                    if (first + 16 > c.nl) hidden = j < c.nl ? hidden : j >= c.L;
                    s[t][e] = hidden ? -INFINITY : s[t][e];
                }
            }
        } else if (OPTS == kAll && (a.window >= 0 || a.dedup)) {
            const Visible vis = visible_to(a, c, aq);
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                const bool globals = 16 * (t0 + t) + 16 > c.nl;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int j = j0 + 16 * t + e;
                    bool hidden = !vis.sees(c.lo + j);
                    if (globals) {
                        const int ki = a.dedup ? g[j - c.nl] : 0;
                        const bool seen = a.dedup && ((ki >> 30 & 1) || vis.sees(ki & 0x3fffffff));
                        hidden = j < c.nl ? hidden : seen || j >= c.L;
                    }
                    s[t][e] = hidden ? -INFINITY : s[t][e];
                }
            }
        } else if (16 * (t0 + KT) > c.L) {  // else every key counts
            int left = c.L - j0;
            asm volatile("" : "+v"(left));  // (or the comparisons are made in every step)
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) s[t][e] = 16 * t + e >= left ? -INFINITY : s[t][e];
        }
        if (OPTS && (a.lb != 0.f || a.gb != 0.f)) {
            if (OPTS > kWindow && a.dedup && a.lb != 0.f) {
                float mg = -INFINITY;
#pragma unroll
                for (int t = 0; t < KT; ++t)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (j0 + 16 * t + e >= c.nl) mg = fmaxf(mg, s[t][e]);
                const bool first = !shifted && swap32(swap16(mg, true), true) > -INFINITY;
                m += first ? a.lb * a.sc : 0.f;
                shifted = shifted || first;
            }
            const float ls = OPTS <= kWindow || shifted || !a.dedup ? a.lb : 0.f;
#pragma unroll
            for (int t = 0; t < KT; ++t) {
                const int from = 16 * (t0 + t);
                // A branch less here is registers less: the others' three ways, or the same test worded as
                // `from + 16 <= c.nl`, cost the fp32 kernels 2 to 10 and with them a wavefront a SIMD at head_dim 24, 32, 48, 72 and 80.
                // us, 40 clips of 24 frames, window and union of 16 / union of 70 global frames, with that and so: 246
                // positions, 4 x 32, 173.4 and 165.1 / 376 and 349; 100, 6 x 48, 147.7 and 141.8 / 311 and 284; 100, 8 x 80, 308 and
                // 287 / 623 and 557; union of 16 alone (fp32), 100, 6 x 48, 149.3 and 136.7.
                if (OPTS == kAll || (POSITIVE && OPTS == kUnion)) {
                    const bool globals = from + 16 > c.nl;
                    if (!globals && ls == 0.f) continue;
#pragma unroll
                    for (int e = 0; e < 4; ++e) s[t][e] += !globals || j0 + 16 * t + e < c.nl ? ls : a.gb;
                } else if (from + 16 <= c.nl) {  // one of lb and gb is zero
                    if (a.lb != 0.f) s[t] += ls;
                } else if (from >= c.nl) {
                    if (a.gb != 0.f) s[t] += a.gb;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) s[t][e] += j0 + 16 * t + e < c.nl ? ls : a.gb;
                }
            }
        }
        float mx = -INFINITY;
#pragma unroll
        for (int t = 0; t < KT; ++t)
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
        for (int t = 0; t < KT; ++t)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x = fmaf(s[t][e], a.sc, nm);
                s[t][e] = POSITIVE ? exp2_positive(x) : __builtin_amdgcn_exp2f(x);
                l += s[t][e];
            }
        return alpha;
    }
    __device__ __forceinline__ float inverse_sum() const
    {
        return 1.0f / swap32(swap16(l, false), false);
    }
};

// A bf16 task whose result has a NaN and whose V rows have an infinity is done again, one query at a time
// on the vector ALUs: zero times an infinity in V is NaN, a small weight times it is not, and the matrix
// products have zeros where there is a weight (below 2^-126, and parts of larger ones).  Here a weight is zero only below 2^-149, as on the
// vector kernel.  (Beside finite values such weights add less than 2^-126 |V|.  Looked for in every step,
// by the smallest score, they were 1 to 6 % of the kernel; a second pass of its loop with positive parts
// cost 3 to 5 % by the registers that the two share.  12 clips of 24 frames x 135 positions, 5 heads of 64: 45 us
// a single call, 53 with a NaN and no infinity in every head, 870 with infinities in every head; the vector
// kernel 200.)
__device__ __forceinline__ bool infinity_in_v(const TileArgs &a, const Task &tk, const Context &cx, const Globals &gl)
{
    const int64_t C = (int64_t)a.h * a.D, FS = (int64_t)a.P * C;
    const __bf16 *V = (const __bf16 *)a.V + cx.base * FS + (int64_t)tk.p * C + (int64_t)tk.g * a.D;
    bool inf = false;
    for (int j = threadIdx.x & 63; j < cx.L; j += 64) {
        const __bf16 *v = row_ptr(V, key_row(a, cx, gl, j >> 4, j), a.fsb);
        for (int d = 0; d < a.D; d += 8) {
            const bf16x8 x = *(const bf16x8 *)(v + d);
#pragma unroll
            for (int e = 0; e < 8; ++e) inf = inf || __builtin_fabsf((float)x[e]) == INFINITY;
        }
    }
    return __any(inf);
}
template <typename TO>
__device__ __forceinline__ void vector_task(const TileArgs &a, const Task &tk, const Context &cx, const Globals &gl,
                                           int from, int to)
{
    const int lane = threadIdx.x & 63, D = a.D;
    const int64_t C = (int64_t)a.h * D, FS = (int64_t)a.P * C;
    const int64_t rowoff = (int64_t)tk.p * C + (int64_t)tk.g * D;
    const __bf16 *K = (const __bf16 *)a.K + cx.base * FS + rowoff, *V = (const __bf16 *)a.V + cx.base * FS + rowoff;
    for (int aq = from; aq < to; ++aq) {
        const Visible vis = visible_to(a, cx, aq);
        const __bf16 *q = (const __bf16 *)a.Q + (int64_t)aq * FS + rowoff;
        // raw score of key j, -inf if it does not exist or is hidden
        auto score = [&](int j) -> float {
            const __bf16 *k = row_ptr(K, key_row(a, cx, gl, j >> 4, j), a.fsb);
            float x = 0.f;
            for (int d = 0; d < D; d += 8) {
                const bf16x8 y = *(const bf16x8 *)(q + d), z = *(const bf16x8 *)(k + d);
#pragma unroll
                for (int e = 0; e < 8; ++e) x = fmaf((float)y[e], (float)z[e], x);
            }
            if (j >= cx.L) return -INFINITY;
            if (j < cx.nl) return vis.sees(cx.lo + j) ? x : -INFINITY;
            const int ki = a.dedup ? gl[j - cx.nl] : 0;
            return a.dedup && ((ki >> 30 & 1) || vis.sees(ki & 0x3fffffff)) ? -INFINITY : x;
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
                const __bf16 *v = row_ptr(V, key_row(a, cx, gl, (j0 + u) >> 4, j0 + u), a.fsb);
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

// Wavefronts per SIMD that the kernel's registers have to leave room for: as many as the loop over pairs alone leaves.
// (With one less, clips of 8 frames, two key tiles: 42.4 -> 45.7 us at head_dim 64, 52.8 -> 59.5 at 80; with the set
// union at 96: 118 -> 133.)  Two under a window or the set union elsewhere, where more would spill with bf16 output
// (under a window with fp32 output five at 64 and four at 72 to 88 fit, and are not asked for): the compiler then
// reaches one wavefront less than the plain kernel.
constexpr int bf16_waves(int NKB, bool FULL, int QT, int OPTS)
{
    return QT == 2 ? 2 : NKB == 1 ? 6 : OPTS > kBiases ? (NKB == 3 && FULL && OPTS < kAll ? 4 : 2) : NKB == 2 && FULL ? 5 : NKB == 3 ? 4 : 2;
}

// NKB = ceil(D / 32); FULL: D = 32 NKB.  QT query tiles share every key row that is fetched.
template <int NKB, bool FULL, int QT, int OPTS, bool OUT_F32>
__global__ __launch_bounds__(256, bf16_waves(NKB, FULL, QT, OPTS)) void tile_attn_bf16_kernel(const TileArgs a)
{
    constexpr int KT = kBf16Tiles;
    constexpr int RS = vrow_bytes(NKB);
    __shared__ __attribute__((aligned(16))) unsigned char smem[4 * KT * 16 * RS];
    __shared__ int gtab[kLdsGlobals];
    const int ginfo = my_global(a);
    const Globals gl{a, (lds_int *)gtab};
    const Task tk = task_of<QT>(a);  // (without a task: the last one's rows, up to the barrier)
    const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
    unsigned char *vs = smem + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * (KT * 16 * RS);
    const int D = a.D;
    const int64_t C = (int64_t)a.h * D, FS = (int64_t)a.P * C;
    const int64_t rowoff = (int64_t)tk.p * C + (int64_t)tk.g * D;
    const Context cx = context_of(a, tk);

    // Rows are fetched four lanes to a row, 64 neighbouring bytes: lane l has chunks 4 kb + l % 4 of row l / 4
    // (past the head: nothing).
    const int lr = lane >> 2, lc = lane & 3;
    const bool last_ok = FULL || 32 * (NKB - 1) + 8 * lc < D;
    auto load_chunks = [&](const __bf16 *p, bf16x8(&r)[NKB]) __attribute__((always_inline)) {
#pragma unroll
        for (int kb = 0; kb + 1 < NKB; ++kb) r[kb] = *(const bf16x8 *)(p + 32 * kb);
        if (last_ok) r[NKB - 1] = *(const bf16x8 *)(p + 32 * (NKB - 1));
    };
    const int64_t laneoff = rowoff + 8 * lc;
    // and written to rows 16 t + .. of the wavefront's LDS (past the head, whatever the register holds: to the
    // row's padding; those chunks stay zero)
    const int put_at = lr * RS + 16 * lc, put_last = lr * RS + (last_ok ? 64 * (NKB - 1) + 16 * lc : 64 * NKB);
    auto put_rows = [&](int t, const bf16x8(&r)[NKB]) __attribute__((always_inline)) {
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
            *(bf16x8 *)(vs + 16 * t * RS + (FULL || kb + 1 < NKB ? put_at + 64 * kb : put_last)) = r[kb];
    };
    if constexpr (!FULL) {
        for (int i = lane; i < KT * RS; i += 64) *(bf16x8 *)(vs + 16 * i) = bf16x8{};
        wave_lds_sync();
    }
    // chunk 4 kb + lane / 16 of row lane % 16 from there: an operand of the matrix instructions
    auto fragment = [&](int t, int kb) __attribute__((always_inline)) {
        return *(const bf16x8 *)(vs + (16 * t + l16) * RS + 64 * kb + 16 * lg);
    };

    const int tiles = (cx.L + 15) / 16;
    const __bf16 *Kw = (const __bf16 *)a.K + cx.base * FS + laneoff, *Vw = (const __bf16 *)a.V + cx.base * FS + laneoff;
    bf16x8 kr[KT][NKB], vr[KT][NKB];
    auto load_tile = [&](int t, int t0) __attribute__((always_inline)) {
        const uint32_t row = key_row(a, cx, gl, t0 + t, 16 * (t0 + t) + lr);
        load_chunks(row_ptr(Kw, row, a.fsb), kr[t]);
        load_chunks(row_ptr(Vw, row, a.fsb), vr[t]);
    };
    bf16x8 q[QT][NKB];
#pragma unroll
    for (int u = 0; u < QT; ++u) {
        const int aq = tk.q0 + min(16 * u + lr, tk.nq - 1);
        load_chunks(row_ptr((const __bf16 *)a.Q + laneoff, aq, a.fsb), q[u]);
    }
    // (the first rows, where they need no table, are asked for before it is waited for)
    const bool odd = tiles & 1, early = 16 * (odd ? 1 : KT) <= cx.nl;
    auto load_first = [&]() __attribute__((always_inline)) {
        load_tile(0, 0);
        if (!odd) load_tile(1, 0);
    };
    if (early) load_first();
    put_globals(a, gtab, ginfo);
    if (!tk.exists) return;
    if (!early) load_first();
    static_assert(QT <= KT, "the query rows fit");
#pragma unroll
    for (int u = 0; u < QT; ++u) put_rows(u, q[u]);
    wave_lds_sync();
#pragma unroll
    for (int u = 0; u < QT; ++u)
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) q[u][kb] = fragment(u, kb);
    wave_lds_sync();

    f32x4 o[QT][NKB][2];
#pragma unroll
    for (int u = 0; u < QT; ++u)
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) o[u][kb][0] = o[u][kb][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    Softmax<false, OPTS> sm[QT];
    const uint64_t hide = OPTS == kUnion ? hidden_entries(a, cx, gl) : 0;

    auto key_tiles = [&](auto n, int t0) __attribute__((always_inline)) {
        constexpr int KT = decltype(n)::value;  // of them in this step
        f32x4 s[QT][KT];
        // K through LDS, then V in its place; the next rows are asked for in the registers that this frees.
#pragma unroll
        for (int t = 0; t < KT; ++t) put_rows(t, kr[t]);
        wave_lds_sync();
#pragma unroll
        for (int t = 0; t < KT; ++t) {
#pragma unroll
            for (int u = 0; u < QT; ++u) s[u][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb) {
                const bf16x8 k = fragment(t, kb);
#pragma unroll
                for (int u = 0; u < QT; ++u)
                    s[u][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k, q[u][kb], s[u][t], 0, 0, 0);
            }
        }
        wave_lds_sync();
        // (rows of V past the list are zeros: their weights are, and zero times an infinity is not)
        if (16 * (t0 + KT) > cx.L) {
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb)
                    vr[t][kb] = 16 * (t0 + t) + lr < cx.L ? vr[t][kb] : bf16x8{};
        }
#pragma unroll
        for (int t = 0; t < KT; ++t) put_rows(t, vr[t]);
        wave_lds_sync();
        if (t0 + KT < tiles) {
#pragma unroll
            for (int t = 0; t < kBf16Tiles; ++t) load_tile(t, t0 + KT);
        }

#pragma unroll
        for (int u = 0; u < QT; ++u) {
            if (u > 0 && 16 * u >= tk.nq) break;
            const float alpha = sm[u].step(a, cx, gl, hide, tk.q0 + min(16 * u + l16, tk.nq - 1), s[u], t0, lane);
            if (__any(alpha != 1.f)) {
#pragma unroll
                for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                    for (int x = 0; x < 2; ++x) o[u][kb][x] *= alpha;
            }
            // The weights as three bf16 numbers each: 8 bits, the next 8, and the 8 that are left.
            uint32_t w[3][2 * KT];
#pragma unroll
            for (int t = 0; t < KT; ++t)
#pragma unroll
                for (int e = 0; e < 4; e += 2) {
                    float x0 = s[u][t][e], x1 = s[u][t][e + 1];
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
            // 4 lg + i / 4, channels 8 (i % 4) + 4 x .. of the block, and so gets keys 4 lg .. 4 lg + 3 of
            // channel 8 (i / 4) + 4 x + i % 4: the operand's layout, with the channels permuted so that a
            // lane ends up with eight neighbouring channels of its query.  (Read again for the second query
            // tile: kept, they would cost a quarter of the wavefronts.)
            wave_lds_sync();
#pragma unroll
            for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
                for (int x = 0; x < 2; ++x) {
                    s16x4 r[KT];
#pragma unroll
                    for (int t = 0; t < KT; ++t)
                        r[t] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                            (__attribute__((address_space(3))) s16x4 *)(vs + (16 * t + 4 * lg + (l16 >> 2)) * RS +
                                                                        64 * kb + 16 * (l16 & 3) + 8 * x));
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        if constexpr (KT == 2) {
                            const u32x4 wk = {w[k][0], w[k][1], w[k][2], w[k][3]};
                            o[u][kb][x] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                __builtin_bit_cast(bf16x8, __builtin_shufflevector(r[0], r[1], 0, 1, 2, 3, 4, 5, 6, 7)),
                                __builtin_bit_cast(bf16x8, wk), o[u][kb][x], 0, 0, 0);
                        } else {
                            const u32x2 wk = {w[k][0], w[k][1]};
                            o[u][kb][x] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(
                                r[0], __builtin_bit_cast(s16x4, wk), o[u][kb][x], 0, 0, 0);
                        }
                    }
                }
        }
    };
    // An odd tile goes alone, and first: behind the pairs it cost them two to four registers, and in some forms a
    // wavefront.  (Half of a pair whose other half is the last key over and over, and alone: 4 clips of 24 frames of
    // 12 global ones, 162 positions, 8 x 160, three tiles, 51.4 and 46.6 us; 24 clips of 4 frames, 325 positions,
    // 8 x 80, one tile, 75.7 and 62.8.)
    if (odd) key_tiles(std::integral_constant<int, 1>{}, 0);
    for (int t0 = odd; t0 < tiles; t0 += KT) key_tiles(std::integral_constant<int, KT>{}, t0);

#pragma unroll
    for (int u = 0; u < QT; ++u) {
        if (16 * u >= tk.nq) break;
        bool nan = false;
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
            for (int x = 0; x < 2; ++x)
                nan = nan || __builtin_isunordered(o[u][kb][x][0], o[u][kb][x][1]) ||
                      __builtin_isunordered(o[u][kb][x][2], o[u][kb][x][3]);
        if (__any(nan) && infinity_in_v(a, tk, cx, gl)) {
            vector_task<std::conditional_t<OUT_F32, float, __bf16>>(a, tk, cx, gl, tk.q0 + 16 * u,
                                                                   tk.q0 + min(16 * u + 16, tk.nq));
            continue;
        }
        const float inv = sm[u].inverse_sum();
        // out as whole rows too: the lane's eight channels of its query go through LDS
        constexpr int OS = OUT_F32 ? 2 * RS : RS;
        wave_lds_sync();
#pragma unroll
        for (int kb = 0; kb < NKB; ++kb) {
            if constexpr (OUT_F32) {
                *(f32x4 *)(vs + l16 * OS + 128 * kb + 32 * lg) = o[u][kb][0] * inv;
                *(f32x4 *)(vs + l16 * OS + 128 * kb + 32 * lg + 16) = o[u][kb][1] * inv;
            } else {
                bf16x8 y;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    y[e] = (__bf16)(o[u][kb][0][e] * inv);
                    y[4 + e] = (__bf16)(o[u][kb][1][e] * inv);
                }
                *(bf16x8 *)(vs + l16 * OS + 64 * kb + 16 * lg) = y;
            }
        }
        wave_lds_sync();
        if (16 * u + lr >= tk.nq) continue;
        const int64_t row = (int64_t)(tk.q0 + 16 * u + lr) * FS + rowoff;
#pragma unroll
        for (int kb = 0; kb < (OUT_F32 ? 2 : 1) * NKB; ++kb) {
            const int c = (OUT_F32 ? 4 : 8) * (4 * kb + lc);  // the lane's first channel
            if (FULL || c < D)
                *(u32x4 *)((unsigned char *)a.O + (row + c) * (OUT_F32 ? 4 : 2)) =
                    *(const u32x4 *)(vs + lr * OS + 64 * kb + 16 * lc);
        }
    }
}

// ---------------------------------------------------------------- fp32

// LDS of one wavefront: the rows of a key tile (or of a query tile), padded
constexpr int krow_bytes(int NC) { return 64 * NC + 16; }

// NC = ceil(D / 16): 16-byte chunks per lane of a Q or K row, 16-channel tiles of O^T; FULL: D = 16 NC.  QT
// query tiles share every key row that is fetched.
template <int NC, bool FULL, int QT, int OPTS>
__global__ __launch_bounds__(256, 2) void tile_attn_f32_kernel(const TileArgs a)
{
    // A row of V, and of O, is NF blocks of 64 channels, then one of 32, then one of 16: lane m has W consecutive
    // channels of a block of 16 W.
    constexpr int NF = NC / 4, N2 = NC / 2 % 2, N1 = NC % 2;
    constexpr int C2 = 64 * NF, C1 = C2 + 32 * N2;  // where the last two start
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    constexpr int RS = krow_bytes(NC);
    __shared__ __attribute__((aligned(16))) unsigned char smem[4 * 16 * RS];
    __shared__ int gtab[kLdsGlobals];
    const int ginfo = my_global(a);
    const Globals gl{a, (lds_int *)gtab};
    const Task tk = task_of<QT>(a);  // (without a task: the last one's rows, up to the barrier)
    const int lane = threadIdx.x & 63, l16 = lane & 15, lg = lane >> 4;
    unsigned char *ks = smem + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * (16 * RS);
    const int D = a.D;
    const int64_t C = (int64_t)a.h * D, FS = (int64_t)a.P * C;
    const int64_t rowoff = (int64_t)tk.p * C + (int64_t)tk.g * D;
    const Context cx = context_of(a, tk);

    // Rows of Q and K are fetched four lanes to a row: lane l has chunks 4 j + l % 4 of row l / 4 (past the
    // head: nothing) ...
    const int lr = lane >> 2, lc = lane & 3;
    const bool last_ok = FULL || 16 * (NC - 1) + 4 * lc < D;
    auto load_chunks = [&](const float *p, f32x4(&r)[NC]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j + 1 < NC; ++j) r[j] = *(const f32x4 *)(p + 16 * j);
        if (last_ok) r[NC - 1] = *(const f32x4 *)(p + 16 * (NC - 1));
    };
    const int64_t laneoff = rowoff + 4 * lc;
    // ... and pass through LDS (past the head, whatever the register holds: to the row's padding; those chunks
    // stay zero): an operand is chunk 4 j + lane / 16 of row lane % 16
    const int put_at = lr * RS + 16 * lc, put_last = lr * RS + (last_ok ? 64 * (NC - 1) + 16 * lc : 64 * NC);
    auto put_rows = [&](const f32x4(&r)[NC]) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NC; ++j)
            *(f32x4 *)(ks + (FULL || j + 1 < NC ? put_at + 64 * j : put_last)) = r[j];
    };
    if constexpr (!FULL) {
        for (int i = lane; i < RS; i += 64) *(f32x4 *)(ks + 16 * i) = f32x4{};
        wave_lds_sync();
    }
    auto fragment = [&](int j) __attribute__((always_inline)) {
        return *(const f32x4 *)(ks + l16 * RS + 64 * j + 16 * lg);
    };

    const int tiles = (cx.L + 15) / 16;
    f32x4 kr[NC];
    f32x4 vf[4][NF ? NF : 1];  // [s: key 4 lg + s][block]
    f32x2 v2[4];
    float v1[4];
    const float *Kw = (const float *)a.K + cx.base * FS + laneoff;
    // (only the last block may reach past the head; channels there: any, those of the result are not stored)
    const float *Vw = (const float *)a.V + cx.base * FS + rowoff;
    auto channel = [&](int base, int w, bool last) __attribute__((always_inline)) {
        return FULL || !last || base + w * l16 < D ? base + w * l16 : 0;
    };
    const int cf = channel(0, 4, false), cl = channel(C2 - 64, 4, true);  // (of the first blocks and of the last one)
    const int c2 = channel(C2, 2, !N1), c1 = channel(C1, 1, true);
    auto load_k = [&](int t) __attribute__((always_inline)) {
        load_chunks(row_ptr(Kw, key_row(a, cx, gl, t, 16 * t + lr), a.fsb), kr);
    };
    auto load_v = [&](int t) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const uint32_t row = key_row(a, cx, gl, t, 16 * t + 4 * lg + s);
#pragma unroll
            for (int b = 0; b < NF; ++b)
                vf[s][b] = *(const f32x4 *)(row_ptr(Vw, row, a.fsb) +
                                            (FULL || N2 || N1 || b + 1 < NF ? cf + 64 * b : cl));
            if constexpr (N2) v2[s] = *(const f32x2 *)(row_ptr(Vw, row, a.fsb) + c2);
            if constexpr (N1) v1[s] = row_ptr(Vw, row, a.fsb)[c1];
        }
    };
    f32x4 q[QT][NC];
#pragma unroll
    for (int u = 0; u < QT; ++u) {
        const int aq = tk.q0 + min(16 * u + lr, tk.nq - 1);
        load_chunks(row_ptr((const float *)a.Q + laneoff, aq, a.fsb), q[u]);
    }
    // (rows that need no table are asked for before it is waited for)
    if (16 <= cx.nl) {
        load_k(0);
        load_v(0);
    }
    put_globals(a, gtab, ginfo);
    if (!tk.exists) return;
    if (16 > cx.nl) {
        load_k(0);
        load_v(0);
    }
#pragma unroll
    for (int u = 0; u < QT; ++u) {
        wave_lds_sync();
        put_rows(q[u]);
        wave_lds_sync();
#pragma unroll
        for (int j = 0; j < NC; ++j) q[u][j] = fragment(j);
    }

    f32x4 o[QT][NC];  // o[4 b + t]: channel 64 b + W m + t of row m, in block b of width W
#pragma unroll
    for (int u = 0; u < QT; ++u)
#pragma unroll
        for (int j = 0; j < NC; ++j) o[u][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    Softmax<true, OPTS> sm[QT];
    const uint64_t hide = OPTS == kUnion ? hidden_entries(a, cx, gl) : 0;

    for (int t = 0; t < tiles; ++t) {
        wave_lds_sync();
        put_rows(kr);
        wave_lds_sync();
        if (t + 1 < tiles) load_k(t + 1);  // (K's registers are free again)
        // (rows of V past the list are zeros: their weights are, and zero times an infinity is not)
        if (16 * t + 16 > cx.L) {
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const bool ok = 16 * t + 4 * lg + s < cx.L;
#pragma unroll
                for (int b = 0; b < NF; ++b) vf[s][b] = ok ? vf[s][b] : f32x4{};
                if constexpr (N2) v2[s] = ok ? v2[s] : f32x2{};
                if constexpr (N1) v1[s] = ok ? v1[s] : 0.f;
            }
        }
        // (two chains a query tile: an instruction of one covers the latency of the other's)
        f32x4 s2[QT][2] = {};
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            const f32x4 k = fragment(j);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int u = 0; u < QT; ++u)
                    s2[u][e & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(k[e], q[u][j][e], s2[u][e & 1], 0, 0, 0);
        }

#pragma unroll
        for (int u = 0; u < QT; ++u) {
            if (u > 0 && 16 * u >= tk.nq) break;
            f32x4 s[1] = {s2[u][0] + s2[u][1]};
            const float alpha = sm[u].step(a, cx, gl, hide, tk.q0 + min(16 * u + l16, tk.nq - 1), s, t, lane);
            if (__any(alpha != 1.f)) {
#pragma unroll
                for (int j = 0; j < NC; ++j) o[u][j] *= alpha;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
#pragma unroll
                for (int b = 0; b < NF; ++b)
#pragma unroll
                    for (int x = 0; x < 4; ++x)
                        o[u][4 * b + x] =
                            __builtin_amdgcn_mfma_f32_16x16x4f32(vf[e][b][x], s[0][e], o[u][4 * b + x], 0, 0, 0);
                if constexpr (N2)
#pragma unroll
                    for (int x = 0; x < 2; ++x)
                        o[u][4 * NF + x] =
                            __builtin_amdgcn_mfma_f32_16x16x4f32(v2[e][x], s[0][e], o[u][4 * NF + x], 0, 0, 0);
                if constexpr (N1)
                    o[u][NC - 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(v1[e], s[0][e], o[u][NC - 1], 0, 0, 0);
            }
        }
        if (t + 1 < tiles) load_v(t + 1);
    }

#pragma unroll
    for (int u = 0; u < QT; ++u) {
        if (16 * u >= tk.nq) break;
        const float inv = sm[u].inverse_sum();
        wave_lds_sync();
        // a block's channels W (4 lg + e) + t of query lane % 16, 4 W contiguous ones, are element e of its tile t
        auto put_block = [&](int W, int first, int channel0) __attribute__((always_inline)) {
#pragma unroll
            for (int x = 0; x < W; ++x) {
                f32x4 y;
#pragma unroll
                for (int z = 0; z < 4; ++z) y[z] = o[u][first + (4 * x + z) % W][(4 * x + z) / W] * inv;
                *(f32x4 *)(ks + l16 * RS + 4 * (channel0 + 4 * W * lg + 4 * x)) = y;
            }
        };
#pragma unroll
        for (int b = 0; b < NF; ++b) put_block(4, 4 * b, 64 * b);
        if constexpr (N2) put_block(2, 4 * NF, C2);
        if constexpr (N1) put_block(1, NC - 1, C1);
        wave_lds_sync();
        if (16 * u + lr >= tk.nq) continue;
        float *op = (float *)a.O + (int64_t)(tk.q0 + 16 * u + lr) * FS + laneoff;
#pragma unroll
        for (int j = 0; j < NC; ++j)
            if (FULL || 16 * j + 4 * lc < D) *(f32x4 *)(op + 16 * j) = *(const f32x4 *)(ks + lr * RS + 64 * j + 16 * lc);
    }
}

// Head sizes with kernels of two query tiles per wavefront; query_tiles() says when they are taken.  They share the rows
// that are fetched and cost registers; others, 6 clips of 24 frames, 1.2 x 10^7 elements, us with one and with two: bf16
// head_dim 80 26.2 and 29.3, 96 22.0 and 25.8; fp32 80 58.4 and 67.0, 96 61.4 and 63.2, 144 67.4 and 72.3, 160 spills.
constexpr bool two_query_tiles(bool f32, int blocks)
{
    return f32 ? blocks <= 4 || blocks == 7 || blocks == 8 : blocks <= 2 || blocks == 4;
}

template <int NKB, bool FULL, bool OUT_F32>
const void *bf16_fn(int qt, int opts)
{
    if constexpr (two_query_tiles(false, NKB))
        if (qt == 2) return (const void *)&tile_attn_bf16_kernel<NKB, FULL, 2, kPlain, OUT_F32>;
    switch (opts) {
    case kPlain: return (const void *)&tile_attn_bf16_kernel<NKB, FULL, 1, kPlain, OUT_F32>;
    case kBiases: return (const void *)&tile_attn_bf16_kernel<NKB, FULL, 1, kBiases, OUT_F32>;
    case kWindow: return (const void *)&tile_attn_bf16_kernel<NKB, FULL, 1, kWindow, OUT_F32>;
    case kUnion: return (const void *)&tile_attn_bf16_kernel<NKB, FULL, 1, kUnion, OUT_F32>;
    default: return (const void *)&tile_attn_bf16_kernel<NKB, FULL, 1, kAll, OUT_F32>;
    }
}
template <int NKB>
const void *bf16_fn(int D, int qt, int opts, bool out_f32)
{
    if (D == 32 * NKB) return out_f32 ? bf16_fn<NKB, true, true>(qt, opts) : bf16_fn<NKB, true, false>(qt, opts);
    return out_f32 ? bf16_fn<NKB, false, true>(qt, opts) : bf16_fn<NKB, false, false>(qt, opts);
}
template <int NC, bool FULL>
const void *f32_fn(int qt, int opts)
{
    if constexpr (two_query_tiles(true, NC))
        if (qt == 2) return (const void *)&tile_attn_f32_kernel<NC, FULL, 2, kPlain>;
    switch (opts) {
    case kPlain: return (const void *)&tile_attn_f32_kernel<NC, FULL, 1, kPlain>;
    case kBiases: return (const void *)&tile_attn_f32_kernel<NC, FULL, 1, kBiases>;
    case kWindow: return (const void *)&tile_attn_f32_kernel<NC, FULL, 1, kWindow>;
    case kUnion: return (const void *)&tile_attn_f32_kernel<NC, FULL, 1, kUnion>;
    default: return (const void *)&tile_attn_f32_kernel<NC, FULL, 1, kAll>;
    }
}
template <int NC>
const void *f32_fn(int D, int qt, int opts)
{
    return D == 16 * NC ? f32_fn<NC, true>(qt, opts) : f32_fn<NC, false>(qt, opts);
}

const void *tile_fn(const dsattn_desc &d, int qt, int opts)
{
    const bool out_f32 = d.out_dtype == DSATTN_F32;
    const int D = d.head_dim;
    if (d.io_dtype == DSATTN_BF16) switch ((D + 31) / 32) {
        case 1: return bf16_fn<1>(D, qt, opts, out_f32);
        case 2: return bf16_fn<2>(D, qt, opts, out_f32);
        case 3: return bf16_fn<3>(D, qt, opts, out_f32);
        case 4: return bf16_fn<4>(D, qt, opts, out_f32);
        case 5: return bf16_fn<5>(D, qt, opts, out_f32);
        default: return nullptr;
        }
    switch ((D + 15) / 16) {
    case 1: return f32_fn<1>(D, qt, opts);
    case 2: return f32_fn<2>(D, qt, opts);
    case 3: return f32_fn<3>(D, qt, opts);
    case 4: return f32_fn<4>(D, qt, opts);
    case 5: return f32_fn<5>(D, qt, opts);
    case 6: return f32_fn<6>(D, qt, opts);
    case 7: return f32_fn<7>(D, qt, opts);
    case 8: return f32_fn<8>(D, qt, opts);
    case 9: return f32_fn<9>(D, qt, opts);
    case 10: return f32_fn<10>(D, qt, opts);
    default: return nullptr;
    }
}

// Query tiles per wavefront.  Two are faster where there are so many wavefronts that the registers they cost, one to three
// wavefronts a SIMD, leave enough rounds.  Time with one over time with two, clips of 24 and of 32 frames (40: not whole
// blocks of 32 channels, the kernel of one tile has four wavefronts a SIMD where that of 64 has five):
//                   bf16 16, 32          40          64    104, 128  fp32 16 - 48          64    104, 112         128
//      5,000 tiles                     1.07  0.94, 1.00  0.89, 0.99                1.00, 1.04  0.88, 0.98  0.99, 1.17
//      9,000         0.89, 0.93        1.02  0.94, 0.94  0.99, 1.00    1.00, 1.05  1.03, 1.03  0.92, 1.03  1.03, 1.02
//     16,000         0.97, 1.00  1.08, 1.01  0.92, 0.93  1.09, 1.03    0.99, 1.08  1.06, 1.05  1.00, 0.96  0.98, 0.98
//     31,000         0.95, 1.03  1.08, 1.11  1.03, 1.01  1.06, 1.06    1.05, 1.12  1.05, 1.02  1.00, 0.98  0.97, 0.97
//     62,000         1.00, 1.11  1.15, 1.13  1.05, 1.04                1.08, 1.13  1.07, 1.06
//    125,000 and up  1.06, 1.12  1.18, 1.18  1.08, 1.11  1.09, 1.13    1.08, 1.19  1.09, 1.10  1.05, 1.05  1.03, 1.04
// Clips of three query tiles leave the second wavefront one: 48 frames 0.85 to 1.00, but 40 from 37,000 tiles on 1.01 to
// 1.04.  Options cost registers too: 157 us with one, 183 with two at 128 with the set union.
int query_tiles(const dsattn_desc &d, int opts)
{
    const bool f32 = d.io_dtype == DSATTN_F32;
    const int nqt = (d.clip_len + 15) / 16, blocks = f32 ? (d.head_dim + 15) / 16 : (d.head_dim + 31) / 32;
    if (opts || nqt == 1 || !two_query_tiles(f32, blocks)) return 1;
    const bool part = !f32 && blocks == 2 && d.head_dim % 32 != 0;
    if (nqt == 3 && !part) return 1;
    const int64_t tiles = (int64_t)d.n_clips * d.spatial * d.heads * nqt;
    const int64_t from = f32 ? (blocks == 7 ? 65536 : 4096)
                             : nqt == 3 ? 36864 : blocks == 1 ? 40960 : blocks == 2 && !part ? 24576 : 12288;
    return tiles >= from ? 2 : 1;
}

// What the scopes' biases take from the local and the global keys' raw scores; returns the factor of the
// scores in the exponent.
// A softmax sees only the difference of the two biases.  It is taken from the lighter scope's scores:
// added to the heavier one's, which are the ones that count, it would take their low bits (a local
// bias of -1e4 cost 1e-4 of the result, one of -1e9 all of the scores).  A heavier bias of 2^64 and
// more swallows the scores beside it in 64 bits too: every key of that scope weighs the same, as on
// the vector kernel.
float bias_shifts(const dsattn_plan_t &pl, float &lb, float &gb)
{
    const dsattn_desc &d = pl.desc;
    const bool globals = !pl.global_idx.empty();
    const bool swallows = std::fabs(globals ? std::max(d.bias_local, d.bias_global) : d.bias_local) >= 0x1p64f;
    const float sc = swallows ? 1e-30f : pl.scale * 1.4426950408889634f;
    const double diff = globals ? ((double)d.bias_global - d.bias_local) * 1.4426950408889634 / sc : 0.0;
    const double hides = 3e38 / std::max(sc, 1.f);  // (any scope; times sc it is still finite)
    lb = (float)std::max(std::min(-diff, 0.0), -hides);
    gb = (float)std::max(std::min(diff, 0.0), -hides);
    return sc;
}

// Which options the kernel of a plan is compiled for.  (bf16 rows of 32 channels under a window alone take the kernel
// for any: window of 8, 60 clips of 24 frames x 200 positions, 4, 5, 8 heads, 93.0, 116.9, 180.3 us and 94.8, 119.2,
// 188.4 in the window's; shorter clips and windows within 1.5 % either way; with a bias 196.6 and 191.8.  Rows of 8 to
// 24 channels: 172.9 and 172.0, 178.4 and 177.5, 186.5 and 186.9, with a window of 4 168.5 and 161.7, 172.5 and 166.9,
// 178.9 and 176.6.)
int opts_of(const dsattn_plan_t &pl)
{
    float lb, gb;
    bias_shifts(pl, lb, gb);
    const bool biases = lb != 0.f || gb != 0.f, windowed = pl.window >= 0;
    const size_t G = pl.global_idx.size();
    if ((pl.desc.flags & DSATTN_FLAG_DEDUP_GLOBAL) && G > 0) return windowed || G > kUnionGlobals ? kAll : kUnion;
    if (windowed) return pl.desc.io_dtype == DSATTN_BF16 && pl.desc.head_dim == 32 && !biases ? kAll : kWindow;
    return biases ? kBiases : kPlain;
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
    // a frame's 16-byte pieces are counted in 32 bits
    if ((int64_t)d.spatial * pl.C * (f32 ? 4 : 2) / 16 > 0xffffffffLL) return;
    const int qt = query_tiles(d, opts_of(pl));
    pl.tile_fn = tile_fn(d, qt, opts_of(pl));
    if (!pl.tile_fn) return;
    pl.launch.n_tasks = (int32_t)(units * ((nqt + qt - 1) / qt));
    pl.launch.block_threads = 256;
    pl.launch.lds_bytes = (f32 ? 4 * 16 * krow_bytes((d.head_dim + 15) / 16)
                               : 4 * kBf16Tiles * 16 * vrow_bytes((d.head_dim + 31) / 32)) +
                          kLdsGlobals * (int)sizeof(int32_t);
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
    a.ginfo = pl.d_global_info;
    a.N = d.n_clips;
    a.F = pl.F;
    a.wl = d.local_ctx;
    a.P = d.spatial;
    a.h = d.heads;
    a.D = d.head_dim;
    a.clip_len = d.clip_len;
    a.lk_max = pl.lk_max;
    const int per_wave = 16 * query_tiles(d, opts_of(pl));
    a.nqg = (d.clip_len + per_wave - 1) / per_wave;
    a.ctx_mode = ctx_mode ? 1 : 0;
    a.G = (int32_t)pl.global_idx.size();
    a.window = std::min(pl.window, pl.F);
    a.dedup = a.G > 0 && (d.flags & DSATTN_FLAG_DEDUP_GLOBAL) ? 1 : 0;
    a.tasks = (uint32_t)d.n_clips * d.spatial * d.heads * a.nqg;
    a.per_xcd = (a.tasks + 4 * 8 - 1) / (4 * 8);
    a.fsb = (uint32_t)((int64_t)d.spatial * pl.C * (d.io_dtype == DSATTN_F32 ? 4 : 2) / 16);
    a.sc = bias_shifts(pl, a.lb, a.gb);
    void *params[] = {&a};
    return hipLaunchKernel(pl.tile_fn, dim3(a.per_xcd * 8), dim3(256), params, 0, st);
}

}  // namespace dsattn
