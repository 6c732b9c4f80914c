// Clip-parallel group normalisation (Section 4.2, "Group normalization") for one GPU that holds
// every clip: the statistics of a channel group are those of the whole video, then
// y = (x - mean) * rstd * gamma + beta.  The paper has every device compute its clip's mean,
// average the means, then compute and average the squared deviations about the global mean: two
// rounds, because averaging per-clip deviations about per-clip means would be wrong.  The same
// global mean and variance come out of ONE pass if every part reports its mean and the sum of squared
// deviations about it, and the parts are merged with what their means differ by; that
// is what is done here (one read of X for the statistics instead of two), and between
// devices it would be one exchange instead of two.
//
// Tensors of up to 32,768 elements a group (a million with 32 groups; gn_small() has the other limits) take one
// launch of gn_small_kernel, larger ones three kernels.  These
// stream X ([F, P, C], C fastest) with 16-byte lanes; a lane's 16 bytes belong to at
// most two groups.  Reductions are deterministic: per-thread fp32 sums about a per-thread pilot,
// a fixed-order merge per workgroup into a table in the caller's workspace, and a small
// finalising kernel in fp64.
#include <hip/hip_bf16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>

#include "plan.h"

namespace dsattn {

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kGnUnroll = 4;  // rows of a bite per row phase of a workgroup

struct GnShape {
    int vec;        // elements per 16-byte lane
    int ch;         // lanes per row = C / vec
    int cg;         // channels per group
    int rpb;        // rows handled together by a workgroup (blockDim.y)
    int bpc;        // workgroups per clip the workspace has room for
    int64_t rows;   // rows of the video, F * P
    int blocks;     // workgroups of the statistics pass
    int apply_blocks;  // workgroups of the apply pass, which needs no room in the workspace
};

bool gn_shape(const dsattn_gn_desc &d, GnShape &s)
{
    s.vec = d.io_dtype == DSATTN_BF16 ? 8 : 4;
    if (d.channels % d.groups != 0 || d.channels % s.vec != 0) return false;
    s.cg = d.channels / d.groups;
    // a 16-byte lane may straddle two groups, not more
    if (s.cg < s.vec && s.vec % s.cg != 0) return false;
    if (s.cg < s.vec) return false;
    s.ch = d.channels / s.vec;
    if (s.ch > 1024) return false;
    s.rpb = std::max(1, 512 / s.ch);
    s.rows = (int64_t)d.n_clips * d.clip_len * d.spatial;
    // Room in the workspace (and bound on the workgroups): about eight per compute unit over the
    // whole tensor, at least one per clip, every one with a few rows.
    const int64_t rows_per_clip = (int64_t)d.clip_len * d.spatial;
    const int64_t want = std::max<int64_t>(1, (256 * 8) / d.n_clips);
    const int64_t max_bpc = std::max<int64_t>(1, rows_per_clip / (kGnUnroll * s.rpb));
    s.bpc = (int)std::min<int64_t>(want, max_bpc);
    // One workgroup of about eight wavefronts per compute unit in the statistics pass (256 to 1,024
    // of them and two to eight loads in flight per thread measure the same within 4 %, and fewer
    // leave the finalising kernel less to add up), twice as many in the apply pass: all are resident
    // and walk the tensor together from one end to the other, which both passes rely on.  And no
    // more than there are bites of kGnUnroll * rpb rows: every one reads at least a row.
    const int64_t bites = (s.rows + kGnUnroll * s.rpb - 1) / (kGnUnroll * s.rpb);
    s.blocks = (int)std::min<int64_t>({(int64_t)d.n_clips * s.bpc, bites, 256});
    s.apply_blocks = (int)std::min<int64_t>(bites, 512);
    return true;
}

__device__ inline void unpack(const uint4 &v, float (&x)[8], __hip_bfloat16 *)
{
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x[2 * i] = __uint_as_float(w[i] << 16);
        x[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
}
__device__ inline void unpack(const uint4 &v, float (&x)[8], float *)
{
    x[0] = __uint_as_float(v.x);
    x[1] = __uint_as_float(v.y);
    x[2] = __uint_as_float(v.z);
    x[3] = __uint_as_float(v.w);
}

// A set of elements as count, sum and sum of squares about some pilot value: sets about different
// pilots are added up in fp64 after moving them to a common one, which takes no division.  The
// pilots are elements of the same group, so the moved sums stay of the size of the spread.
struct GnSums {
    double n, s1, s2;
};
__device__ inline void gn_add(GnSums &a, double n, double s1, double s2, double shift)
{
    a.n += n;
    a.s1 += s1 + n * shift;
    a.s2 += s2 + shift * (2.0 * s1 + n * shift);
}

// What a workgroup reports of a group: mean (two floats) and sum of squared deviations about it.  (The
// count follows from the workgroup's rows.)
struct alignas(16) GnPart {
    float mean, mean_lo;
    double m2;
};
static_assert(sizeof(GnPart) == 16, "");

// Statistics pass: one read of X gives, per workgroup and group, the mean and the
// sum of squared deviations about that mean of the elements the workgroup saw.  Every thread
// accumulates sum(x - p) and sum((x - p)^2) about a pilot p of its own, the first element it reads, in fp32
// that moves to fp64 every 32 rows; one thread per group then adds up in fp64, in a fixed order, the
// threads that hold the group's channels about the pilot of the first of them.  A thread's rows come from
// the whole video, so its deviations are of the size of the group's spread, however large the mean is:
// nothing cancels that the spread does not outweigh.  Thread (x, y) = (lane of the row, row phase).  A lane's
// VEC channels lie in group g0 (the first `split` of them) and, when the lane straddles a
// boundary, in group g0 + 1.  Means travel as a pair of floats (leading part, remainder), so that
// a mean much larger than the spread loses nothing, sums of squared deviations as fp64: the sum over
// a workgroup's part is beyond fp32 long before a square of it is.  partial is [workgroup][groups] of
// GnPart.
//
// Bound by HBM reads.  All workgroups are resident and take the rows in interleaved bites, so the
// chip reads the tensor as one linear stream.  (Merging the threads with Chan's update, two fp64
// divisions per step, kept one thread per group busy for some 4 us at the end of every workgroup.)
template <typename T>
__global__ __launch_bounds__(1024) void gn_moments_kernel(const uint4 *__restrict__ X,
                                                          GnPart *__restrict__ partial, int ch,
                                                          int cg, int groups, int64_t rows_all)
{
    constexpr int VEC = sizeof(T) == 2 ? 8 : 4;
    constexpr int UNR = kGnUnroll;  // independent row loads in flight per thread
    // [4][blockDim.y][ch] doubles: sum, sum of squares for g0, then g0 + 1; then [3] floats: rows, pilots;
    // then, of more than one share, [shares][groups][3] doubles
    extern __shared__ double red[];
    const int lane = threadIdx.x, ry = threadIdx.y, ny = blockDim.y;
    const int g0 = (lane * VEC) / cg;
    const int split = min(VEC, (g0 + 1) * cg - lane * VEC);
    const uint4 *base = X + lane;
    // Per element slot of the lane: running sums of (x - pilot) and (x - pilot)^2.  The pilot of a
    // slot is an element of the slot's group in the lane's first row, so every slot of a group is taken about
    // the same value and the slots' sums add up to the group's; three vector operations per element.
    // (A thread without a first row has none at all.)
    float pv[VEC], a[VEC], q[VEC];
    const int64_t first = (int64_t)blockIdx.x * UNR * ny + ry;
    float x0[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (first < rows_all) unpack(base[first * ch], x0, (T *)nullptr);
    const float p0 = x0[0], p1 = split < VEC ? x0[VEC - 1] : x0[0];
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
        pv[i] = i < split ? p0 : p1;
        a[i] = q[i] = 0.f;
    }
    // The fp32 sums are moved to fp64 every 32 rows: with 256 workgroups a thread may have some five
    // hundred, and one fp32 sum over them rounds more than the shorter sums of eight times as many
    // workgroups do: 1 / sigma was off by 1.0e-6 at 2,304 x 160 x 1,280 bf16, by 0.7e-7 so.  (No
    // slower: 482 us a call, 486 without.)
    constexpr int kMove = 8;  // bites
    double sa[VEC] = {}, sq[VEC] = {};
    auto move = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            sa[i] += (double)a[i];
            sq[i] += (double)q[i];
            a[i] = q[i] = 0.f;
        }
    };
    int rows = 0, bites = 0;
    auto add_row = [&](const uint4 &v) __attribute__((always_inline)) {
        float x[8];
        unpack(v, x, (T *)nullptr);
        ++rows;
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            const float d = x[i] - pv[i];
            a[i] += d;
            q[i] = fmaf(d, d, q[i]);
        }
    };
    const int64_t bite = (int64_t)UNR * ny;
    for (int64_t rb = (int64_t)blockIdx.x * bite; rb < rows_all; rb += (int64_t)gridDim.x * bite) {
        const int64_t r = rb + ry;
        if (rb + bite <= rows_all) {
            uint4 v[UNR];
#pragma unroll
            for (int u = 0; u < UNR; ++u) v[u] = base[(r + (int64_t)u * ny) * ch];
#pragma unroll
            for (int u = 0; u < UNR; ++u) add_row(v[u]);
        } else {
            for (int u = 0; u < UNR; ++u)
                if (r + (int64_t)u * ny < rows_all) add_row(base[(r + (int64_t)u * ny) * ch]);
        }
        if (++bites % kMove == 0) move();
    }
    move();

    double a0 = 0.0, q0 = 0.0, a1 = 0.0, q1 = 0.0;
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
        const bool lo = i < split;
        a0 += lo ? sa[i] : 0.0;
        q0 += lo ? sq[i] : 0.0;
        a1 += lo ? 0.0 : sa[i];
        q1 += lo ? 0.0 : sq[i];
    }
    const int t = ry * ch + lane, nt = ny * ch;
    float *const redf = (float *)(red + 4 * nt);
    red[0 * nt + t] = a0;
    red[1 * nt + t] = q0;
    red[2 * nt + t] = a1;
    red[3 * nt + t] = q1;
    redf[0 * nt + t] = (float)rows;
    redf[1 * nt + t] = p0;
    redf[2 * nt + t] = p1;
    __syncthreads();
    // A few threads per group share its row phases, then one of them adds up what they have.  (One thread per
    // group from the start was a chain of LDS reads as long as phases x lanes, some 3 us at the end of every
    // workgroup: 64 x 60 x 640 bf16 18.5 -> 15.1 us a call, 296 x 696 x 320 76.0 -> 71.7.)
    // (One share, where a thread has a group to itself: no table, which many groups would have no room for.)
    const int shares = max(1, min(min(nt / groups, ny), 8));
    double *const shared_sums = red + 4 * nt + (3 * nt + 1) / 2;  // [shares][groups][3], of more than one share
    auto first_pilot = [&](int g) __attribute__((always_inline)) -> double {
        // (row phase 0 of every workgroup has read at least one row: its pilot is an element)
        const int l0 = (g * cg) / VEC;
        return l0 * VEC >= g * cg ? redf[1 * nt + l0] : redf[2 * nt + l0];
    };
    auto report = [&](int g, const GnSums &m) __attribute__((always_inline)) {
        const double mean = first_pilot(g) + m.s1 / m.n, m2 = m.s2 - m.s1 * m.s1 / m.n;
        const float hi = (float)mean;
        GnPart part;
        part.mean = hi;
        part.mean_lo = (float)(mean - (double)hi);
        part.m2 = m2 < 0.0 ? 0.0 : m2;  // (a NaN stays one)
        partial[(int64_t)blockIdx.x * groups + g] = part;
    };
    for (int gs = t; gs < groups * shares; gs += nt) {
        const int g = gs % groups, share = gs / groups;
        const int l0 = (g * cg) / VEC, l1 = ((g + 1) * cg - 1) / VEC;
        const double P = first_pilot(g);
        GnSums m = {0.0, 0.0, 0.0};
        for (int y = share; y < ny; y += shares)
            for (int l = l0; l <= l1; ++l) {
                const int e = y * ch + l, k = l * VEC >= g * cg ? 0 : 1;  // the lane's first group, or its second
                const int channels = min((l + 1) * VEC, (g + 1) * cg) - max(l * VEC, g * cg);
                const double n = (double)redf[e] * channels;
                if (n > 0.0)
                    gn_add(m, n, red[2 * k * nt + e], red[(2 * k + 1) * nt + e],
                           (double)redf[(1 + k) * nt + e] - P);
            }
        if (shares == 1) {
            report(g, m);
            continue;
        }
        double *const at = shared_sums + 3 * (int64_t)gs;
        at[0] = m.n;
        at[1] = m.s1;
        at[2] = m.s2;
    }
    if (shares == 1) return;
    __syncthreads();
    for (int g = t; g < groups; g += nt) {
        GnSums m = {0.0, 0.0, 0.0};
        for (int share = 0; share < shares; ++share) {
            const double *const at = shared_sums + 3 * ((int64_t)share * groups + g);
            m.n += at[0];
            m.s1 += at[1];
            m.s2 += at[2];
        }
        report(g, m);
    }
}

// One workgroup per group adds up the workgroups' moments in fp64, in a fixed order, about the
// first one's mean: stats[g] = mean, stats[groups + g] = 1 / sqrt(M2 / n + eps) (the biased
// variance), also to the caller's own array when there is one.
__global__ __launch_bounds__(256) void gn_finalize_kernel(const GnPart *__restrict__ partial,
                                                          float *__restrict__ stats,
                                                          float *__restrict__ out, int n_blocks,
                                                          int groups, int cg, int64_t rows_all, int bite,
                                                          float eps)
{
    __shared__ double rn[4], rm[4], rq[4];
    const int g = blockIdx.x, t = threadIdx.x;
    const GnPart f = partial[g];
    const double P = (double)f.mean + (double)f.mean_lo;
    const int64_t bites = (rows_all + bite - 1) / bite, last = (bites - 1) % n_blocks;
    GnSums m = {0.0, 0.0, 0.0};
    for (int i = t; i < n_blocks; i += 256) {
        const GnPart p = partial[(int64_t)i * groups + g];
        // workgroup i took bites i, i + n_blocks, ..; the last one of all may be cut short
        const int64_t rows = ((bites - 1 - i) / n_blocks + 1) * bite - (i == last ? bites * bite - rows_all : 0);
        gn_add(m, (double)rows * cg, 0.0, p.m2, ((double)p.mean + (double)p.mean_lo) - P);
    }
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) {
        m.n += __shfl_xor(m.n, w);
        m.s1 += __shfl_xor(m.s1, w);
        m.s2 += __shfl_xor(m.s2, w);
    }
    if (t % 64 == 0) {
        rn[t / 64] = m.n;
        rm[t / 64] = m.s1;
        rq[t / 64] = m.s2;
    }
    __syncthreads();
    if (t == 0) {
        for (int w = 1; w < 4; ++w) {
            rn[0] += rn[w];
            rm[0] += rm[w];
            rq[0] += rq[w];
        }
        const double d = rm[0] / rn[0];
        double var = rq[0] / rn[0] - d * d;
        var = var < 0.0 ? 0.0 : var;  // (a NaN stays one)
        const float mean = (float)(P + d), rstd = (float)(1.0 / sqrt(var + (double)eps));
        stats[g] = mean;
        stats[groups + g] = rstd;
        if (out) {
            out[g] = mean;
            out[groups + g] = rstd;
        }
    }
}

// Apply pass: y = (x - mean) * rstd * gamma + beta, the statistics pass's walk from the other
// end.  A thread keeps one lane of the row, so its channels' mean, factors and offset are loaded
// once and stay in registers.  (rstd * gamma as one factor, which may leave fp32's range where y does
// not, is 0.6 % faster: 483 against 486 us a call at 2,304 x 160 x 1,280 bf16.)  (Fetched anew for every 16 bytes of X, with gamma and beta that was
// 64 bytes of table reads per 16 bytes of tensor and 1,630 us at 2,304 x 160 x 1,280 bf16.)  The walk
// goes backwards because what the statistics pass read last is still in the 256 MB cache.
template <typename T, bool STREAM>
__global__ __launch_bounds__(1024) void gn_apply_kernel(const uint4 *X, uint4 *Y,
                                                        const float *__restrict__ stats,
                                                        const float *__restrict__ gamma,
                                                        const float *__restrict__ beta, int ch,
                                                        int cg, int groups, int64_t rows_all)
{
    constexpr int VEC = sizeof(T) == 2 ? 8 : 4;
    constexpr int UNR = kGnUnroll;
    const int lane = threadIdx.x, ry = threadIdx.y, ny = blockDim.y;
    const int g0 = (lane * VEC) / cg;
    const int split = min(VEC, (g0 + 1) * cg - lane * VEC);
    float mu[VEC], rs[VEC], ga[VEC], be[VEC];
#pragma unroll
    for (int k = 0; k < VEC; ++k) {
        const int c = lane * VEC + k, g = k < split ? g0 : g0 + 1;
        mu[k] = stats[g];
        rs[k] = stats[groups + g];
        ga[k] = gamma ? gamma[c] : 1.f;
        be[k] = beta ? beta[c] : 0.f;
    }
    auto load = [&](int64_t i) __attribute__((always_inline)) -> uint4 {
        if constexpr (STREAM) {
            const u32x4 x = __builtin_nontemporal_load((const u32x4 *)(X + i));
            return make_uint4(x[0], x[1], x[2], x[3]);
        }
        return X[i];
    };
    auto one = [&](int64_t i, const uint4 &v) __attribute__((always_inline)) {
        float x[8], y[8];
        unpack(v, x, (T *)nullptr);
#pragma unroll
        for (int k = 0; k < VEC; ++k) y[k] = fmaf((x[k] - mu[k]) * rs[k], ga[k], be[k]);
        uint4 o;
        if constexpr (sizeof(T) == 2) {
            uint32_t w[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const __bf16 lo = (__bf16)y[2 * k], hi = (__bf16)y[2 * k + 1];  // RNE
                w[k] = (uint32_t)__builtin_bit_cast(unsigned short, lo) |
                       ((uint32_t)__builtin_bit_cast(unsigned short, hi) << 16);
            }
            o = make_uint4(w[0], w[1], w[2], w[3]);
        } else {
            o = make_uint4(__float_as_uint(y[0]), __float_as_uint(y[1]), __float_as_uint(y[2]),
                           __float_as_uint(y[3]));
        }
        if constexpr (STREAM)
            __builtin_nontemporal_store(u32x4{o.x, o.y, o.z, o.w}, (u32x4 *)(Y + i));
        else
            Y[i] = o;
    };
    const int64_t bite = (int64_t)UNR * ny;
    const int64_t bites = (rows_all + bite - 1) / bite;
    for (int64_t b = bites - 1 - blockIdx.x; b >= 0; b -= gridDim.x) {
        const int64_t r = b * bite + ry;
        const int64_t i0 = r * ch + lane, step = (int64_t)ny * ch;
        if ((b + 1) * bite <= rows_all) {
            uint4 v[UNR];
#pragma unroll
            for (int u = 0; u < UNR; ++u) v[u] = load(i0 + u * step);
#pragma unroll
            for (int u = 0; u < UNR; ++u) one(i0 + u * step, v[u]);
        } else {
            for (int u = 0; u < UNR; ++u)
                if (r + (int64_t)u * ny < rows_all) one(i0 + u * step, load(i0 + u * step));
        }
    }
}

// Small tensors in one launch: a workgroup holds all of a group in registers, PER pairs of neighbouring
// channels a thread, and goes from mean to squared deviations to result without another read.  A group's
// rows are pieces of 2 cg or 4 cg bytes, so lines are fetched by the several groups that share them, and
// there are only as many workgroups as groups; what it saves is two launches and the gaps between them.
// A thread's sums are fp32 over 16 elements at a time about its own first element (an outlier rounds the sums of
// one thread, not of all), everything beyond that is fp64.  In place it works too: nothing is written before the
// group has been read.
constexpr int kGnSmallThreads = 1024;
constexpr int kGnSmallMaxCg = 256;
template <typename T, int PER>
__global__ __launch_bounds__(kGnSmallThreads) void gn_small_kernel(const T *X, T *Y, const float *__restrict__ gamma,
                                                                   const float *__restrict__ beta, float *out, int C,
                                                                   int cg, int groups, int rows, float eps)
{
    constexpr int NT = kGnSmallThreads, NW = NT / 64;
    typedef T pair __attribute__((ext_vector_type(2)));
    __shared__ double part[2][NW];
    __shared__ float sg[kGnSmallMaxCg], sb[kGnSmallMaxCg];
    const int g = blockIdx.x, t = threadIdx.x, lane = t & 63, wv = t >> 6;
    X += g * cg;
    Y += g * cg;
    if (t < cg) {
        sg[t] = gamma ? gamma[g * cg + t] : 1.f;
        sb[t] = beta ? beta[g * cg + t] : 0.f;
    }
    // Pairs t + i NT of the group: row and channel are counted along.
    const int hp = cg / 2, n2 = rows * hp;
    const int dr = NT / hp, dc = 2 * (NT - dr * hp);
    const int row0 = t / hp, c0 = 2 * (t - row0 * hp);
    pair x[PER];
    auto walk = [&](auto &&visit) __attribute__((always_inline)) {
        int at = row0 * C + c0, c = c0;  // elements from the group's first (a small tensor: they fit)
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            if (t + i * NT < n2) visit(i, at, c);
            const bool over = c + dc >= cg;
            c += over ? dc - cg : dc;
            at += over ? (dr + 1) * C + dc - cg : dr * C + dc;
        }
    };
    walk([&](int i, int at, int) { x[i] = *(const pair *)(X + at); });
    auto total = [&](double s, int which) __attribute__((always_inline)) -> double {
#pragma unroll
        for (int w = 32; w > 0; w >>= 1) s += __shfl_xor(s, w);
        if (lane == 0) part[which][wv] = s;
        __syncthreads();
        double sum = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) sum += part[which][w];
        return sum;
    };
    const double n = 2.0 * n2, mine = t < n2 ? 2.0 * ((n2 - 1 - t) / NT + 1) : 0.0;
    const float pilot = t < n2 ? (float)x[0][0] : 0.f;
    auto sums = [&](auto &&f) __attribute__((always_inline)) -> double {
        double s = 0.0;
#pragma unroll
        for (int i0 = 0; i0 < PER; i0 += 8) {
            float a = 0.f;
#pragma unroll
            for (int i = i0; i < std::min(PER, i0 + 8); ++i)
                if (t + i * NT < n2) a = f((float)x[i][1], f((float)x[i][0], a));
            s += (double)a;
        }
        return s;
    };
    const double s = sums([&](float v, float a) { return a + (v - pilot); });
    const double mean = total(s + mine * (double)pilot, 0) / n;
    const float mu = (float)mean;
    const double off = mean - (double)mu;
    const double q = total(sums([&](float v, float a) { return fmaf(v - mu, v - mu, a); }), 1) / n - off * off;
    const float rs = (float)(1.0 / sqrt((q < 0.0 ? 0.0 : q) + (double)eps));  // (a NaN stays one)
    if (t == 0 && out) {
        out[g] = mu;
        out[groups + g] = rs;
    }
    walk([&](int i, int at, int c) {
        *(pair *)(Y + at) = pair{(T)fmaf(((float)x[i][0] - mu) * rs, sg[c], sb[c]),
                                 (T)fmaf(((float)x[i][1] - mu) * rs, sg[c + 1], sb[c + 1])};
    });
}

// Where it is the faster one.  32 groups, us a call with three launches and with one, bf16: 16 x 30 x 960 14.7 and
// 7.8 (eight pairs a thread), 32 x 40 x 640 15.2 and 9.4, 16 x 51 x 1,280 15.2 and 10.3, 32 x 100 x 320 15.4 and
// 12.9; fp32: 14.7 and 7.7, 14.6 and 8.9, 14.2 and 9.6, but 14.1 and 15.0 (3,200 rows of short pieces).  With 32
// pairs a thread, 64 x 40 x 640 bf16, 20.6 against 15.1.
// Many groups: a piece of a row is an access of its own however short it is, and the pieces of all groups count.  bf16,
// rows x channels / groups: 1,200 x 2,560 / 320 (384,000 pieces) 20.0 and 16.8, 2,560 x 1,024 / 128 (328,000) 16.4 and
// 14.8, 4,096 x 1,024 / 128 (524,000) 17.5 and 20.1, 2,000 x 2,560 / 320 (640,000) 20.7 and 25.1, 4,096 x 8,192 /
// 1,024 (4,194,000) 49.6 and 135; fp32, eight channels a group: 896 x 3,200 / 400 (358,000) 17.4 and 12.8, 2,560 x
// 2,048 / 256 (655,000) 19.7 and 21.0; four: 256 x 4,096 / 1,024 (262,000) 16.0 and 16.0, 640 x 2,048 / 512 (328,000)
// 14.7 and 14.1, 1,200 x 1,280 / 320 (384,000) 15.8 and 16.0, 640 x 3,200 / 800 (512,000) 18.2 and 21.4.
bool gn_small(const dsattn_gn_desc &d, const GnShape &s)
{
    const int64_t most_rows = d.io_dtype == DSATTN_BF16 ? 4096 : 2560;
    const int64_t most_pieces = s.cg < 8 ? 2 << 17 : 3 << 17;
    return s.cg % 2 == 0 && s.cg <= kGnSmallMaxCg && d.groups >= 8 && s.rows <= most_rows &&
           s.rows * s.cg <= 2 * 16 * kGnSmallThreads && s.rows * d.groups <= most_pieces;
}

int gn_validate(const dsattn_gn_desc *d, GnShape &s, const char *who)
{
    if (!d) return fail(DSATTN_EINVAL, "%s: null descriptor", who);
    if (d->clip_len < 1 || d->n_clips < 1 || d->spatial < 1 || d->channels < 1 || d->groups < 1)
        return fail(DSATTN_EINVAL, "%s: sizes must be positive", who);
    if (d->io_dtype != DSATTN_F32 && d->io_dtype != DSATTN_BF16)
        return fail(DSATTN_EINVAL, "%s: unknown dtype", who);
    if (!(d->eps >= 0.f) || std::isinf(d->eps))
        return fail(DSATTN_EINVAL, "%s: eps must be finite and >= 0", who);
    if (d->channels % d->groups != 0)
        return fail(DSATTN_EINVAL, "%s: channels must split evenly into groups", who);
    if ((int64_t)d->clip_len * d->n_clips * d->spatial * d->channels > ((int64_t)1 << 40) ||
        d->n_clips > 65535)
        return fail(DSATTN_EINVAL, "%s: problem too large", who);
    if (!gn_shape(*d, s))
        return fail(DSATTN_EUNSUPPORTED,
                    "%s: need channels %% %d == 0, channels per group >= %d and channels <= %d", who,
                    d->io_dtype == DSATTN_BF16 ? 8 : 4, d->io_dtype == DSATTN_BF16 ? 8 : 4,
                    d->io_dtype == DSATTN_BF16 ? 8192 : 4096);
    return DSATTN_OK;
}

size_t gn_workspace_bytes(const dsattn_gn_desc &d, const GnShape &s)
{
    // moments [N][bpc][groups][4] + statistics [2 * groups] (mean, then 1/sqrt(var + eps))
    return (4 * (size_t)d.n_clips * s.bpc * d.groups + 2 * (size_t)d.groups) * sizeof(float);
}

// From this size on a tensor is more than the eight L2s hold together, and the apply pass streams
// past the caches: X is not needed again, and Y would push out the part of X that the statistics
// pass has left in the 256 MB cache.  Measured (plain / streaming): 2,304 x 160 x 1,280 bf16 548 / 502 us,
// 64 x 2,560 x 320 bf16 77 / 64 us, 384 x 640 x 640 fp32 368 / 320 us.
constexpr size_t kGnStreamBytes = (size_t)32 << 20;

// Enqueues the kernels; everything is validated.
hipError_t gn_enqueue(const dsattn_gn_desc &d, const GnShape &s, const void *X, const float *gamma,
                      const float *beta, void *Y, float *stats, void *workspace, hipStream_t st)
{
    if (gn_small(d, s)) {
        const bool few = s.rows * s.cg <= 2 * 8 * kGnSmallThreads;
        const dim3 grid(d.groups), block(kGnSmallThreads);
#define DSATTN_GN_SMALL(T, PER)                                                                   \
    hipLaunchKernelGGL((gn_small_kernel<T, PER>), grid, block, 0, st, (const T *)X, (T *)Y, gamma, beta, stats, \
                       d.channels, s.cg, d.groups, (int)s.rows, d.eps)
        if (d.io_dtype == DSATTN_BF16) {
            if (few)
                DSATTN_GN_SMALL(__bf16, 8);
            else
                DSATTN_GN_SMALL(__bf16, 16);
        } else {
            if (few)
                DSATTN_GN_SMALL(float, 8);
            else
                DSATTN_GN_SMALL(float, 16);
        }
#undef DSATTN_GN_SMALL
        return hipGetLastError();
    }
    float *partial = (float *)workspace;
    float *wstats = partial + 4 * (size_t)d.n_clips * s.bpc * d.groups;
    const dim3 grid(s.blocks), block(s.ch, s.rpb);
    const int nt = s.ch * s.rpb, shares = std::max(1, std::min({nt / d.groups, s.rpb, 8}));
    // (at most 45,056 bytes: more than one share takes several row phases, and then there are 512 threads at most)
    const size_t lds = (size_t)nt * 4 * sizeof(double) + (size_t)(3 * nt + 1) / 2 * 8 +
                       (shares > 1 ? (size_t)shares * d.groups * 3 * sizeof(double) : 0);

    const bool stream = (size_t)s.rows * s.ch * 16 >= kGnStreamBytes;
#define DSATTN_GN_RUN(T)                                                                          \
    do {                                                                                          \
        hipLaunchKernelGGL((gn_moments_kernel<T>), grid, block, lds, st, (const uint4 *)X,        \
                           (GnPart *)partial, s.ch, s.cg, d.groups, s.rows);                      \
        hipLaunchKernelGGL(gn_finalize_kernel, dim3(d.groups), dim3(256), 0, st,                  \
                           (const GnPart *)partial, wstats, stats, s.blocks, d.groups, s.cg,      \
                           s.rows, kGnUnroll * s.rpb, d.eps);                                     \
        auto *apply = stream ? &gn_apply_kernel<T, true> : &gn_apply_kernel<T, false>;             \
        hipLaunchKernelGGL(apply, dim3(s.apply_blocks), block, 0, st, (const uint4 *)X, (uint4 *)Y,   \
                           (const float *)wstats, gamma, beta, s.ch, s.cg, d.groups, s.rows);     \
    } while (0)
    if (d.io_dtype == DSATTN_BF16)
        DSATTN_GN_RUN(__hip_bfloat16);
    else
        DSATTN_GN_RUN(float);
#undef DSATTN_GN_RUN
    return hipGetLastError();
}

// Scratch of dsattn_groupnorm_static: the per-workgroup moments and the statistics live in a
// file-scope device array instead of a caller's workspace, so that the entry point allocates
// nothing.  Every device the library runs on holds its own copy of the array at its own address
// until the process ends.  In host code the array's name is only a handle for
// hipGetSymbolAddress; the address it returns for the current device is what the kernels get.
constexpr size_t kGnStaticBytes = (size_t)4 << 20;
constexpr int kGnMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[kGnStaticBytes];

// Device address of the array on the current device, looked up once per device.
hipError_t gn_static_scratch(void **out)
{
    static std::mutex mu;
    static void *addr[kGnMaxDevices] = {};
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kGnMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[dev] = p;
    }
    *out = addr[dev];
    return hipSuccess;
}

}  // namespace
}  // namespace dsattn

using namespace dsattn;

extern "C" {

int dsattn_groupnorm_workspace(const dsattn_gn_desc *desc, size_t *bytes)
{
    GnShape s;
    if (!bytes) return fail(DSATTN_EINVAL, "dsattn_groupnorm_workspace: null argument");
    const int rc = gn_validate(desc, s, "dsattn_groupnorm_workspace");
    if (rc != DSATTN_OK) return rc;
    *bytes = gn_workspace_bytes(*desc, s);
    return DSATTN_OK;
}

int dsattn_groupnorm(const dsattn_gn_desc *desc, const void *X, const float *gamma,
                     const float *beta, void *Y, float *stats, void *workspace,
                     size_t workspace_bytes, void *stream)
{
    GnShape s;
    const int rc = gn_validate(desc, s, "dsattn_groupnorm");
    if (rc != DSATTN_OK) return rc;
    const dsattn_gn_desc &d = *desc;
    if (!X || !Y || !workspace) return fail(DSATTN_EINVAL, "dsattn_groupnorm: null pointer");
    if (((uintptr_t)X | (uintptr_t)Y | (uintptr_t)workspace) & 15u)
        return fail(DSATTN_EINVAL, "dsattn_groupnorm: pointers must be 16-byte aligned");
    if (workspace_bytes < gn_workspace_bytes(d, s))
        return fail(DSATTN_EINVAL, "dsattn_groupnorm: workspace too small (%zu < %zu bytes)",
                    workspace_bytes, gn_workspace_bytes(d, s));
    const hipError_t e = gn_enqueue(d, s, X, gamma, beta, Y, stats, workspace, (hipStream_t)stream);
    if (e != hipSuccess) return fail(DSATTN_EHIP, "dsattn_groupnorm: %s", hipGetErrorString(e));
    return DSATTN_OK;
}

size_t dsattn_groupnorm_static_max_bytes(void) { return kGnStaticBytes; }

int dsattn_groupnorm_static(const dsattn_gn_desc *desc, const void *X, const float *gamma,
                            const float *beta, void *Y, float *stats, void *stream)
{
    GnShape s;
    const int rc = gn_validate(desc, s, "dsattn_groupnorm_static");
    if (rc != DSATTN_OK) return rc;
    const dsattn_gn_desc &d = *desc;
    if (!X || !Y) return fail(DSATTN_EINVAL, "dsattn_groupnorm_static: null pointer");
    if (((uintptr_t)X | (uintptr_t)Y) & 15u)
        return fail(DSATTN_EINVAL, "dsattn_groupnorm_static: pointers must be 16-byte aligned");
    const size_t need = gn_workspace_bytes(d, s);
    if (need > kGnStaticBytes)
        return fail(DSATTN_EUNSUPPORTED,
                    "dsattn_groupnorm_static: this shape needs %zu bytes of scratch, the static "
                    "array holds %zu; use dsattn_groupnorm with a workspace",
                    need, (size_t)kGnStaticBytes);
    void *ws = nullptr;
    hipError_t e = gn_static_scratch(&ws);
    if (e == hipSuccess)
        e = gn_enqueue(d, s, X, gamma, beta, Y, stats, ws, (hipStream_t)stream);
    if (e != hipSuccess)
        return fail(DSATTN_EHIP, "dsattn_groupnorm_static: %s", hipGetErrorString(e));
    return DSATTN_OK;
}

}  // extern "C"
