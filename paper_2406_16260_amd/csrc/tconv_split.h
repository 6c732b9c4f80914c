// fp32 projections and convolutions on the bf16 matrix instructions: an fp32 number is the sum of three
// bf16 numbers (24 bits in 8 + 8 + 8; where one is too small for that, its tile is done again in fp32), products
// of bf16 numbers are exact in fp32, and of the nine products of two numbers the six of 2^-16 and more are summed
// in fp32; the three that are left out are below 2^-25 of the largest.  Errors against 64 bits are a third of
// those of the fp32 instructions, whose sums are rounded after every fourth channel instead of every 32nd (2-norm,
// relative, 128 to 3,840 products a sum: 0.65e-7 to 3.8e-7 against 2.0e-7 to 1.1e-6).
//
// Same implicit GEMM and tiles as the other kernels (rows m = f * P + p, taps as row offsets of X, stages of 32
// channels of one tap, taps innermost, tiles numbered group, row, column).  A stage's rows come into registers
// while the stage before is multiplied out, are split there and written to LDS as three planes of 64-byte rows;
// 16-byte chunks are XOR-swizzled by row / 4 (of the 16 lanes that a read serves together two and two still share their
// banks).  Two workgroups share a compute unit: one splits while the other multiplies.
//
// What bounds it: the vector instructions of the splitting, beside the matrix instructions: both are busy for half of the
// time that the compute units are, the LDS for 39 % (a third of that with bank conflicts).  7,152 x 1,024 x 1,024
// 83 us = 181 TFLOP/s of fp32 products, 120 us on the fp32 instructions (whose peak is 157 TFLOP/s); 10,240 x 640 x 640
// three sets 146 against 205 us, one 52 against 77.  The look at the operands is 1 % of a projection and 3 to 6 % of a
// convolution of 5 taps (4,880 x 960 x 640: 217 -> 230 us).
#pragma once

namespace dsattn {
namespace {

// A workgroup of 2 x 2 wavefronts computes a (32 MB) x (32 MB) tile.
template <int MB>
__global__ __launch_bounds__(256, 2) void tconv_split_kernel(const ConvArgs a)
{
    constexpr int B = 32 * MB;             // tile edge
    constexpr int PLANE = 2 * B * 64;      // bytes of a plane: B rows of X, then B rows of W, 32 channels each
    constexpr int NLD = 2 * B * 8 / 256;   // 16-byte pieces per thread and stage
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    int *incomplete = (int *)(smem + 3 * PLANE);  // a wavefront has met an operand that is not the sum of its parts
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

    const int tile = (int)(blockIdx.x % kXcds) * a.per_xcd + (int)(blockIdx.x / kXcds);
    if (tile >= a.tiles) return;  // whole workgroup: no barrier has been reached yet
    const int tiles_grp = a.tiles_m * a.tiles_n;
    const int grp = tile / tiles_grp;
    const int rem = tile - grp * tiles_grp;
    const int mt = rem / a.tiles_n;
    const int64_t m0 = (int64_t)mt * B;
    const int n0 = (rem - mt * a.tiles_n) * B;
    const float *gbias = a.bias[grp];
    float *gY = (float *)a.Y[grp];

    const int t = threadIdx.x, lane = t & 63, l16 = lane & 15, lg = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wv >> 1, wn = wv & 1;
    const int taps = 2 * a.n + 1;

    // Thread t fetches piece t % 8 of rows t / 8 + 32 l of X, then of W.  Rows outside the video and pieces past
    // c_in read as zeros through the descriptors' range checks.
    const int lr = t >> 3, lc = t & 7;
    const int rowbytes = a.Cin * 4;
    constexpr uint32_t kOob = 0xfffffff0u;
    const int64_t rb = max((int64_t)0, m0 - (int64_t)a.n * a.P);  // first row the tile can touch
    const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
        (void *)((const float *)a.X + rb * a.Cin), 0,
        (int)min((a.M - rb) * a.Cin * 4, (int64_t)0x7fffffff), 0x00020000);
    const __amdgpu_buffer_rsrc_t wres =
        __builtin_amdgcn_make_buffer_rsrc((void *)a.W[grp], 0, (int)a.w_bytes, 0x00020000);
    const uint32_t off = (uint32_t)(lr * rowbytes + lc * 16);
    u32x4 raw[NLD];
    int su_kc = 0, su_t = 0;
    auto load_stage = [&]() __attribute__((always_inline)) {
        const bool live = su_kc * 32 + lc * 4 < a.Cin;
        const int64_t mshift = m0 + (int64_t)(su_t - a.n) * a.P;
        const uint32_t xs = off + (uint32_t)((int)(mshift - rb) * rowbytes + su_kc * kRow);
        const uint32_t ws = off + (uint32_t)((su_t * a.Cout + n0) * rowbytes + su_kc * kRow);
#pragma unroll
        for (int l = 0; l < NLD / 2; ++l) {
            raw[l] = __builtin_amdgcn_raw_buffer_load_b128(
                xres, live ? xs + (uint32_t)(32 * l * rowbytes) : kOob, 0, 0);
            raw[NLD / 2 + l] = __builtin_amdgcn_raw_buffer_load_b128(
                wres, live ? ws + (uint32_t)(32 * l * rowbytes) : kOob, 0, 0);
        }
        su_t = su_t + 1 == taps ? 0 : su_t + 1;
        su_kc += su_t == 0 ? 1 : 0;
    };
    // a piece is four channels: 8 bytes of chunk lc / 2 in every plane.  `lost`: bits of third parts that no bf16
    // number has
    uint32_t lost = 0;
    auto put_stage = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int l = 0; l < NLD; ++l) {
            const int row = lr + 32 * l;  // (W's rows follow X's)
            unsigned char *at = smem + row * 64 + (((lc >> 1) ^ ((row >> 2) & 3)) << 4) + ((lc & 1) << 3);
            f32x4 x = __builtin_bit_cast(f32x4, raw[l]);
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                bf16x4 h;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float r = x[e];  // (a bit_cast of x[e] itself would be element 0's)
                    h[e] = (__bf16)r;      // nearest even
                    if (p == 2) lost |= __builtin_bit_cast(uint32_t, r) & 0xffffu;
                }
                *(bf16x4 *)(at + p * PLANE) = h;
                const u32x2 w = __builtin_bit_cast(u32x2, h);
                x[0] -= __builtin_bit_cast(float, w[0] << 16);
                x[1] -= __builtin_bit_cast(float, w[0] & 0xffff0000u);
                x[2] -= __builtin_bit_cast(float, w[1] << 16);
                x[3] -= __builtin_bit_cast(float, w[1] & 0xffff0000u);
            }
        }
    };

    // big: products of the leading parts; small: the five others
    f32x4 big[MB][MB], small[MB][MB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j) big[i][j] = small[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // fragment of a plane: row lane % 16 of a 16-row block, chunk lane / 16
    const int sw = (lg ^ ((l16 >> 2) & 3)) << 4;  // (blocks start at multiples of 16 rows)
    const unsigned char *fa = smem + (wm * 16 * MB + l16) * 64 + sw;
    const unsigned char *fb = smem + (B + wn * 16 * MB + l16) * 64 + sw;

    // Of wavefronts that share a SIMD the one that splits goes first: until it is done its workgroup multiplies
    // nothing, while matrix instructions that wait a few cycles cost only those.  In a single round (two workgroups
    // of 128 x 128 on a compute unit, four of 64 x 64) and where the last one is more than half full; else the
    // workgroups do better drawn apart, so that the first to end make room.  us, without and with: 10,240 x 640 x 640 (400 tiles of 128 x 128)
    // 54.6 and 51.6, 3,328 x 1,280 x 1,280, three sets (780) 198 and 184, 2,560 x 1,280 x 1,280 (800 of 64 x 64)
    // 71.2 and 62.4; but 5,120 x 640 x 640, three sets (600 of 128 x 128) 87.3 and 90.1, 10,240 rows of them (1,200)
    // 138 and 145, 3,360 x 1,280 x 1,280 (1,060 of 64 x 64) 2 % of a layer slower.
    constexpr int kRound = MB == 4 ? 512 : 1024;
    const bool first = a.tiles <= kRound || (a.tiles - 1) % kRound >= kRound / 2;

    load_stage();
    for (int ks = 0; ks < a.KS; ++ks) {
        if (first) __builtin_amdgcn_s_setprio(1);
        put_stage();
        __builtin_amdgcn_s_setprio(0);
        if (ks + 1 == a.KS) {  // (read behind the loop's last barrier)
            const bool any = __any(lost != 0);
            if (lane == 0) incomplete[wv] = any;
        }
        __syncthreads();
        if (ks + 1 < a.KS) load_stage();
        bf16x8 x[3][MB];
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int i = 0; i < MB; ++i) x[p][i] = *(const bf16x8 *)(fa + p * PLANE + i * 1024);
#pragma unroll
        for (int j = 0; j < MB; ++j) {
            bf16x8 w[3];
#pragma unroll
            for (int p = 0; p < 3; ++p) w[p] = *(const bf16x8 *)(fb + p * PLANE + j * 1024);
            // (the smallest first)
            constexpr int kProducts[5][2] = {{0, 2}, {2, 0}, {1, 1}, {0, 1}, {1, 0}};
#pragma unroll
            for (int q = 0; q < 5; ++q)
#pragma unroll
                for (int i = 0; i < MB; ++i)
                    small[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        w[kProducts[q][0]], x[kProducts[q][1]][i], small[i][j], 0, 0, 0);
#pragma unroll
            for (int i = 0; i < MB; ++i)
                big[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[0], x[0][i], big[i][j], 0, 0, 0);
        }
        __syncthreads();
    }

    // Lane l holds channels 4 (l / 16) + e of row l % 16 of every 16 x 16 block.
    const int64_t mrow0 = m0 + wm * 16 * MB;
    const int cbase = n0 + wn * 16 * MB;
    bool again = (incomplete[0] | incomplete[1] | incomplete[2] | incomplete[3]) != 0;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < MB; ++j) {
            big[i][j] += small[i][j];
#pragma unroll
            for (int e = 0; e < 4; ++e) again = again || !(__builtin_fabsf(big[i][j][e]) < INFINITY);
        }
    // Operands that are not the sum of their parts (the smallest part of a number below 2^-110 may be below bf16's
    // last bit, 2^-133) and results that are not finite (the parts of an infinity, of a NaN, or of a number whose
    // leading part rounds to an infinity): done again on the fp32 instructions, operands from memory as the
    // instructions take them: lane l has row l % 16, channels 4 (l / 16) .. of every 16, one of them an instruction.
    // (10,240 x 640 x 640, 52.6 us: 102 with a NaN in X, a wavefront's part of one row of tiles, 157 with one in every
    // row; one thread an output, as on the vector kernel, 3,640 and 9,630.  On the fp32 kernel 77.)
    if (__any(again)) {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < MB; ++j) big[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int tap = 0; tap < taps; ++tap) {
            const int64_t ms = mrow0 + l16 + (int64_t)(tap - a.n) * a.P;  // X's row for the lane's first one
            const uint32_t xs = (uint32_t)((int)(ms - rb) * rowbytes + 16 * lg);
            const uint32_t ws = (uint32_t)((tap * a.Cout + cbase + l16) * rowbytes + 16 * lg);
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int j = 0; j < MB; ++j) small[i][j] = big[i][j];
            for (int c = 0; c < a.Cin; c += 16) {
                const bool live = c + 4 * lg < a.Cin;
                f32x4 xf[MB], wf[MB];
#pragma unroll
                for (int i = 0; i < MB; ++i) {
                    const uint32_t at = (uint32_t)(16 * i * rowbytes + 4 * c);
                    xf[i] = __builtin_bit_cast(
                        f32x4, __builtin_amdgcn_raw_buffer_load_b128(xres, live ? xs + at : kOob, 0, 0));
                    wf[i] = __builtin_bit_cast(
                        f32x4, __builtin_amdgcn_raw_buffer_load_b128(wres, live ? ws + at : kOob, 0, 0));
                }
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int j = 0; j < MB; ++j)
#pragma unroll
                        for (int i = 0; i < MB; ++i)
                            big[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(wf[j][e], xf[i][e], big[i][j], 0, 0, 0);
            }
            // (a frame outside the video adds nothing, not even its zeros times an infinite weight)
#pragma unroll
            for (int i = 0; i < MB; ++i)
                if (ms + 16 * i < 0 || ms + 16 * i >= a.M)
#pragma unroll
                    for (int j = 0; j < MB; ++j) big[i][j] = small[i][j];
        }
    }
    f32x4 bias[MB] = {};
    if (gbias) {
#pragma unroll
        for (int j = 0; j < MB; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) bias[j][e] = gbias[min(cbase + 16 * j + 4 * lg + e, a.Cout - 1)];
    }
    if ((a.Cout & 3) == 0) {
        // through the wavefront's quarter of the LDS, 16 rows at a time, and out as full rows
        constexpr int SR = 64 * MB + 16, CPR = 4 * MB;
        static_assert(4 * 16 * SR <= 3 * PLANE, "the staging area fits");
        unsigned char *stg = smem + wv * (16 * SR);
#pragma unroll
        for (int i = 0; i < MB; ++i) {
#pragma unroll
            for (int j = 0; j < MB; ++j)
                *(f32x4 *)(stg + l16 * SR + 64 * j + 16 * lg) = big[i][j] + bias[j];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int it = 0; it < 16 * CPR / 64; ++it) {
                const int q = lane + 64 * it, row = q / CPR, pc = q - row * CPR;
                const int64_t m = mrow0 + 16 * i + row;
                if (m < a.M && cbase + 4 * pc < a.Cout)
                    *(f32x4 *)(gY + m * a.Cout + cbase + 4 * pc) = *(const f32x4 *)(stg + row * SR + 16 * pc);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < MB; ++j)
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            const int64_t m = mrow0 + 16 * i + l16;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int co = cbase + 16 * j + 4 * lg + e;
                if (m < a.M && co < a.Cout) gY[m * a.Cout + co] = big[i][j][e] + bias[j][e];
            }
        }
}

}  // namespace
}  // namespace dsattn
