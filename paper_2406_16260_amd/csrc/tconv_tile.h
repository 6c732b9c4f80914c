// One-tile-per-workgroup siblings of the persistent convolution kernel: the same implicit GEMM (rows
// m = f * P + p, taps as row offsets of X, 128-byte LDS rows filled straight from global memory,
// XOR-swizzled 16-byte chunks) with smaller tiles, for
//   * bf16 problems whose 256 x 320 tiles would leave compute units idle, and
//   * fp32 tensors, on v_mfma_f32_16x16x4_f32: fp32 products and fp32 sums, nothing is rounded to
//     16 bits.
// A stage is 128 bytes of every row (64 bf16 or 32 fp32 channels of one tap, taps innermost).
//
// tconv_tile_kernel: two LDS slots, so that two to five workgroups share a compute unit and one's
// loads and barriers are hidden behind the others' multiplies.  A 16-byte fragment of lane l is row
// l % 16, chunk 4 kk + l / 16 of the stage: one operand of v_mfma_f32_16x16x32_bf16, or element s of
// it the operand of the s-th of four v_mfma_f32_16x16x4_f32 (which channels an instruction
// contracts is free as long as both operands agree).
// tconv_pipe_kernel: one workgroup per compute unit, software-pipelined, for problems of one round; with
// 128 x 64 tiles and six slots for those of few tiles and many stages, where the latency of weights from
// beyond the L2 is what a stage takes (6,400 x 1,280 x 320, 3 taps: 31.0 us with two slots of 64 x 64, 23.3).
//
// What bounds them.  fp32: the fp32 matrix rate (157 TFLOP/s; 40,000 x 1,280 x 1,280 reaches 131, 10,240 x
// 640 x 640 takes 77 us where one thread per output took 16,370 us).  Four slots measured the same
// as two, 128 x 160 tiles up to 1.5 % faster on large problems and 40 % slower on small ones.
// Small bf16: the stages of a tile are dependent (0.5 to 0.9 us each, 20 of them at 1,280 channels), and a single
// round starts and drains once: of the time that the compute units are busy the matrix cores are 33 % (pipelined 128 x
// 128) and 45 % (128 x 160, three sets), the LDS 19 and 23 %.  (The path from L2 into LDS alone does 33 TB/s.)
#pragma once

namespace dsattn {
namespace {

// s_waitcnt of at most n outstanding vector memory operations, and all LDS operations done
__host__ __device__ constexpr int waitcnt_vm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4); }

// the same, with LDS operations left alone
__host__ __device__ constexpr int waitcnt_vm_only(int n) { return waitcnt_vm(n) | (15 << 8); }

// A workgroup of WVM x WVN wavefronts computes a (16 MB WVM) x (16 NB WVN) tile.  HALO: of more taps
// than one, see the multiplies.
template <typename T, int MB, int NB, int WVM, int WVN, bool OUT_F32, bool HALO = false>
__global__ __launch_bounds__(64 * WVM * WVN, 2) void tconv_tile_kernel(const ConvArgs a)
{
    constexpr int S = 2;  // slots
    constexpr int NW = WVM * WVN;
    constexpr int BM = 16 * MB * WVM, BN = 16 * NB * WVN;
    constexpr int GA = BM / 8 / NW, GB = BN / 8 / NW;  // 8-row groups (one load instruction) per wavefront
    static_assert(GA * 8 * NW == BM && GB * 8 * NW == BN, "the wavefronts share the loads evenly");
    constexpr int NL = GA + GB;
    constexpr int ABYTES = BM * kRow, BUF = (BM + BN) * kRow;
    constexpr int kDepth = kRow / (int)sizeof(T);  // channels of a stage
    constexpr int kChunk = 16 / (int)sizeof(T);    // channels of a 16-byte chunk
    constexpr bool kF32 = sizeof(T) == 4;
    using Frag = std::conditional_t<kF32, f32x4, bf16x8>;  // a lane's 16 bytes of an operand row
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

    // workgroup -> tile: XCD x (= blockIdx % 8) owns a contiguous run of tiles
    const int tile = (int)(blockIdx.x % kXcds) * a.per_xcd + (int)(blockIdx.x / kXcds);
    if (tile >= a.tiles) return;  // whole workgroup: no barrier has been reached yet
    const int tiles_grp = a.tiles_m * a.tiles_n;
    const int grp = tile / tiles_grp;
    const int rem = tile - grp * tiles_grp;
    const int mt = rem / a.tiles_n;
    const int64_t m0 = (int64_t)mt * BM;
    const int n0 = (rem - mt * a.tiles_n) * BN;
    const float *gbias = a.bias[grp];
    void *gY = a.Y[grp];

    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wv / WVN, wn = wv - wm * WVN;

    // the bias of this lane's channels, asked for ahead of the stages
    const int cbase = n0 + wn * 16 * NB;
    // (past c_out: the last one, for channels that are not stored)
    f32x4 bias[NB] = {};
    if (gbias) {
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                bias[j][e] = gbias[min(cbase + 16 * j + 4 * (lane >> 4) + e, a.Cout - 1)];
    }

    // Global -> LDS: lane l fetches chunk (l % 8) ^ (l / 8) of row l / 8 of an 8-row group.  Rows
    // outside the video and chunks past c_in read as zeros through the descriptor's range check.
    const int lr = lane >> 3;
    const int lc = (lane & 7) ^ lr;
    const int rowbytes = a.Cin * (int)sizeof(T);
    constexpr uint32_t kOob = 0xfffffff0u;
    const int64_t rb = max((int64_t)0, m0 - (int64_t)a.n * a.P);  // first row the tile can touch
    const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
        (void *)((const T *)a.X + rb * a.Cin), 0,
        (int)min((a.M - rb) * a.Cin * (int64_t)sizeof(T), (int64_t)0x7fffffff), 0x00020000);
    const __amdgpu_buffer_rsrc_t wres =
        __builtin_amdgcn_make_buffer_rsrc((void *)a.W[grp], 0, (int)a.w_bytes, 0x00020000);
    const uint32_t xoff = (uint32_t)((wv * (8 * GA) + lr) * rowbytes + lc * 16);
    const uint32_t woff = (uint32_t)((wv * (8 * GB) + lr) * rowbytes + lc * 16);
    const int taps = 2 * a.n + 1, blocks = HALO ? (a.Cin + kDepth - 1) / kDepth : 0;
    // a tile with rows that have no frame at some tap takes the taps outermost
    const int64_t reach = (int64_t)a.n * a.P;
    const bool halo = HALO && (m0 < reach || m0 + BM + reach > a.M);
    int su_kc = 0, su_t = 0, su_slot = 0;
    auto issue_stage = [&](bool exists) __attribute__((always_inline)) {
        const bool live = exists && su_kc * kDepth + lc * kChunk < a.Cin;
        const int64_t mshift = m0 + (int64_t)(su_t - a.n) * a.P;
        const uint32_t xs = xoff + (uint32_t)((int)(mshift - rb) * rowbytes + su_kc * kRow);
        const uint32_t ws = woff + (uint32_t)((su_t * a.Cout + n0) * rowbytes + su_kc * kRow);
        unsigned char *as = smem + su_slot * BUF + wv * (GA * 1024);
        unsigned char *bs = smem + su_slot * BUF + ABYTES + wv * (GB * 1024);
#pragma unroll
        for (int l = 0; l < GA; ++l)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                xres, (__attribute__((address_space(3))) void *)(as + l * 1024), 16,
                live ? xs + (uint32_t)(8 * l * rowbytes) : kOob, 0, 0, 0);
#pragma unroll
        for (int l = 0; l < GB; ++l)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                wres, (__attribute__((address_space(3))) void *)(bs + l * 1024), 16,
                live ? ws + (uint32_t)(8 * l * rowbytes) : kOob, 0, 0, 0);
        su_slot = su_slot + 1 == S ? 0 : su_slot + 1;
        // (selected as values: as branches the compiler kept the two counters in scratch memory)
        const int kc = su_kc + 1, t = su_t + 1;
        su_kc = halo ? (kc == blocks ? 0 : kc) : (t == taps ? kc : su_kc);
        su_t = halo ? (kc == blocks ? t : su_t) : (t == taps ? 0 : t);
    };

    f32x4 acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    int koff[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) koff[kk] = (((4 * kk) | (lane >> 4)) ^ (lane & 7)) * 16;
    const int abase = (wm * 16 * MB + (lane & 15)) * kRow;
    const int bbase = ABYTES + (wn * 16 * NB + (lane & 15)) * kRow;

#pragma unroll
    for (int s = 0; s < S - 1; ++s) issue_stage(s < a.KS);
    int slot = 0;
    auto stages = [&](int from, int to) __attribute__((always_inline)) {
        for (int ks = from; ks < to; ++ks) {
            // This wavefront's loads of stage ks have landed and its reads of stage ks - 1 are done;
            // behind the barrier everybody's are, and the slot of stage ks - 1 is free.
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(waitcnt_vm((S - 2) * NL));
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            issue_stage(ks + S - 1 < a.KS);  // (past the end: out-of-range loads, the same count)
            const unsigned char *buf = smem + slot * BUF;
            slot = slot + 1 == S ? 0 : slot + 1;
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                Frag af[MB], bf[NB];
#pragma unroll
                for (int i = 0; i < MB; ++i) af[i] = *(const Frag *)(buf + abase + i * (16 * kRow) + koff[kk]);
#pragma unroll
                for (int j = 0; j < NB; ++j) bf[j] = *(const Frag *)(buf + bbase + j * (16 * kRow) + koff[kk]);
                if constexpr (kF32) {
#pragma unroll
                    for (int s = 0; s < 4; ++s)
#pragma unroll
                        for (int j = 0; j < NB; ++j)
#pragma unroll
                            for (int i = 0; i < MB; ++i)
                                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                                    bf[j][s], af[i][s],
                                    acc[i][j], 0, 0, 0);
                } else {
#pragma unroll
                    for (int j = 0; j < NB; ++j)
#pragma unroll
                        for (int i = 0; i < MB; ++i)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                bf[j], af[i], acc[i][j],
                                0, 0, 0);
                }
            }
        }
    };
    // HALO: a tap's frames outside the video add nothing, not even zero times an infinite weight: in
    // the tiles that have such rows a tap's channels are contracted together, and those rows then
    // get back the sums that they had before it.  (Free: convolutions of 32 to 384 frames are 0.5 to
    // 2 % faster than without it; kept and given back per stage, taps innermost, it was 4 to 16 %.)
    if (halo) {
        for (int t = 0; t < taps; ++t) {
            f32x4 kept[MB][NB];
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
                for (int j = 0; j < NB; ++j) kept[i][j] = acc[i][j];
            stages(t * blocks, (t + 1) * blocks);
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                const int64_t row =
                    m0 + (int64_t)(t - a.n) * a.P + wm * 16 * MB + 16 * i + (lane & 15);
                const bool outside = row < 0 || row >= a.M;
#pragma unroll
                for (int j = 0; j < NB; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        acc[i][j][e] = outside ? kept[i][j][e] : acc[i][j][e];
            }
        }
    } else {
        stages(0, a.KS);
    }

    // ---- epilogue: lane l holds channels 4 (l / 16) + e of row l % 16 of every 16 x 16 block
    const int64_t mrow0 = m0 + wm * 16 * MB;
    // every wavefront's loads have landed and its reads of the ring are done; the ring becomes the
    // staging area
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    constexpr int ESO = OUT_F32 ? 4 : 2;
    if ((a.Cout * ESO & 15) == 0) {
        // rows of whole 16-byte pieces: through the wavefront's own part of the ring, MP blocks of 16
        // rows at a time, and out as full rows (32 NB or 64 NB contiguous bytes)
        constexpr int SR = 16 * NB * ESO + 16;      // padded: the rows' pieces spread over the banks
        constexpr int CPR = NB * ESO;               // 16-byte pieces per row
        constexpr int MP = NW * MB * 16 * SR <= S * BUF ? MB : MB / 2;
        static_assert(MB % MP == 0 && NW * MP * 16 * SR <= S * BUF, "the staging area fits in the ring");
        unsigned char *stg = smem + wv * (MP * 16 * SR);
#pragma unroll
        for (int ip = 0; ip < MB; ip += MP) {
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const int cl = 16 * j + 4 * (lane >> 4);
#pragma unroll
                for (int i = 0; i < MP; ++i) {
                    const f32x4 y = acc[ip + i][j] + bias[j];
                    unsigned char *at = stg + (16 * i + (lane & 15)) * SR + cl * ESO;
                    if constexpr (OUT_F32) {
                        *(f32x4 *)at = y;
                    } else {
                        bf16x4 yb;
#pragma unroll
                        for (int e = 0; e < 4; ++e) yb[e] = (__bf16)y[e];
                        *(bf16x4 *)at = yb;
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            constexpr int kPieces = 16 * MP * CPR;
#pragma unroll
            for (int it = 0; it < (kPieces + 63) / 64; ++it) {
                const int q = lane + 64 * it;
                const int row = q / CPR, pc = q - row * CPR;
                const int64_t m = mrow0 + 16 * ip + row;
                if (q < kPieces && m < a.M && cbase * ESO + pc * 16 < a.Cout * ESO)
                    *(uint4 *)((unsigned char *)gY + (m * a.Cout + cbase) * ESO + pc * 16) =
                        *(const uint4 *)(stg + row * SR + pc * 16);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int cl = 16 * j + 4 * (lane >> 4);
        const int co = cbase + cl;
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            const int64_t m = mrow0 + 16 * i + (lane & 15);
            if (m >= a.M) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (co + e < a.Cout) {
                    const float y = acc[i][j][e] + bias[j][e];
                    if constexpr (OUT_F32)
                        ((float *)gY)[m * a.Cout + co + e] = y;
                    else
                        ((__bf16 *)gY)[m * a.Cout + co + e] = (__bf16)y;
                }
        }
    }
}

// The bf16 tile kernel: 32 x 32 accumulators of v_mfma_f32_32x32x16_bf16 (one wavefront per SIMD can
// issue these back to back, which it cannot do with 16x16x32), (32 MB) x (32 NB) per wavefront.
// A wavefront's instruction stream is software-pipelined across the stage barrier: the fragments of
// the next 16 channels are read from LDS, and the loads of the stage S - 1 ahead are issued, between
// the multiplies of the current 16.  For that a stage has to be in LDS one barrier before its first
// multiply: S = 4 slots hold the stage in use, the next one, and two on their way.
template <int MB, int NB, int WVM, int WVN, int S, bool OUT_F32>
__global__ __launch_bounds__(64 * WVM * WVN, 1) void tconv_pipe_kernel(const ConvArgs a)
{
    constexpr int NW = WVM * WVN;
    constexpr int BM = 32 * MB * WVM, BN = 32 * NB * WVN;
    constexpr int GA = BM / 8 / NW, GB = BN / 8 / NW;
    static_assert(GA * 8 * NW == BM && GB * 8 * NW == BN, "the wavefronts share the loads evenly");
    static_assert(GA % 2 == 0 && GB % 2 == 0, "a load's group is even or odd for all wavefronts");
    constexpr int NL = GA + GB;
    constexpr int ABYTES = BM * kRow, BUF = (BM + BN) * kRow;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

    const int tile = (int)(blockIdx.x % kXcds) * a.per_xcd + (int)(blockIdx.x / kXcds);
    if (tile >= a.tiles) return;
    const int tiles_grp = a.tiles_m * a.tiles_n;
    const int grp = tile / tiles_grp;
    const int rem = tile - grp * tiles_grp;
    const int mt = rem / a.tiles_n;
    const int64_t m0 = (int64_t)mt * BM;
    const int n0 = (rem - mt * a.tiles_n) * BN;
    const float *gbias = a.bias[grp];
    void *gY = a.Y[grp];

    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wv / WVN, wn = wv - wm * WVN;
    const int cbase = n0 + wn * 32 * NB;

    // the bias of this lane's channels, asked for ahead of the stages
    f32x4 bias[NB][4] = {};
    if (gbias) {
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    bias[j][q][e] = gbias[min(cbase + 32 * j + 8 * q + 4 * (lane >> 5) + e, a.Cout - 1)];
    }

    // Chunks are swizzled by row / 2 here: the 16 lanes that a 16-byte LDS read serves together are rows 0 - 3,
    // 12 - 15, 20 - 23 and 24 - 27 of a fragment of 32 rows (or the other 16), and rows alternate between the two
    // halves of the banks, so row / 2 % 8 is what tells those of one half apart.  (By row % 8 every read was a
    // two-way conflict.  2,560 x 1,280 x 1,280 on 128 x 128 tiles: LDS 37 % busy, half of that with conflicts, and 19 % with
    // 6 % of it so; 13.9 us either way: a single round's latencies, not the LDS, are what it waits for.)
    const int lr = lane >> 3;
    // the chunk a lane fetches of a row of an even 8-row group; of an odd one it is the other half's
    const int lc = (lane & 7) ^ (lr >> 1);
    const int rowbytes = a.Cin * 2;
    constexpr uint32_t kOob = 0xfffffff0u;
    const int64_t rb = max((int64_t)0, m0 - (int64_t)a.n * a.P);
    const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
        (void *)((const __bf16 *)a.X + rb * a.Cin), 0,
        (int)min((a.M - rb) * a.Cin * 2, (int64_t)0x7fffffff), 0x00020000);
    const __amdgpu_buffer_rsrc_t wres =
        __builtin_amdgcn_make_buffer_rsrc((void *)a.W[grp], 0, (int)a.w_bytes, 0x00020000);
    int xoff[GA], woff[GB];  // byte offset of this lane's row and chunk within the tile's rows
#pragma unroll
    for (int l = 0; l < GA; ++l) {
        xoff[l] = (wv * (8 * GA) + lr + 8 * l) * rowbytes + (lc ^ (l & 1) << 2) * 16;
        asm volatile("" : "+v"(xoff[l]));
    }
#pragma unroll
    for (int l = 0; l < GB; ++l) {
        woff[l] = (wv * (8 * GB) + lr + 8 * l) * rowbytes + (lc ^ (l & 1) << 2) * 16;
        asm volatile("" : "+v"(woff[l]));
    }
    const int taps = 2 * a.n + 1;
    int su_kc = 0, su_t = 0, su_slot = 0, su_ks = 0;
    bool ld_live[2] = {false, false};  // of even and odd groups
    uint32_t ld_xs = 0, ld_ws = 0;
    unsigned char *ld_as = smem, *ld_bs = smem;
    auto stage_setup = [&]() __attribute__((always_inline)) {
        ld_live[0] = su_ks < a.KS && su_kc * kBK + lc * 8 < a.Cin;
        ld_live[1] = su_ks < a.KS && su_kc * kBK + (lc ^ 4) * 8 < a.Cin;
        const int64_t mshift = m0 + (int64_t)(su_t - a.n) * a.P;
        ld_xs = (uint32_t)((int)(mshift - rb) * rowbytes + su_kc * kRow);
        ld_ws = (uint32_t)((su_t * a.Cout + n0) * rowbytes + su_kc * kRow);
        ld_as = smem + su_slot * BUF + wv * (GA * 1024);
        ld_bs = smem + su_slot * BUF + ABYTES + wv * (GB * 1024);
        su_slot = su_slot + 1 == S ? 0 : su_slot + 1;
        ++su_ks;
        if (++su_t == taps) {
            su_t = 0;
            ++su_kc;
        }
    };
    auto issue_one = [&](int l) __attribute__((always_inline)) {
        if (l < GA)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                xres, (__attribute__((address_space(3))) void *)(ld_as + l * 1024), 16,
                ld_live[l & 1] ? (uint32_t)xoff[l] + ld_xs : kOob, 0, 0, 0);
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                wres, (__attribute__((address_space(3))) void *)(ld_bs + (l - GA) * 1024), 16,
                ld_live[(l - GA) & 1] ? (uint32_t)woff[l - GA] + ld_ws : kOob, 0, 0, 0);
    };

    f32x16 acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    // fragment of 16 channels kq: lane l is row l % 32, chunk 2 kq + l / 32
    int koff[4];
#pragma unroll
    for (int kq = 0; kq < 4; ++kq) koff[kq] = (((2 * kq) | (lane >> 5)) ^ (lane >> 1 & 7)) * 16;
    const int abase = (wm * 32 * MB + (lane & 31)) * kRow;
    const int bbase = ABYTES + (wn * 32 * NB + (lane & 31)) * kRow;
    constexpr int NF = MB + NB;
    bf16x8 fr[2][NF];
    auto read_one = [&](int set, const unsigned char *base, int kq, int f) __attribute__((always_inline)) {
        fr[set][f] = f < MB ? *(const bf16x8 *)(base + abase + f * (32 * kRow) + koff[kq])
                            : *(const bf16x8 *)(base + bbase + (f - MB) * (32 * kRow) + koff[kq]);
    };

    // start: stages 0 .. S - 2 on their way, stage 0 landed, its first fragments read
#pragma unroll
    for (int s = 0; s < S - 1; ++s) {
        stage_setup();
#pragma unroll
        for (int l = 0; l < NL; ++l) issue_one(l);
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(waitcnt_vm((S - 2) * NL));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int f = 0; f < NF; ++f) read_one(0, smem, 0, f);

    constexpr int NM = MB * NB;  // multiplies of 16 channels
    int slot = 0;
    for (int ks = 0; ks < a.KS; ++ks) {
        const unsigned char *buf = smem + slot * BUF;
        slot = slot + 1 == S ? 0 : slot + 1;
        const unsigned char *nbuf = smem + slot * BUF;
        stage_setup();
        // This wavefront's loads of stage ks + 1 have landed; behind the barrier everybody's have,
        // and every wavefront is through with stage ks - 1, whose slot the loads below fill.
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(waitcnt_vm_only((S - 3) * NL));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int kq = 0; kq < 4; ++kq) {
            const int set = kq & 1;
#pragma unroll
            for (int m = 0; m < NM; ++m) {
                const int g = kq * NM + m;  // multiplies since the barrier
#pragma unroll
                for (int l = 0; l < NL; ++l)
                    if ((l * (4 * NM)) / NL == g) {
                        issue_one(l);
                        __builtin_amdgcn_sched_barrier(0);
                    }
#pragma unroll
                for (int f = 0; f < NF; ++f)
                    if ((f * NM) / NF == m) {
                        read_one(set ^ 1, kq < 3 ? buf : nbuf, (kq + 1) & 3, f);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                const int j = m / MB, i = m - j * MB;
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[set][MB + j], fr[set][i], acc[i][j],
                                                                   0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

    // ---- epilogue: element e of lane l is channel 8 (e / 4) + 4 (l / 32) + e % 4 and row l % 32 of
    // its 32 x 32 block
    const int64_t mrow0 = m0 + wm * 32 * MB;
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    constexpr int ESO = OUT_F32 ? 4 : 2;
    if ((a.Cout * ESO & 15) == 0) {
        constexpr int SR = 32 * NB * ESO + 16;
        constexpr int CPR = 2 * NB * ESO;  // 16-byte pieces per row
        constexpr int MP = NW * MB * 32 * SR <= S * BUF ? MB : 1;
        static_assert(NW * MP * 32 * SR <= S * BUF, "the staging area fits in the ring");
        unsigned char *stg = smem + wv * (MP * 32 * SR);
#pragma unroll
        for (int ip = 0; ip < MB; ip += MP) {
#pragma unroll
            for (int j = 0; j < NB; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
#pragma unroll
                    for (int i = 0; i < MP; ++i) {
                        unsigned char *at = stg + (32 * i + (lane & 31)) * SR + (32 * j + 8 * q + 4 * (lane >> 5)) * ESO;
                        if constexpr (OUT_F32) {
                            f32x4 y;
#pragma unroll
                            for (int e = 0; e < 4; ++e) y[e] = acc[ip + i][j][4 * q + e] + bias[j][q][e];
                            *(f32x4 *)at = y;
                        } else {
                            bf16x4 y;
#pragma unroll
                            for (int e = 0; e < 4; ++e) y[e] = (__bf16)(acc[ip + i][j][4 * q + e] + bias[j][q][e]);
                            *(bf16x4 *)at = y;
                        }
                    }
                }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            constexpr int kPieces = 32 * MP * CPR;
#pragma unroll
            for (int it = 0; it < (kPieces + 63) / 64; ++it) {
                const int q = lane + 64 * it;
                const int row = q / CPR, pc = q - row * CPR;
                const int64_t m = mrow0 + 32 * ip + row;
                if (q < kPieces && m < a.M && cbase * ESO + pc * 16 < a.Cout * ESO)
                    *(f32x4 *)((unsigned char *)gY + (m * a.Cout + cbase) * ESO + pc * 16) =
                        *(const f32x4 *)(stg + row * SR + pc * 16);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            const int64_t m = mrow0 + 32 * i + (lane & 31);
            if (m >= a.M) continue;
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int co = cbase + 32 * j + 8 * q + 4 * (lane >> 5) + e;
                    if (co >= a.Cout) continue;
                    const float y = acc[i][j][4 * q + e] + bias[j][q][e];
                    if constexpr (OUT_F32)
                        ((float *)gY)[m * a.Cout + co] = y;
                    else
                        ((__bf16 *)gY)[m * a.Cout + co] = (__bf16)y;
                }
        }
}

}  // namespace
}  // namespace dsattn
