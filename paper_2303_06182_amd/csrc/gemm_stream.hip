// Grouped expert GEMM for a handful of rows per expert:  C = A * B^T (+ bias, ReLU), bf16 activations, fp32 sums,
// weights bf16, e4m3 or mxfp4.  The weights are a stream that is read once; everything here serves its rate.
//
// What bounds it: HBM reads.  The tiled kernel (gemm_bf16.hip) moves the same bytes through LDS stages and barriers
// with one 32 x 128 tile per block, so a decoder step with few active experts has fewer tiles than the chip has CUs
// and each of them walks the whole of K alone.  Here
//  * a block owns 16 * NC output columns of one tile of at most 32 rows, and its W waves cut K between them: every
//    wave streams K / W of those columns' weights straight into MFMA operand registers (v_mfma_f32_16x16x32_bf16,
//    the weights as first operand), DP steps of loads in flight, no barrier, no LDS;
//  * at the end of the tile the W partial sums meet in LDS (added in wave order: the result is the same on every
//    run), and bias, scale, ReLU and the one rounding to bf16 happen there;
//  * a tile with at most 16 rows runs half the MFMAs and activation loads.
// Along K a lane may hold any elements as long as both operands agree, so its run is the one that makes full
// requests: 8 elements twice for bf16 (16 rows x 64 bytes; the second request finds the line in the L1), 16 for
// e4m3 and 32 for mxfp4, where the quantisers' blocked orders make every request one contiguous 1 KB.
// Those contiguous streams are read with the non-temporal policy; half lines must not be (their second half would
// be fetched again).
#include <mutex>
#include <type_traits>

#include "gemm_bf16_dev.h"
#include "moe_internal.h"

namespace moe355 {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

static constexpr int kStreamGroupM = 4;  // row tiles that take turns on the same columns (experts with several share their weights in L2)

// An address that is the same for every lane, kept in scalar registers: the loads then take it plus a 32-bit lane
// offset.  Left to itself the compiler carries one 64-bit vector pointer per load through the loop and spills.
__device__ __forceinline__ const uint8_t *scalar_base(const uint8_t *ptr)
{
    asm volatile("" : "+s"(ptr));
    return ptr;
}

// BQ: weight storage as in gemm_bf16.hip (0 bf16, 8 e4m3, 4 mxfp4).  DP1 / DP2: K steps in flight per wave for tiles
// of up to 16 / 32 rows (the step count of a wave is a multiple of both).  RAGGED (bf16): any K and N that are
// multiples of 8: the waves' shares of K differ by a step, both operands are zero past the end of K (their loads
// repeat the row's last 16 bytes), columns past N repeat the last weight row and are not stored.
template <int BQ, bool RELU, int NC, int W, int DP1, int DP2, bool RAGGED = false>
__global__ __launch_bounds__(W * 64, W == 8 ? 4 : 3) void gemm_stream_kernel(GemmParams p)
{
    constexpr bool B8 = BQ == 8, B4 = BQ == 4;
    static_assert(!RAGGED || BQ == 0, "8- and 4-bit weights come in whole blocks");
    constexpr int KSTEP = B4 ? 128 : 64;       // K elements of one step
    constexpr int NF = KSTEP / 32;             // MFMA operands along K per step
    constexpr int NB = BQ == 0 ? 2 : 1;        // 16-byte weight loads per step and 16 columns
    constexpr int BSTEP = B4 ? 2048 : B8 ? 1024 : 128;  // bytes a step advances in the weights
    constexpr int COLS = 16 * NC;
    constexpr bool TURNED = !B4 && !RAGGED;
    constexpr int LROW = COLS + 4;             // floats per LDS row of partial sums
    constexpr int NBUF = NC > 2 ? 1 : 2;       // two tiles' worth saves one of the two barriers per tile
    constexpr bool SC4 = B4 && (DP1 == 4 || NC == 4);       // block scales of four steps in one 16-byte load (a wave's steps are a multiple of 4)
    __shared__ float red[NBUF][W][32][LROW];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r16 = lane & 15, kq = lane >> 4;
    const int K = p.K;
    const int all_steps = (K + KSTEP - 1) / KSTEP;
    const int s_begin = all_steps * wave / W, n_steps = all_steps * (wave + 1) / W - s_begin;  // not RAGGED: K / W each
    const int KW = RAGGED ? 0 : K / W;
    const int n_tiles = (p.N + COLS - 1) / COLS;
    const int m_tiles = uniform_load(p.num_tiles);
    const int live = m_tiles * n_tiles, chunk = (live + 7) >> 3, xcd = blockIdx.x & 7, slots = gridDim.x >> 3;

    if (p.c_zero_row >= 0 && blockIdx.x == 0) {  // the all-zero row that the next GEMM may read
        uint16_t *z = static_cast<uint16_t *>(p.C) + (int64_t)p.c_zero_row * p.ldc;
        for (int i = tid * 8; i < p.N; i += W * 64 * 8) *reinterpret_cast<uint4 *>(z + i) = make_uint4(0, 0, 0, 0);
    }

    int buf = 0;
    for (int seq = blockIdx.x >> 3; seq < chunk && xcd * chunk + seq < live; seq += slots) {
        const int lid = xcd * chunk + seq;
        const int grp = lid / (kStreamGroupM * n_tiles), within = lid - grp * (kStreamGroupM * n_tiles);
        const int gsz = min(kStreamGroupM, m_tiles - grp * kStreamGroupM);
        const int mt = grp * kStreamGroupM + within % gsz, n0 = within / gsz * COLS;
        int expert, row0;
        uniform_load2(p.tile_expert + mt, p.tile_row + mt, expert, row0);
        const int row_end = min(uniform_load(p.offsets + expert + 1), row0 + 32);
        const int slot = p.b_slot ? uniform_load(p.b_slot + expert) : expert;
        int turn = 0;  // the step of its part of K that a wave begins with
        if constexpr (TURNED)
            if (p.turned) turn = (int)((uint32_t)(expert * 5 + n0 / COLS) % (uint32_t)n_steps);
        (void)turn;

        // weights: a base that is the same for every lane (expert, columns, the wave's part of K) + a lane offset
        const uint8_t *bbase;
        uint32_t boff;        // the lane's offset
        uint32_t bcol;        // bytes between two blocks of 16 columns (mxfp4: between two groups of 32)
        const uint8_t *sbase = nullptr;
        uint32_t soff = 0;
        if constexpr (BQ == 0) {
            bbase = static_cast<const uint8_t *>(p.B) + ((int64_t)slot * p.strideB + (int64_t)n0 * p.ldb + s_begin * KSTEP) * 2;
            boff = (uint32_t)r16 * (uint32_t)p.ldb * 2u + kq * 16;
            bcol = 16u * (uint32_t)p.ldb * 2u;
        } else if constexpr (B8) {  // [16 rows][64 bytes] blocks, along K inside a 16-row group
            bbase = static_cast<const uint8_t *>(p.B) + (int64_t)slot * p.strideB + (int64_t)n0 * K + wave * (KW / 64) * 1024;
            boff = r16 * 64 + kq * 16;
            bcol = 16u * (uint32_t)K;
        } else {  // [32 rows][32 bytes] blocks, along K inside a 32-row group; a step covers two blocks
            bbase = static_cast<const uint8_t *>(p.B) + (int64_t)slot * p.strideB + (int64_t)(n0 >> 5) * (K / 2) * 32 +
                    (n0 & 16) * 32 + wave * (KW / 64) * 1024;
            boff = (kq >> 1) * 1024 + r16 * 32 + (kq & 1) * 16;
            bcol = 16u * (uint32_t)K;
            sbase = p.b_blk_scale + (int64_t)expert * p.stride_blk_scale + (int64_t)(n0 >> 5) * ((K + 511) >> 9) * 512 +
                    (n0 & 16) * 16;
            soff = r16 * 16;
        }
        auto bblock = [&](int c) { return B4 ? (c >> 1) * bcol + (c & 1) * 512u : c * bcol; };
        const uint32_t sgroup = ((uint32_t)(K + 511) >> 9) * 512u;
        (void)sgroup;

        auto tile = [&](auto rc, auto dpc) {
            constexpr int R = decltype(rc)::value, DP = decltype(dpc)::value;
            uint32_t aoff[R];
            const uint8_t *aptr[R], *bptr[NC];  // RAGGED: the lane's rows at its first k of the wave's first step
#pragma unroll
            for (int r = 0; r < R; ++r) {
                int gr = min(row0 + r * 16 + r16, row_end - 1);  // rows past the end repeat the last one, their results are not stored
                if (p.a_rows) gr = p.a_rows[gr];
                if constexpr (RAGGED) aptr[r] = static_cast<const uint8_t *>(p.A) + (int64_t)gr * p.lda * 2;
                aoff[r] = (uint32_t)gr * (uint32_t)p.lda * 2u + kq * (B4 ? 64 : B8 ? 32 : 16);
            }
            if constexpr (RAGGED) {
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    bptr[c] = static_cast<const uint8_t *>(p.B) + ((int64_t)slot * p.strideB + (int64_t)min(n0 + c * 16 + r16, p.N - 1) * p.ldb) * 2;
            }
            (void)aptr, (void)bptr;
            const uint8_t *abase = static_cast<const uint8_t *>(p.A) + s_begin * (KSTEP * 2);
            u32x4 bq[DP][NC][NB], aq[DP][R][NF];
            uint32_t sc[DP][NC];
            u32x4 sc_now[NC], sc_next[NC];  // mxfp4: the scale bytes of a 512-element group of the lane's rows
            (void)sc, (void)sc_now, (void)sc_next;
            f32x4 acc[R][NC];
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[r][c][i] = 0.f;
            auto load = [&](int d, int s) {
                if constexpr (RAGGED) {
#pragma unroll
                    for (int f = 0; f < NF; ++f) {
                        const int k = min((s_begin + s) * KSTEP + f * 32 + kq * 8, K - 8);
#pragma unroll
                        for (int c = 0; c < NC; ++c) bq[d][c][f] = *reinterpret_cast<const u32x4 *>(bptr[c] + (int64_t)k * 2);
#pragma unroll
                        for (int r = 0; r < R; ++r) aq[d][r][f] = *reinterpret_cast<const u32x4 *>(aptr[r] + (int64_t)k * 2);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    return;
                }
                if constexpr (TURNED) {
                    s += turn;
                    if (s >= n_steps) s -= n_steps;
                }
                const uint8_t *as = scalar_base(abase + s * (KSTEP * 2));
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const uint8_t *bs = scalar_base(bbase + s * BSTEP + bblock(c));
#pragma unroll
                    for (int j = 0; j < NB; ++j) {
                        const u32x4 *src = reinterpret_cast<const u32x4 *>(bs + boff + j * 64);
                        if constexpr (BQ == 0)
                            bq[d][c][j] = *src;
                        else
                            bq[d][c][j] = __builtin_nontemporal_load(src);
                    }
                }
                if constexpr (B4 && !SC4) {
                    const int g = wave * (KW / 128) + s;  // four scale bytes per step: byte 4 (g mod 4) + kq of group g / 4
                    const uint8_t *ss = sbase + (g >> 2) * 512 + (g & 3) * 4;
#pragma unroll
                    for (int c = 0; c < NC; ++c) sc[d][c] = scalar_base(ss + (c >> 1) * sgroup + (c & 1) * 256)[soff + kq];
                }
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int f = 0; f < NF; ++f)
                        aq[d][r][f] = *reinterpret_cast<const u32x4 *>(as + aoff[r] + (BQ == 0 ? f * 64 : f * 16));
                __builtin_amdgcn_sched_barrier(0);
            };
            auto load_scales = [&](int s) {  // of steps s .. s + 3
                const uint8_t *ss = sbase + ((wave * (KW / 128) + s) >> 2) * 512;
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    sc_next[c] = *reinterpret_cast<const u32x4 *>(scalar_base(ss + (c >> 1) * sgroup + (c & 1) * 256) + soff);
            };
            auto compute = [&](int d, int quarter) {
                if constexpr (RAGGED) {  // quarter: the step
#pragma unroll
                    for (int f = 0; f < NF; ++f)
                        if ((s_begin + quarter) * KSTEP + f * 32 + kq * 8 >= K) {
#pragma unroll
                            for (int c = 0; c < NC; ++c) bq[d][c][f] = u32x4{0, 0, 0, 0};
#pragma unroll
                            for (int r = 0; r < R; ++r) aq[d][r][f] = u32x4{0, 0, 0, 0};
                        }
                }
#pragma unroll
                for (int f = 0; f < NF; ++f)
#pragma unroll
                    for (int c = 0; c < NC; ++c) {
                        u32x4 w;
                        if constexpr (BQ == 0) {
                            w = bq[d][c][f];
                        } else if constexpr (B8) {  // every e4m3 value is a bf16 value
#pragma unroll
                            for (int h = 0; h < 2; ++h) {
                                const uint32_t raw = bq[d][c][0][2 * f + h];
                                const f32x2 lo = __builtin_amdgcn_cvt_pk_f32_fp8(raw, false);
                                const f32x2 hi = __builtin_amdgcn_cvt_pk_f32_fp8(raw, true);
                                w[2 * h] = pack_bf16(lo[0], lo[1]);
                                w[2 * h + 1] = pack_bf16(hi[0], hi[1]);
                            }
                        } else {
                            const uint32_t raw = bq[d][c][0][f];
                            const uint32_t byte = SC4 ? (sc_now[c][quarter] >> (8 * kq)) & 0xffu : sc[d][c];
                            const float scale = __uint_as_float(byte << 23);  // 2^(byte - 127)
                            const bf16x2 e0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(raw, scale, 0);
                            const bf16x2 e1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(raw, scale, 1);
                            const bf16x2 e2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(raw, scale, 2);
                            const bf16x2 e3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(raw, scale, 3);
                            w[0] = __builtin_bit_cast(uint32_t, e0);
                            w[1] = __builtin_bit_cast(uint32_t, e1);
                            w[2] = __builtin_bit_cast(uint32_t, e2);
                            w[3] = __builtin_bit_cast(uint32_t, e3);
                        }
#pragma unroll
                        for (int r = 0; r < R; ++r)
                            acc[r][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w),
                                                                                __builtin_bit_cast(bf16x8, aq[d][r][f]),
                                                                                acc[r][c], 0, 0, 0);
                    }
                __builtin_amdgcn_sched_barrier(0);
            };
            if constexpr (RAGGED) {
                // whole rounds with the next round's loads behind each step, then the last one to two rounds
#pragma unroll
                for (int d = 0; d < DP; ++d) load(d, d);
                int s = 0;
                for (; s + 2 * DP <= n_steps; s += DP)
#pragma unroll
                    for (int d = 0; d < DP; ++d) {
                        compute(d, s + d);
                        load(d, s + DP + d);
                    }
#pragma unroll
                for (int d = 0; d < DP; ++d) {
                    if (s + d < n_steps) compute(d, s + d);
                    if (s + DP + d < n_steps) load(d, s + DP + d);
                }
#pragma unroll
                for (int d = 0; d < DP; ++d)
                    if (s + DP + d < n_steps) compute(d, s + DP + d);
            } else if constexpr (SC4) {  // the loop below goes four steps at a time, the scales one such group ahead
                static_assert(4 % DP == 0, "a group of four steps is whole rounds of the load ring");
                load_scales(0);
#pragma unroll
                for (int d = 0; d < DP; ++d) load(d, d);
                for (int s = 4; s < n_steps; s += 4) {
#pragma unroll
                    for (int c = 0; c < NC; ++c) sc_now[c] = sc_next[c];
                    load_scales(s);
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        compute(q % DP, q);
                        load(q % DP, s - 4 + q + DP);
                    }
                }
#pragma unroll
                for (int c = 0; c < NC; ++c) sc_now[c] = sc_next[c];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    compute(q % DP, q);
                    if (q + DP < 4) load(q % DP, n_steps - 4 + q + DP);
                }
            } else {
#pragma unroll
                for (int d = 0; d < DP; ++d) load(d, d);
                for (int s = DP; s < n_steps; s += DP)
#pragma unroll
                    for (int d = 0; d < DP; ++d) {
                        compute(d, 0);
                        load(d, s + d);
                    }
#pragma unroll
                for (int d = 0; d < DP; ++d) compute(d, 0);
            }
            // lane: row r16 of block r, columns 4 kq .. 4 kq + 3 of block c
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    *reinterpret_cast<f32x4 *>(&red[buf][wave][r * 16 + r16][c * 16 + kq * 4]) = acc[r][c];
        };
        if (row_end - row0 <= 16)
            tile(std::integral_constant<int, 1>{}, std::integral_constant<int, DP1>{});
        else
            tile(std::integral_constant<int, 2>{}, std::integral_constant<int, DP2>{});

        // With two buffers one barrier per tile is enough: behind it the partial sums of this tile are complete and every
        // wave has read those of the tile before, whose buffer the next tile writes.
        __syncthreads();
        const float b_scale = (B8 && p.b_scale) ? __int_as_float(uniform_load(reinterpret_cast<const int32_t *>(p.b_scale) + expert)) : 1.f;
        const uint16_t *bias = static_cast<const uint16_t *>(p.bias);
        for (int i = tid; i < (row_end - row0) * (COLS / 2); i += W * 64) {
            const int r = i / (COLS / 2), c = (i % (COLS / 2)) * 2;
            if (RAGGED && n0 + c >= p.N) continue;  // N is even
            float v0 = red[buf][0][r][c], v1 = red[buf][0][r][c + 1];
#pragma unroll
            for (int w = 1; w < W; ++w) {
                v0 += red[buf][w][r][c];
                v1 += red[buf][w][r][c + 1];
            }
            if constexpr (B8) {
                v0 *= b_scale;
                v1 *= b_scale;
            }
            if (bias) {
                const uint32_t bb = *reinterpret_cast<const uint32_t *>(bias + (int64_t)expert * p.strideBias + n0 + c);
                v0 += __uint_as_float(bb << 16);
                v1 += __uint_as_float(bb & 0xffff0000u);
            }
            uint32_t o = pack_bf16(v0, v1);
            if (RELU) o = relu_bf16x2(o);
            *reinterpret_cast<uint32_t *>(static_cast<uint16_t *>(p.C) + (int64_t)(row0 + r) * p.ldc + n0 + c) = o;
        }
        if constexpr (NBUF == 2)
            buf ^= 1;
        else
            __syncthreads();
    }
}

template <int BQ, bool RELU, int NC, int W, int DP1, int DP2, bool RAGGED = false>
static int launch_stream_t(const GemmParams &p_in, int num_cus, hipStream_t s)
{
    GemmParams p = p_in;
    if (p.chosen) {
        *p.chosen = kChosenStream + 16 * NC;
        return MOE_OK;
    }
    auto kern = gemm_stream_kernel<BQ, RELU, NC, W, DP1, DP2, RAGGED>;
    static std::once_flag once;
    static int blocks_per_cu = 1;
    static hipError_t setup_rc = hipSuccess;
    std::call_once(once, [&]() {
        int occ = 0;
        setup_rc = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kern, W * 64, 0);
        blocks_per_cu = occ < 1 ? 1 : (occ > 16 ? 16 : occ);
    });
    MOE_HIP_CHECK(setup_rc);
    const int64_t tiles = (int64_t)(p.max_m_tiles < p.M ? p.max_m_tiles : p.M) * ceil_div(p.N, 16 * NC);  // every tile has a row
    int64_t grid = (int64_t)num_cus * blocks_per_cu;
    if (grid > tiles) grid = tiles;
    grid = align_up(grid, 8);
    // FFN in us, a wave's part of K from its beginning / turned: 16 experts 2048 -> 8192, 4 active 57 / 52, 8 active 90 / 86, 16 active 192 / 182; 64
    // experts 1024 -> 4096 50 / 49; e4m3: 16 experts 2048 -> 8192, 1 row each 119 / 89, 4 active 27 / 24, 64 experts 1024 -> 4096, 1 row each 104 / 90.
    // With K of 2048 not for few columns (second GEMM of 128 experts 512 -> 2048, 8 active, bf16 20.8 / 21.3; 64 experts, e4m3 29.4 / 30.8).
    p.turned = p.K % (2 * kTurnedK) == 0 || (p.K % kTurnedK == 0 && p.N >= 2048);
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(W * 64), 0, s, p);
    MOE_LAUNCH_CHECK("gemm_stream_kernel");
    return MOE_OK;
}

// K steps of a wave when W waves share K, 0 when they do not divide it
template <int BQ>
static int stream_steps(int K, int W)
{
    const int step = (BQ == 4 ? 128 : 64) * W;
    return K % step == 0 ? K / step : 0;
}

// Which calls this kernel takes from the tiled one, and how it cuts them.  m_up bounds the row tiles from above on the
// host (the true count is on the device).  Measured per GEMM on layers of 128 experts 2048 -> 8192, 512 experts
// 1024 -> 4096 and 64 experts 512 -> 2048, top-2, 1 ... 6144 tokens; us, this kernel / the tiled one:
//  * bf16: only while the tiled kernel's 32 x 128 tiles are fewer than 1.5 per CU (1 token 14.5 / 98.6, 8 tokens
//    94 / 121 on the 2048 layer's second GEMM); from there on that kernel reads whole lines with the non-temporal
//    policy (6.3 TB/s) and this one cannot (1.9 tiles per CU 94 / 80, 64 tokens 494 / 447).  Between 1 and 1.5 tiles per CU
//    only up to 8 rows per expert on average: with more, tiles of 17 ... 32 rows come up (16 experts 2048 -> 8192, second GEMM:
//    8 rows 112 / 133, 12 rows even 117 / 132, skewed 160 / 135; 8 experts, 36 rows 123 / 108).  And not for K below 256,
//    where a wave has a step or none (a layer of 64 experts 64 -> 64, 512 tokens: 34.9 / 31.1).
//  * e4m3 and mxfp4: up to 64 / 128 rows in all, or while the tiled kernel has at most one 128-column / two 256-column
//    tiles per CU (rows 1 token: 11 / 54 and 10 / 82 on the 2048 layer's second GEMM; 16 tokens 84 / 90 and 51 / 75 on
//    its first).  With more rows it is a matter of their spread: a tile of 17 ... 32 rows reads its activations 16 rows at a
//    time, four times slower per byte than whole lines, so that evenly spread rows still gain (256 tokens over
//    128 experts, mxfp4: 200 / 224) but a few hot experts cost more than that (same layer, skewed, 128 tokens: e4m3 304 / 185,
//    mxfp4 162 / 111).  The host does not know the spread, but the mean bounds it:
//    e4m3, up to half a tile per CU: any (8 experts 512 -> 2048, 24 rows, second GEMM 9 / 18, skewed 13 / 18); up to
//    one: 20 rows per expert (second GEMM, even, skewed, more skewed; 8 experts 2048 -> 8192, 20 rows
//    39 / 55, 43 / 54, 60 / 54, 24 rows 45 / 54, 60 / 55, 60 / 54; 32 experts 512 -> 2048, 24 rows 19 / 18 for all); else up to 64
//    rows, one per expert (32 experts 2048 -> 8192, 2 rows, second GEMM 87 / 81, 83 / 78, 79 / 63; 8 experts, 4 rows, first
//    33 / 30), or two with less than 1.5 tiles per CU (16 experts 2048 -> 8192, second GEMM 46 / 56).
//    mxfp4, up to one tile per CU: any (16 experts 2048 -> 8192, 30 rows, second GEMM 63 / 80 for every spread); up to two: 16 rows
//    per expert (second GEMM, even, skewed, more skewed; 64 experts 1024 -> 4096, 16 rows 40 / 44, 51 / 54, 53 / 55, 30 rows
//    63 / 57, 62 / 56, 71 / 56; 32 experts 2048 -> 8192, 24 rows 99 / 104, 100 / 103, 115 / 103); else up to 64 rows, 128 with
//    less than six tiles per CU, two per expert (first GEMM; 64 experts 1024 -> 4096, 2 rows 25 / 35, 26 / 35, 24 / 25; 128
//    experts 2048 -> 8192, 128 rows 119 / 131, 111 / 124, 94 / 76; 16 experts 2048 -> 8192, 8 rows 37 / 35, 38 / 35, 49 / 36).
template <int BQ>
static bool stream_pays(const GemmParams &p, int num_cus, int64_t m_up)
{
    const int64_t tiles = m_up * ceil_div(p.N, BQ == 4 ? 256 : 128), E = p.num_experts;
    if (BQ == 0)
        return p.K >= 256 && (tiles <= num_cus || (2 * tiles < 3 * (int64_t)num_cus && p.M <= 8 * E));
    if (BQ == 8) {
        if (tiles <= num_cus) return 2 * tiles <= num_cus || p.M <= 20 * E;
        return p.M <= 64 && p.M <= (2 * tiles < 3 * (int64_t)num_cus ? 2 * E : E);
    }
    if (tiles <= 2 * (int64_t)num_cus) return tiles <= num_cus || p.M <= 16 * E;
    return p.M <= (tiles < 6 * (int64_t)num_cus ? 128 : 64) && p.M <= 2 * E;
}

template <int BQ, bool RELU>
static int launch_stream_q(const GemmParams &p, int num_cus, hipStream_t s, bool *taken)
{
    const int64_t m_up = p.max_m_tiles < p.M ? p.max_m_tiles : p.M;  // every tile has a row
    const bool pays = stream_pays<BQ>(p, num_cus, m_up);
    if constexpr (BQ == 0) {
        if (pays && (p.N % 32 != 0 || stream_steps<BQ>(p.K, 4) == 0 || stream_steps<BQ>(p.K, 4) % 2 != 0)) {
            *taken = true;
            return m_up * ceil_div(p.N, 32) < num_cus ? launch_stream_t<BQ, RELU, 1, 8, 2, 2, true>(p, num_cus, s)
                                                      : launch_stream_t<BQ, RELU, 2, 4, 2, 2, true>(p, num_cus, s);
        }
    }
    if (p.N % 32 != 0 || !pays) return MOE_OK;
    *taken = true;
    const int n8 = stream_steps<BQ>(p.K, 8), n4 = stream_steps<BQ>(p.K, 4);
    // fewer than one 32-column tile per CU: 16 columns and eight waves each (1 token, bf16 21.2 -> 14.5 us; with more
    // tiles than that the wider ones are faster: 2 tokens 28.4 against 35.1)
    if (m_up * (p.N / 32) < num_cus && n8 >= 2) {
        if (n8 % 4 == 0) return launch_stream_t<BQ, RELU, 1, 8, 4, 2>(p, num_cus, s);
        if (n8 % 2 == 0) return launch_stream_t<BQ, RELU, 1, 8, 2, 2>(p, num_cus, s);
    }
    if constexpr (BQ == 4) {
        // 4-bit weights: 64 columns halve the activation and scale loads per weight byte (64 tokens 295 -> 271 us per
        // layer), as many waves as keep four steps each, so that their scales come as one load
        const int n2 = stream_steps<BQ>(p.K, 2), n1 = stream_steps<BQ>(p.K, 1);
        if (p.N % 64 == 0 && m_up * (p.N / 64) >= 2 * (int64_t)num_cus) {
            if (n4 > 0 && n4 % 4 == 0) return launch_stream_t<BQ, RELU, 4, 4, 2, 1>(p, num_cus, s);
            if (n2 > 0 && n2 % 4 == 0) return launch_stream_t<BQ, RELU, 4, 2, 2, 1>(p, num_cus, s);
            if (n1 > 0 && n1 % 4 == 0) return launch_stream_t<BQ, RELU, 4, 1, 2, 1>(p, num_cus, s);
        }
    }
    if (n4 > 0 && n4 % 4 == 0) return launch_stream_t<BQ, RELU, 2, 4, 4, 2>(p, num_cus, s);
    if (n4 > 0 && n4 % 2 == 0) return launch_stream_t<BQ, RELU, 2, 4, 2, 2>(p, num_cus, s);
    if constexpr (BQ == 4) {
        const int n1 = stream_steps<BQ>(p.K, 1);
        if (n1 > 0 && n1 % 4 == 0) return launch_stream_t<BQ, RELU, 2, 1, 4, 2>(p, num_cus, s);
    }
    *taken = false;
    return MOE_OK;
}

// *taken = false: this kernel does not serve the call (nothing was launched).  p: a grouped GEMM over a map of tiles
// of at most 32 rows, bf16 output.
int launch_gemm_stream(const GemmParams &p, int wbits, bool relu, int num_cus, hipStream_t s, bool *taken)
{
    *taken = false;
    // 32-bit lane offsets into A (a gathered A is the token array: its caller checked that it fits)
    if (!p.a_rows && (int64_t)p.M * p.lda * 2 >= (1ll << 32)) return MOE_OK;
    if (wbits == 8) return relu ? launch_stream_q<8, true>(p, num_cus, s, taken) : launch_stream_q<8, false>(p, num_cus, s, taken);
    if (wbits == 4) return relu ? launch_stream_q<4, true>(p, num_cus, s, taken) : launch_stream_q<4, false>(p, num_cus, s, taken);
    return relu ? launch_stream_q<0, true>(p, num_cus, s, taken) : launch_stream_q<0, false>(p, num_cus, s, taken);
}

}  // namespace moe355
