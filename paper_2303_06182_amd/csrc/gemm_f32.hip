// fp32 GEMM  C = A * B^T (+ bias, ReLU), plain or grouped, for the fp32 storage type (the accuracy configuration:
// fp32 products and fp32 sums, 1e-5 tolerance).  Two kernels on the fp32 matrix pipes (64 flop per clock and SIMD):
//  * gemm_f32_wave_kernel: 32 x 32 outputs per block, K cut between the block's W waves.  A wave fills an LDS ring of its
//    own (RING steps of 32 k: 32 + 32 rows of 128 bytes) with global_load_lds_dwordx4 and multiplies it with
//    v_mfma_f32_16x16x4_f32; no barrier in the K loop, since nobody else reads the ring.  The W partial sums meet in LDS
//    at the end, added in wave order.  Small and medium batches are bound by the serial chain of MFMAs behind one tile
//    and by how evenly few tiles spread over the CUs: this cuts both by four.  (Operand fragments loaded straight into
//    registers instead: neighbouring lanes then belong to different rows, a request of 64 lanes takes four times as
//    long, and 512 tokens over 8 experts 512 -> 2048 took 57 + 55 us.)
//  * gemm_f32_tile_kernel (K a multiple of 32, large batches): 64 x 64 x 32 tile, four waves of 32 x 32 outputs each on
//    v_mfma_f32_32x32x2_f32, shared LDS stages: half the operand bytes per flop.  Operand rows
//    are 128 bytes per K tile, laid out in LDS like the bf16 kernel's (16-byte chunk c of row r at chunk
//    position c ^ ((r >> 1) & 7): conflict-free 16-byte fragment reads), filled by global_load_lds_dwordx4
//    three stages deep.  One 16-byte fragment read feeds four MFMAs: the instruction contracts over two
//    k slots per step, lanes 0-31 supplying one and lanes 32-63 the other, and WHICH k a slot stands for
//    is free as long as both operands agree -- so the lower lanes take chunk 2j, the upper lanes chunk
//    2j + 1, and the four floats of a chunk are four steps.
#include <mutex>

#include "moe_internal.h"

namespace moe355 {

typedef __attribute__((address_space(3))) void lds_void_f;
typedef __attribute__((address_space(1))) void glb_void_f;
typedef float floatx16 __attribute__((ext_vector_type(16)));
// Fragment reads go through a vector type: an LDS read that carries type-based alias information (float4 is a
// struct of floats) is ordered by the compiler after every direct-to-LDS load in flight (vmcnt(0) in front of
// the read), which would undo the pipeline; the explicit vmcnt before each barrier is what orders them.
typedef float floatx4 __attribute__((ext_vector_type(4)));

static constexpr int MBM = 64, MBN = 64, MBK = 32, MSTAGES = 3;

template <bool RELU, bool GROUPED>
__global__ __launch_bounds__(256) void gemm_f32_tile_kernel(GemmParams p)
{
    // [stage][A rows 0..63 | B rows 0..63][32 floats], chunk-swizzled
    extern __shared__ __attribute__((aligned(1024))) float smem_dyn[];
    float (*smem)[(MBM + MBN) * MBK] = reinterpret_cast<float (*)[(MBM + MBN) * MBK]>(smem_dyn);

    const int n_tiles = (p.N + MBN - 1) / MBN;
    const int mt = blockIdx.x / n_tiles;
    const int nt = blockIdx.x - mt * n_tiles;
    int row0, row_end, expert = 0;
    if (GROUPED) {
        if (mt >= p.num_tiles[0]) return;
        expert = p.tile_expert[mt];
        row0 = p.tile_row[mt];
        row_end = p.offsets[expert + 1];
    } else {
        row0 = mt * MBM;
        row_end = p.M;
        if (row0 >= row_end) return;
    }
    const int n0 = nt * MBN;
    const float *Ag = static_cast<const float *>(p.A);
    const float *Bg = static_cast<const float *>(p.B) + (int64_t)((GROUPED && p.b_slot) ? p.b_slot[expert] : expert) * p.strideB;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;

    // Loads: one wave instruction fills 8 rows x 128 B of LDS in lane order (lane -> 16 bytes at 16 * lane),
    // so the swizzle is applied on the global side: the lane that fills chunk position cp of row r fetches
    // chunk cp ^ ((r >> 1) & 7).  Wave w fills rows 16 w .. 16 w + 15 of A and of B.  Rows past the end of
    // the batch / of the matrix re-read the last valid row; their products are never stored.
    const float *a_src[2], *b_src[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int r = wave * 16 + i * 8 + (lane >> 3);
        const int c = (lane & 7) ^ ((r >> 1) & 7);
        int gr = min(row0 + r, row_end - 1);
        if (GROUPED && p.a_rows) gr = p.a_rows[gr];
        a_src[i] = Ag + (int64_t)gr * p.lda + c * 4;
        b_src[i] = Bg + (int64_t)min(n0 + r, p.N - 1) * p.ldb + c * 4;
    }
    auto issue = [&](int kt, int stage) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
            __builtin_amdgcn_global_load_lds((const glb_void_f *)(a_src[i] + kt * MBK),
                                             (lds_void_f *)(&smem[stage][(wave * 16 + i * 8) * MBK]), 16, 0, 0);
#pragma unroll
        for (int i = 0; i < 2; ++i)
            __builtin_amdgcn_global_load_lds((const glb_void_f *)(b_src[i] + kt * MBK),
                                             (lds_void_f *)(&smem[stage][(MBM + wave * 16 + i * 8) * MBK]), 16, 0, 0);
    };
    constexpr int LPS = 4;  // load instructions per wave and stage

    // fragment addresses: row lane % 32 of the wave's 32-row block, chunk 2 j + lane / 32
    const int fr = lane & 31, fh = lane >> 5;
    const int ar = wm * 32 + fr, br = MBM + wn * 32 + fr;
    const int a_swz = (ar >> 1) & 7, b_swz = (br >> 1) & 7;

    floatx16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;

    const int KT = p.K / MBK;
    // the loads run MSTAGES - 1 K tiles ahead; past the end they re-read the last K tile into a stage
    // nobody reads any more, so every iteration issues the same number and the vmcnt arithmetic is fixed
#pragma unroll
    for (int i = 0; i < MSTAGES - 1; ++i) issue(min(i, KT - 1), i);
    // s_waitcnt through the builtin (the compiler's wait-count bookkeeping cannot see into inline assembly):
    // vmcnt in bits 3:0, expcnt (bits 6:4) at "no wait", lgkmcnt (bits 11:8) 0 or "no wait"
    constexpr int kWaitStage = ((MSTAGES - 2) * LPS) | (7 << 4);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(kWaitStage | (15 << 8));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    int stage = 0, lstage = MSTAGES - 1;
    for (int kt = 0; kt < KT; ++kt) {
        issue(min(kt + MSTAGES - 1, KT - 1), lstage);  // into the stage the previous iteration read
        lstage = lstage + 1 == MSTAGES ? 0 : lstage + 1;
        const float *sa = &smem[stage][ar * MBK], *sb = &smem[stage][br * MBK];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const floatx4 a4 = *reinterpret_cast<const floatx4 *>(sa + (((2 * j + fh) ^ a_swz) << 2));
            const floatx4 b4 = *reinterpret_cast<const floatx4 *>(sb + (((2 * j + fh) ^ b_swz) << 2));
            // weights first: a lane then owns one output row and 4 x 4 consecutive output columns
#pragma unroll
            for (int q = 0; q < 4; ++q) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(b4[q], a4[q], acc, 0, 0, 0);
        }
        // the K tile read next has landed (this wave's part; the barrier covers the others'), and every
        // fragment read of this stage has returned before another wave may refill it
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(kWaitStage);  // and lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        stage = stage + 1 == MSTAGES ? 0 : stage + 1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no LDS write may outlive the block

    // lane: output row wm*32 + lane%32; register 4 g + i: column wn*32 + 8 g + 4 (lane/32) + i
    const int row = row0 + wm * 32 + fr;
    if (row >= row_end) return;
    const float *bias = static_cast<const float *>(p.bias);
    if (bias) bias += (int64_t)expert * p.strideBias;
    float *c_row = static_cast<float *>(p.C) + (int64_t)row * p.ldc;
    const bool vec_ok = (p.ldc & 3) == 0;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const int col = n0 + wn * 32 + g * 8 + fh * 4;
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[i] = acc[g * 4 + i];
            if (col + i < p.N) {
                if (bias) v[i] += bias[col + i];
                if (p.bias_f32) v[i] += p.bias_f32[col + i];
            }
            if (RELU) v[i] = v[i] > 0.f ? v[i] : 0.f;
        }
        if (vec_ok && col + 3 < p.N) {
            *reinterpret_cast<float4 *>(c_row + col) = make_float4(v[0], v[1], v[2], v[3]);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (col + i < p.N) c_row[col + i] = v[i];
        }
    }
}

static constexpr int kF32GroupM = 4;  // row tiles that take turns on the same columns
static constexpr int kF32Ring = 2;    // LDS slots of a wave: 16 KB, two blocks of four waves per CU

// A ring row is 128 bytes, a whole line of its operand row (with 64-byte rows every line was fetched twice by the time
// its second half was wanted: 115 TFLOP/s became 76 on large batches); the 16 bytes at position q of row r hold K chunk
// q ^ ((r >> 1) & 7), which keeps a fragment read (16 rows, one chunk each) on 16 different bank groups; the
// permutation is applied on the global side of the load.
template <int W, bool RELU, bool GROUPED>
__global__ __launch_bounds__(W * 64) void gemm_f32_wave_kernel(GemmParams p)
{
    constexpr int RING = kF32Ring;
    constexpr int SLOT = 64 * 128;  // bytes: 32 rows of A, then 32 rows of B, 32 k each
    constexpr int LROW = 32 + 4;   // floats per row of partial sums
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem_wave[];  // [W][RING][SLOT], later the partial sums
    static_assert(W * RING * SLOT >= W * 32 * LROW * 4, "the partial sums reuse the ring");

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r16 = lane & 15, kq = lane >> 4;
    const int n_tiles = (p.N + 31) / 32;
    const int m_tiles = GROUPED ? p.num_tiles[0] : (p.M + 31) / 32;
    // the grid covers the host's upper bound of the tiles; XCD x takes a contiguous range of the list, so that the row
    // tiles of an expert find its weights in one L2
    const int live = m_tiles * n_tiles, chunk = (live + 7) >> 3;
    const int seq = blockIdx.x >> 3, lid = (blockIdx.x & 7) * chunk + seq;
    if (seq >= chunk || lid >= live) return;
    const int grp = lid / (kF32GroupM * n_tiles), within = lid - grp * (kF32GroupM * n_tiles);
    const int gsz = min(kF32GroupM, m_tiles - grp * kF32GroupM);
    const int mt = grp * kF32GroupM + within % gsz, n0 = within / gsz * 32;
    int row0, row_end, expert = 0;
    if (GROUPED) {
        expert = p.tile_expert[mt];
        row0 = p.tile_row[mt];
        row_end = p.offsets[expert + 1];
    } else {
        row0 = mt * 32;
        row_end = p.M;
    }
    const float *Bg = static_cast<const float *>(p.B) + (int64_t)((GROUPED && p.b_slot) ? p.b_slot[expert] : expert) * p.strideB;

    // this wave's steps of 32 k
    const int steps = (p.K + 31) >> 5;
    const int s_begin = steps * wave / W, n = steps * (wave + 1) / W - s_begin;
    uint8_t *ring = smem_wave + wave * (RING * SLOT);
    // load i fills ring rows 8 i .. 8 i + 7 (0 .. 3: A, 4 .. 7: B): lane l lands at byte 16 l, i.e. position l % 8 of row l / 8
    constexpr int LOADS = 8;
    const float *src[LOADS];
    int ld_k[2];  // the lane's first k of a step: rows 8 i + l / 8 with i even / odd
#pragma unroll
    for (int i = 0; i < LOADS; ++i) {
        const int r = (i & 3) * 8 + (lane >> 3);
        if (i < 2) ld_k[i] = ((lane & 7) ^ ((r >> 1) & 7)) * 4;
        if (i < 4) {
            int gr = min(row0 + r, row_end - 1);  // rows past the end repeat the last one; they are not stored
            if (GROUPED && p.a_rows) gr = p.a_rows[gr];
            src[i] = static_cast<const float *>(p.A) + (int64_t)gr * p.lda;
        } else {
            src[i] = Bg + (int64_t)min(n0 + r, p.N - 1) * p.ldb;
        }
    }
    const int k_last = p.K - 4;  // the last 16 bytes of a row
    auto load = [&](int slot, int s) {  // step s of this wave; past K: the row's end again, multiplied as zeros or not at all
        const int k0 = min((s_begin + s) * 32 + ld_k[0], k_last), k1 = min((s_begin + s) * 32 + ld_k[1], k_last);
#pragma unroll
        for (int i = 0; i < LOADS; ++i)
            __builtin_amdgcn_global_load_lds((const glb_void_f *)(src[i] + ((i & 1) ? k1 : k0)),
                                             (lds_void_f *)(ring + slot * SLOT + i * 1024), 16, 0, 0);
    };
    floatx4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[i][j][c] = 0.f;
    const uint8_t *frag = ring + r16 * 128;
    const int swz = (r16 >> 1) & 7;  // == (row >> 1) & 7 of every row this lane reads
    // Every step issues one slot's loads, so "at most (RING - 1) * LOADS outstanding" means that the step's own have
    // landed.  A slot is refilled behind the MFMAs that consumed its fragments.
    constexpr int kWait = ((RING - 1) * LOADS) | (7 << 4) | (15 << 8);
    static_assert((RING - 1) * LOADS < 16, "vmcnt in the low four bits");
#pragma unroll
    for (int d = 0; d < RING; ++d) load(d, d);
    for (int s = 0; s < n; s += RING)
#pragma unroll
        for (int d = 0; d < RING; ++d) {
            if (s + d >= n) break;
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(kWait);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
            floatx4 f[2][4];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int i = 0; i < 4; ++i)  // blocks of 16 rows: 0, 1 of A, 2, 3 of B
                    f[h][i] = *reinterpret_cast<const floatx4 *>(frag + d * SLOT + i * 2048 + (((h * 4 + kq) ^ swz) << 4));
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if ((s_begin + s + d) * 32 + h * 16 + kq * 4 > k_last) {  // K ends in this step: both operands, so that not even a NaN counts twice
#pragma unroll
                    for (int i = 0; i < 4; ++i) f[h][i] = floatx4{0.f, 0.f, 0.f, 0.f};
                }
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j)  // weights first: a lane then owns 4 consecutive columns of one row
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[h][2 + j][c], f[h][i][c], acc[i][j], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("" ::: "memory");
            load(d, s + d + RING);
        }
    // the ring becomes the partial sums: no load of any wave may still be in flight
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    float *red = reinterpret_cast<float *>(smem_wave);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
            *reinterpret_cast<floatx4 *>(red + (wave * 32 + i * 16 + r16) * LROW + j * 16 + kq * 4) = acc[i][j];
    __syncthreads();
    const float *bias = static_cast<const float *>(p.bias);
    if (bias) bias += (int64_t)expert * p.strideBias;
    // rows of C and of the biases stay 16-byte aligned then (their bases are)
    const bool vec_ok = (p.ldc & 3) == 0 && (p.N & 3) == 0;
    for (int i = threadIdx.x; i < 32 * 8; i += W * 64) {
        const int r = i >> 3, c4 = (i & 7) * 4, col = n0 + c4;
        if (row0 + r >= row_end || col >= p.N) continue;
        floatx4 v = *reinterpret_cast<const floatx4 *>(red + r * LROW + c4);
#pragma unroll
        for (int w = 1; w < W; ++w) v += *reinterpret_cast<const floatx4 *>(red + (w * 32 + r) * LROW + c4);
        float *c = static_cast<float *>(p.C) + (int64_t)(row0 + r) * p.ldc + col;
        if (vec_ok) {
            if (bias) v += *reinterpret_cast<const floatx4 *>(bias + col);
            if (p.bias_f32) v += *reinterpret_cast<const floatx4 *>(p.bias_f32 + col);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (RELU) v[q] = v[q] > 0.f ? v[q] : 0.f;
            *reinterpret_cast<floatx4 *>(c) = v;
            continue;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (col + q >= p.N) break;
            float o = v[q];
            if (bias) o += bias[col + q];
            if (p.bias_f32) o += p.bias_f32[col + q];
            if (RELU) o = o > 0.f ? o : 0.f;
            c[q] = o;
        }
    }
}

// variant 1: 32-row tiles, K cut between the waves of a block; 0: 64-row tiles.
// The 64 x 64 tiles win once they fill the chip evenly without help; a short K moves that point down, because each
// wave's quarter of it then no longer hides a tile's start.  us, wave / tile kernel, top-2: K = 2048, N = 512, 8 experts:
// 512 tokens 37 / 46, 1024 56 / 76, 4096 176 / 178; K = 512, N = 2048: 512 tokens 37 / 35, 1024 65 / 61, 2048
// 117 / 91; K = 1024, N = 4096: 256 tokens 71 / 81, 512 110 / 114, 1024 194 / 166; K = 4096, N = 1024: 512 tokens
// 105 / 146, 2048 344 / 348, 4096 650 / 619.  Where the two GEMMs of a layer differ a second tile map (5 us) is paid
// for, so the line lies where the tile kernel gains that much.
int gemm_f32_variant(int64_t n_rows, int E, int N, int K, int num_cus)
{
    if (K % MBK != 0) return 1;
    const int64_t tiles = (n_rows / MBM + (E < n_rows ? E : n_rows) / 2) * ceil_div(N, MBN);
    return tiles * 1024 > 8 * (int64_t)num_cus * (K < 1024 ? K : 1024) ? 0 : 1;
}

int gemm_f32_block_m(int variant) { return variant == 0 ? MBM : 32; }

template <int W, bool RELU, bool GROUPED>
static int launch_f32_wave(const GemmParams &p, int64_t m_tiles, hipStream_t s)
{
    constexpr size_t smem = (size_t)W * kF32Ring * 8192;
    auto kern = gemm_f32_wave_kernel<W, RELU, GROUPED>;
    static std::once_flag once;
    static hipError_t setup_rc = hipSuccess;
    std::call_once(once, [&]() {
        setup_rc = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    });
    MOE_HIP_CHECK(setup_rc);
    const int64_t grid = align_up(m_tiles * ceil_div(p.N, 32), 8);
    if (grid > 0x7fffffff) {
        set_error("GEMM grid too large");
        return MOE_ERR_UNSUPPORTED;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(W * 64), smem, s, p);
    MOE_LAUNCH_CHECK("gemm_f32_wave_kernel");
    return MOE_OK;
}

template <bool RELU, bool GROUPED>
static int launch_f32(const GemmParams &p, int variant, int num_cus, hipStream_t s)
{
    const int bm = gemm_f32_block_m(variant);
    const int64_t m_tiles = GROUPED ? (p.max_m_tiles < p.M ? p.max_m_tiles : p.M) : ceil_div(p.M, bm);
    if (m_tiles <= 0 || p.N <= 0) return MOE_OK;
    // few tiles: eight waves share K (16 tokens, 4096 -> 1024: 37 -> 31 us; equal from there down, slower above)
    if (variant != 0)
        return m_tiles * ceil_div(p.N, 32) < 2 * (int64_t)num_cus ? launch_f32_wave<8, RELU, GROUPED>(p, m_tiles, s)
                                                                  : launch_f32_wave<4, RELU, GROUPED>(p, m_tiles, s);
    const int64_t grid = m_tiles * ceil_div(p.N, MBN);
    if (grid > 0x7fffffff) {
        set_error("GEMM grid too large");
        return MOE_ERR_UNSUPPORTED;
    }
    constexpr size_t smem = (size_t)MSTAGES * (MBM + MBN) * MBK * sizeof(float);
    hipLaunchKernelGGL((gemm_f32_tile_kernel<RELU, GROUPED>), dim3((unsigned)grid), dim3(256), smem, s, p);
    MOE_LAUNCH_CHECK("gemm_f32_tile_kernel");
    return MOE_OK;
}

int launch_gemm_f32(const GemmParams &p, bool grouped, int variant, bool relu, int num_cus, hipStream_t s)
{
    if (p.K < 8 || p.K % 8 != 0 || p.lda % 4 != 0 || p.ldb % 4 != 0 || p.strideB % 4 != 0 ||
        reinterpret_cast<uintptr_t>(p.A) % 16 != 0 || reinterpret_cast<uintptr_t>(p.B) % 16 != 0) {
        set_error("fp32 GEMM: K = %d must be a multiple of 8 and the operand rows 16-byte aligned", p.K);
        return MOE_ERR_UNSUPPORTED;
    }
    if (!grouped) variant = gemm_f32_variant(p.M, 0, p.N, p.K, num_cus);
    if (grouped) return relu ? launch_f32<true, true>(p, variant, num_cus, s) : launch_f32<false, true>(p, variant, num_cus, s);
    return relu ? launch_f32<true, false>(p, variant, num_cus, s) : launch_f32<false, false>(p, variant, num_cus, s);
}

}  // namespace moe355
