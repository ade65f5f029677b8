// Gate GEMM with the routing decision in its epilogue: logits = x * Wg^T (+ offset) on bf16 MFMAs, and,
// straight from the accumulators, the softmax / top-k of every token and the per-tile expert histogram.
//
// Paper: the gate is a light linear layer (Sec. 2.4) whose only purpose is the top-1 / top-2 decision
// (Sec. 2.3); dynamic gating then counts the occurrences of each expert (Sec. 5.1).  None of the three
// steps needs the [T,E] logits in memory, so with E <= 128 (one column tile) they never leave the
// registers unless the caller asks for them: the kernel streams x once and writes T*k indices and
// weights -- an HBM-bound stream of x.
//
// Tile: BM = 32 * WAVES token rows x BN = 32 * NI experts (all of them) x 64 along D; every wave owns 32
// rows and ALL columns, as NI blocks of v_mfma_f32_32x32x16_bf16 with the gate weights as first operand:
// lane l then holds, for token row (l & 31), the columns 32 ni + 8 g + 4 (l >> 5) + i in accumulator
// 4 g + i of block ni.  A token's E logits therefore sit in exactly two lanes (l and l ^ 32), 16 * NI
// each, in ascending column order: the k rounds of "largest remaining logit, ties to the lower expert"
// run inside the lane and finish with one exchange between the two.
//
// K pipeline: STAGES LDS stages filled by global_load_lds_dwordx4 (no register staging), STAGES - 1 K
// tiles in flight; rows of 128 B, 16-byte chunk c of row r at chunk slot c ^ ((r >> 1) & 7) (conflict-free
// fragment reads on gfx950's 64-bank LDS), the swizzle applied on the global side of the load.  A block
// is one tile (no persistence: the epilogue is short and there is nothing to keep resident); the tile
// height is chosen so that the launch still has a tile per CU.
// (Measured at T = 65536, D = 2048, E = 128 on MI355X: 50 us when x is partly served by the last-level cache,
// 78 us when every launch reads a different copy of x, about 100 us inside the layer behind the previous
// step's writes.  A bare read of x in the same order -- a CU owning 256 consecutive rows, no arithmetic --
// takes 57 us cold, whatever the bytes per row visit (128 B .. 1 KB) or the depth of the prefetch.  A variant
// that keeps the x rows out of LDS -- each lane loading its own fragments straight into registers four K
// tiles ahead, only the gate weights staged -- measured the same cold and 20 % slower warm, and was dropped.)
#include <mutex>

#include "gemm_bf16_dev.h"
#include "moe_internal.h"

namespace moe355 {

struct GateTopkParams {
    const uint16_t *x;    // [T, K] bf16
    const uint16_t *wg;   // [E, K] bf16
    const float *bias;    // [E] fp32 or NULL
    float *logits;        // [T, E] fp32 or NULL
    int32_t *idx;         // [T, k]
    float *w;             // [T, k]
    int32_t *hist;        // [tiles, E] or NULL: hist[tile, e] = assignments of the tile's tokens to expert e
    int T, E, K, k, renorm;
};

// Where the lane's chunk of K tile kt of row `row` of a tile is, at = that of K tile 0.  Gate and selection in us where K ends inside a
// K tile, a two-stage GEMM, top-k and histogram kernels / this: 3001 tokens, 1000 dimensions, 24 experts 23.9 / 10.4; 1137 tokens, 1496
// dimensions, 47 experts 31.2 / 13.2.
__device__ __forceinline__ const uint16_t *gt_inside(const uint16_t *at, int row, int kt, int K)
{
    const int kc = (threadIdx.x & 7) ^ ((row >> 1) & 7);
    return kt * 64 + kc * 8 < K ? at + kt * 64 : chunk_of_zeros;
}

// RAGGED: K ends inside a K tile.  (An instance of its own: with the question in the K loop whole K tiles cost 3 to 5 % more, 20000 tokens, 2048
// dimensions, 64 experts 21.4 / 21.9 us, 16385 tokens, 1024 dimensions, 16 experts 9.2 / 9.7, 30000 tokens, 2048 dimensions, 96 experts 29.4 / 30.3.)
template <int WAVES, int NI, int STAGES, bool RAGGED>
__global__ __launch_bounds__(WAVES * 64) void gate_topk_kernel(GateTopkParams p)
{
    constexpr int THREADS = WAVES * 64;
    constexpr int BM = 32 * WAVES, BN = 32 * NI, BK = 64;
    constexpr int A_IT = 4;                // 1 KB load instructions per wave and stage: BM / 8 rows-of-8 over WAVES waves
    constexpr int B_IT = NI * 4 / WAVES;   // BN / 8 over WAVES waves
    static_assert((NI * 4) % WAVES == 0, "the gate weight tile must split evenly over the waves");
    static_assert(STAGES >= 2 && STAGES <= 4, "two to four LDS stages");
    constexpr int LPS = A_IT + B_IT;
    constexpr int NS = NI * 16;            // logits a lane holds
    static_assert(NS <= 64, "the taken-mask is 64 bits");

    extern __shared__ __attribute__((aligned(1024))) uint8_t gt_smem[];
    uint16_t *sA = reinterpret_cast<uint16_t *>(gt_smem);  // [STAGES][BM * 64]
    uint16_t *sB = sA + STAGES * BM * BK;                   // [STAGES][BN * 64]

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int row0 = blockIdx.x * BM;
    const int K = p.K, T = p.T, E = p.E;
    const int KT = (K + BK - 1) / BK;

    // ---- global -> LDS: instruction i of wave w fills tile rows (w * IT + i) * 8 .. + 7; lane L lands in row
    // (L >> 3), chunk slot (L & 7) and fetches K chunk (L & 7) ^ ((row >> 1) & 7).  Rows past the end of x or
    // Wg repeat the last one (their results are never used).
    const uint16_t *a_ptr[A_IT];
    const uint16_t *b_ptr[B_IT];
#pragma unroll
    for (int i = 0; i < A_IT; ++i) {
        const int r = (wave * A_IT + i) * 8 + (lane >> 3);
        const int kc = (lane & 7) ^ ((r >> 1) & 7);
        const int gr = min(row0 + r, T - 1);
        a_ptr[i] = p.x + (int64_t)gr * K + kc * 8;
    }
#pragma unroll
    for (int i = 0; i < B_IT; ++i) {
        const int r = (wave * B_IT + i) * 8 + (lane >> 3);
        const int kc = (lane & 7) ^ ((r >> 1) & 7);
        const int gn = min(r, E - 1);
        b_ptr[i] = p.wg + (int64_t)gn * K + kc * 8;
    }
    auto issue = [&](int kt, int buf) {
        if (RAGGED && (kt + 1) * BK > K) {  // uniform: K ends inside this K tile
#pragma unroll
            for (int i = 0; i < A_IT; ++i) {
                const int r = (wave * A_IT + i) * 8;
                __builtin_amdgcn_global_load_lds((const glb_void *)gt_inside(a_ptr[i], r + (lane >> 3), kt, K),
                                                 (lds_void *)(sA + buf * BM * BK + r * BK), 16, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < B_IT; ++i) {
                const int r = (wave * B_IT + i) * 8;
                __builtin_amdgcn_global_load_lds((const glb_void *)gt_inside(b_ptr[i], r + (lane >> 3), kt, K),
                                                 (lds_void *)(sB + buf * BN * BK + r * BK), 16, 0, 0);
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < A_IT; ++i)
            __builtin_amdgcn_global_load_lds((const glb_void *)(a_ptr[i] + kt * BK),
                                             (lds_void *)(sA + buf * BM * BK + (wave * A_IT + i) * 8 * BK), 16, 0, 0);
#pragma unroll
        for (int i = 0; i < B_IT; ++i)
            __builtin_amdgcn_global_load_lds((const glb_void *)(b_ptr[i] + kt * BK),
                                             (lds_void *)(sB + buf * BN * BK + (wave * B_IT + i) * 8 * BK), 16, 0, 0);
    };
    // "at most STAGES - 2 stages' loads of this wave outstanding": the K tile needed next has landed.  Every
    // iteration issues the same number of loads (past the end it re-reads the last K tile into a stage nobody
    // reads any more), which keeps this arithmetic fixed.
    constexpr int WAITN = (STAGES - 2) * LPS;
    static_assert(WAITN < 64, "vmcnt is a 6-bit counter");
    auto wait_loads = [&]() {
        constexpr int kWaitImm = (WAITN & 15) | ((WAITN >> 4) << 14) | (7 << 4) | (15 << 8);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(kWaitImm);
        asm volatile("" ::: "memory");
    };
    auto block_barrier = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    f32x16 acc[NI];
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[ni][r] = 0.f;

    const int frag_row = lane & 31;
    const int half = lane >> 5;
    const int swz = (lane >> 1) & 7;  // == (row >> 1) & 7 for every tile row this lane reads

#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s) issue(min(s, KT - 1), s);
    int cur = 0, nxt = STAGES - 1;
    for (int kt = 0; kt < KT; ++kt) {
        wait_loads();
        block_barrier();  // stage `cur` is complete for every wave; everybody is done reading stage `nxt`
        issue(min(kt + STAGES - 1, KT - 1), nxt);
        const uint16_t *cA = sA + cur * BM * BK + (wave * 32 + frag_row) * BK;
        const uint16_t *cB = sB + cur * BN * BK + frag_row * BK;
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            const int chunkpos = ((ks * 2 + half) ^ swz) << 3;
            const bf16x8 af = *reinterpret_cast<const bf16x8 *>(cA + chunkpos);
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                const bf16x8 bf = *reinterpret_cast<const bf16x8 *>(cB + ni * 32 * BK + chunkpos);
                acc[ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf, af, acc[ni], 0, 0, 0);
            }
        }
        cur = (cur + 1 == STAGES) ? 0 : cur + 1;
        nxt = (nxt + 1 == STAGES) ? 0 : nxt + 1;
    }
    // no load may still be writing LDS when the histogram reuses it
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    block_barrier();

    // ---- epilogue: this lane's logits in ascending column order
    const int row = row0 + wave * 32 + frag_row;
    const bool live = row < T;
    auto col_of = [&](int s) { return (s >> 4) * 32 + ((s >> 2) & 3) * 8 + 4 * half + (s & 3); };
    float v[NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) v[s] = acc[s >> 4][s & 15];
    if (p.bias) {  // uniform over the grid.  All offsets are requested before the first is added (columns past E read
                   // the last one): a load per column behind its own predicate makes 16 * NI dependent memory latencies
        float off[NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) off[s] = p.bias[min(col_of(s), E - 1)];
#pragma unroll
        for (int s = 0; s < NS; ++s) v[s] += off[s];
    }
    if (p.logits && live) {
        float *dst = p.logits + (int64_t)row * E;
        if ((E & 3) == 0) {
#pragma unroll
            for (int q = 0; q < NS / 4; ++q) {
                const int c = col_of(4 * q);
                if (c < E) *reinterpret_cast<float4 *>(dst + c) = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
            }
        } else {
#pragma unroll
            for (int s = 0; s < NS; ++s)
                if (col_of(s) < E) dst[col_of(s)] = v[s];
        }
    }

    const float NEG_INF = -__builtin_huge_valf();
    constexpr int NONE = 0x7fffffff;
    uint64_t taken = 0;  // bit s: slot s already selected, or past the last expert
#pragma unroll
    for (int s = 0; s < NS; ++s)
        if (col_of(s) >= E) taken |= 1ull << s;

    float sel_v[MOE_MAX_K];
    int sel_e[MOE_MAX_K];
#pragma unroll
    for (int j = 0; j < MOE_MAX_K; ++j) {
        sel_v[j] = NEG_INF;
        sel_e[j] = 0;
        if (j >= p.k) continue;  // uniform over the grid
        float bv = NEG_INF;
        int bs = -1;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const bool free_slot = !((taken >> s) & 1ull);
            if (free_slot && (bs < 0 || v[s] > bv)) {  // strict: the first (lowest) column keeps a tie
                bv = v[s];
                bs = s;
            }
        }
        int be = bs >= 0 ? col_of(bs) : NONE;
        // the other half of the row: (value desc, column asc) decides
        const float ov = __shfl_xor(bv, 32, 64);
        const int oe = __shfl_xor(be, 32, 64);
        if (oe != NONE && (be == NONE || ov > bv || (ov == bv && oe < be))) {
            bv = ov;
            be = oe;
        }
        // both lanes agree for finite inputs; take the lower lane's view so that the bookkeeping stays
        // consistent whatever the inputs are
        bv = __shfl(bv, frag_row, 64);
        be = __shfl(be, frag_row, 64);
        sel_v[j] = bv;
        sel_e[j] = be == NONE ? 0 : be;
        if (be != NONE && ((be >> 2) & 1) == half) {  // the column lives in this lane: mark its slot
            const int s_own = (be >> 5) * 16 + ((be >> 3) & 3) * 4 + (be & 3);
            taken |= 1ull << s_own;
        }
    }

    // gate weights in fp32: exp(l - max) over the selected (renormalised) or over all experts
    const float m = sel_v[0];
    float denom = 0.f;
    if (p.renorm) {
#pragma unroll
        for (int j = 0; j < MOE_MAX_K; ++j)
            if (j < p.k) denom += expf(sel_v[j] - m);
    } else {
        float part = 0.f;
#pragma unroll
        for (int s = 0; s < NS; ++s)
            if (col_of(s) < E) part += expf(v[s] - m);
        denom = part + __shfl_xor(part, 32, 64);
    }
    if (live && half == 0) {
#pragma unroll
        for (int j = 0; j < MOE_MAX_K; ++j) {
            if (j < p.k) {
                p.idx[(int64_t)row * p.k + j] = sel_e[j];
                p.w[(int64_t)row * p.k + j] = expf(sel_v[j] - m) / denom;
            }
        }
    }

    // ---- the tile's expert histogram (LDS atomics on integers: the sums do not depend on the order)
    if (p.hist) {
        int *hist = reinterpret_cast<int *>(gt_smem);
        for (int e = tid; e < E; e += THREADS) hist[e] = 0;
        __syncthreads();
        if (live && half == 0) {
#pragma unroll
            for (int j = 0; j < MOE_MAX_K; ++j)
                if (j < p.k) atomicAdd(&hist[sel_e[j]], 1);
        }
        __syncthreads();
        for (int e = tid; e < E; e += THREADS) p.hist[(int64_t)blockIdx.x * E + e] = hist[e];
    }
}

// The same for batches with at most one short tile (32, 64 or 128 rows) per CU, whose time is the latency of the K loop and of the
// selection.  With one wave for 32 rows and all columns a K tile takes 1 us: 20 loads and 16 MFMAs of a wave, one after the other.
// Here the column blocks have waves of their own (RG x NI waves of one 32x32 block), which share a K tile's loads; a wave reads a K
// tile's fragments at once.  A logit is the same sum in the same order.  Then the logits cross LDS and G lanes share a token.
// us, launches on the same inputs, a wave per 32 rows / this, 2048 dimensions, 128 experts: 512 tokens 29.9 / 11.9, 4096 30.0 / 12.5, 8192 30.3 / 13.8,
// 12000 30.9 / 17.3, 16384 28.5 / 19.7, 20000 35.9 / 23.2; 1024 dimensions, 64 experts: 8192 tokens 12.9 / 8.5; 96 experts, 4096 tokens 17.1 / 9.5;
// 512 dimensions, 64 experts, 16384 tokens 9.7 / 7.8; 2048 dimensions, 16 experts, 8192 tokens 12.9 / 10.7.
template <int RG, int NI, int STAGES, bool RAGGED>
__global__ __launch_bounds__(RG *NI * 64) void gate_topk_wide_kernel(GateTopkParams p)
{
    constexpr int W = RG * NI, THREADS = W * 64, BM = 32 * RG, BK = 64;
    constexpr int STAGE = (RG + NI) * 32 * BK;            // one stage in bf16: the rows, then the gate weights
    constexpr int LOADS = 4 * (RG + NI), LPS = (LOADS + W - 1) / W;  // of 1 KB, and of a wave (the last one again where they do not come out)
    constexpr int WAITN = (STAGES - 2) * LPS;
    static_assert(STAGES >= 3 && WAITN < 64, "vmcnt is a 6-bit counter");
    constexpr int G = NI == 1 ? 2 : NI == 4 ? 8 : 4, V = NI * 32 / G;  // lanes of a token, columns of a lane
    constexpr int LD = NI * 32 + 4;                                    // floats per row of logits in LDS
    static_assert(BM * LD * 4 <= STAGES * STAGE * 2, "the logits fit where the stages were");

    extern __shared__ __attribute__((aligned(1024))) uint8_t gt_smem[];
    uint16_t *stages = reinterpret_cast<uint16_t *>(gt_smem);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), rg = wave / NI, ni = wave % NI;
    const int row0 = blockIdx.x * BM;
    const int K = p.K, T = p.T, E = p.E, KT = (K + BK - 1) / BK;

    // load i of the wave fills 8 rows of 128 bytes; layout, swizzle and the rows past the end as in the kernel above
    const uint16_t *src[LPS];
    int dst[LPS];
#pragma unroll
    for (int i = 0; i < LPS; ++i) {
        const int ld = min(wave + i * W, LOADS - 1), r = ld * 8 + (lane >> 3);
        const int kc = (lane & 7) ^ ((r >> 1) & 7);
        dst[i] = ld * 8 * BK;
        src[i] = ld < 4 * RG ? p.x + (int64_t)min(row0 + r, T - 1) * K + kc * 8 : p.wg + (int64_t)min(r - BM, E - 1) * K + kc * 8;
    }
    auto issue = [&](int kt, int stage) {
        if (RAGGED && (kt + 1) * BK > K) {  // uniform: K ends inside this K tile
#pragma unroll
            for (int i = 0; i < LPS; ++i)
                __builtin_amdgcn_global_load_lds((const glb_void *)gt_inside(src[i], min(wave + i * W, LOADS - 1) * 8 + (lane >> 3), kt, K),
                                                 (lds_void *)(stages + stage * STAGE + dst[i]), 16, 0, 0);
            return;
        }
#pragma unroll
        for (int i = 0; i < LPS; ++i)
            __builtin_amdgcn_global_load_lds((const glb_void *)(src[i] + kt * BK), (lds_void *)(stages + stage * STAGE + dst[i]), 16, 0, 0);
    };
    auto block_barrier = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    const int frag_row = lane & 31, half = lane >> 5, swz = (lane >> 1) & 7;
#pragma unroll 1
    for (int s = 0; s < STAGES - 1; ++s) issue(min(s, KT - 1), s);
    int cur = 0, nxt = STAGES - 1;
    for (int kt = 0; kt < KT; ++kt) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt((WAITN & 15) | ((WAITN >> 4) << 14) | (7 << 4) | (15 << 8));
        asm volatile("" ::: "memory");
        block_barrier();  // stage `cur` is complete for every wave; everybody is done reading stage `nxt`
        const uint16_t *cA = stages + cur * STAGE + (rg * 32 + frag_row) * BK, *cB = stages + cur * STAGE + (BM + ni * 32 + frag_row) * BK;
        bf16x8 af[BK / 16], bf[BK / 16];  // all reads first: one LDS latency per K tile
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            const int chunkpos = ((ks * 2 + half) ^ swz) << 3;
            bf[ks] = *reinterpret_cast<const bf16x8 *>(cB + chunkpos);
            af[ks] = *reinterpret_cast<const bf16x8 *>(cA + chunkpos);
        }
        __builtin_amdgcn_sched_barrier(0);
        issue(min(kt + STAGES - 1, KT - 1), nxt);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[ks], af[ks], acc, 0, 0, 0);
        cur = (cur + 1 == STAGES) ? 0 : cur + 1;
        nxt = (nxt + 1 == STAGES) ? 0 : nxt + 1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no load may still be writing LDS
    __syncthreads();

    // ---- the logits: lane -> row frag_row, columns 8 g + 4 half + i of the wave's block
    float *logits = reinterpret_cast<float *>(gt_smem);
#pragma unroll
    for (int g = 0; g < 4; ++g)
        *reinterpret_cast<float4 *>(logits + (rg * 32 + frag_row) * LD + ni * 32 + 8 * g + 4 * half) =
            make_float4(acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]);
    __syncthreads();
    const int sub = tid % G, token = tid / G;  // of the tile
    const bool mine = token < BM;              // whole waves
    const int row = row0 + token;
    const bool live = mine && row < T;
    auto col_of = [&](int s) { return (s >> 2) * (4 * G) + 4 * sub + (s & 3); };  // ascending with s
    int sel_e[MOE_MAX_K];
    if (mine) {
        float v[V];
#pragma unroll
        for (int q = 0; q < V / 4; ++q) {
            const float4 f = *reinterpret_cast<const float4 *>(logits + token * LD + col_of(4 * q));
            v[4 * q] = f.x, v[4 * q + 1] = f.y, v[4 * q + 2] = f.z, v[4 * q + 3] = f.w;
        }
        if (p.bias) {
            float off[V];
#pragma unroll
            for (int s = 0; s < V; ++s) off[s] = p.bias[min(col_of(s), E - 1)];
#pragma unroll
            for (int s = 0; s < V; ++s) v[s] += off[s];
        }
        if (p.logits && live) {
            float *out = p.logits + (int64_t)row * E;
#pragma unroll
            for (int q = 0; q < V / 4; ++q) {
                const int c = col_of(4 * q);
                if ((E & 3) == 0) {
                    if (c < E) *reinterpret_cast<float4 *>(out + c) = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        if (c + i < E) out[c + i] = v[4 * q + i];
                }
            }
        }
        const float NEG_INF = -__builtin_huge_valf();
        constexpr int NONE = 0x7fffffff;
        uint32_t taken = 0;  // bit s: slot s already selected, or past the last expert
#pragma unroll
        for (int s = 0; s < V; ++s)
            if (col_of(s) >= E) taken |= 1u << s;
        float sel_v[MOE_MAX_K];
#pragma unroll
        for (int j = 0; j < MOE_MAX_K; ++j) {
            sel_v[j] = NEG_INF;
            sel_e[j] = 0;
            if (j >= p.k) continue;  // uniform over the grid
            float bv = NEG_INF;
            int be = NONE;
#pragma unroll
            for (int s = 0; s < V; ++s)
                if (!((taken >> s) & 1u) && (be == NONE || v[s] > bv)) {  // strict: the first (lowest) column keeps a tie
                    bv = v[s];
                    be = col_of(s);
                }
#pragma unroll
            for (int off = G / 2; off >= 1; off >>= 1) {
                const float ov = __shfl_xor(bv, off, 64);
                const int oe = __shfl_xor(be, off, 64);
                if (oe != NONE && (be == NONE || ov > bv || (ov == bv && oe < be))) {
                    bv = ov;
                    be = oe;
                }
            }
            // the lanes agree for finite inputs; the first one's view keeps the bookkeeping consistent whatever the inputs are
            bv = __shfl(bv, lane - sub, 64);
            be = __shfl(be, lane - sub, 64);
            sel_v[j] = bv;
            sel_e[j] = be == NONE ? 0 : be;
            if (be != NONE && (be >> 2) % G == sub) taken |= 1u << (be / (4 * G) * 4 + (be & 3));
        }
        const float m = sel_v[0];
        float denom = 0.f;
        if (p.renorm) {
#pragma unroll
            for (int j = 0; j < MOE_MAX_K; ++j)
                if (j < p.k) denom += expf(sel_v[j] - m);
        } else {
#pragma unroll
            for (int s = 0; s < V; ++s)
                if (col_of(s) < E) denom += expf(v[s] - m);
#pragma unroll
            for (int off = G / 2; off >= 1; off >>= 1) denom += __shfl_xor(denom, off, 64);
        }
        if (live && sub == 0) {
#pragma unroll
            for (int j = 0; j < MOE_MAX_K; ++j) {
                if (j < p.k) {
                    p.idx[(int64_t)row * p.k + j] = sel_e[j];
                    p.w[(int64_t)row * p.k + j] = expf(sel_v[j] - m) / denom;
                }
            }
        }
    }
    if (p.hist) {
        int *hist = reinterpret_cast<int *>(gt_smem) + BM * LD;  // behind the logits, which a wave may still read
        for (int e = tid; e < E; e += THREADS) hist[e] = 0;
        __syncthreads();
        if (live && sub == 0) {
#pragma unroll
            for (int j = 0; j < MOE_MAX_K; ++j)
                if (j < p.k) atomicAdd(&hist[sel_e[j]], 1);
        }
        __syncthreads();
        for (int e = tid; e < E; e += THREADS) p.hist[(int64_t)blockIdx.x * E + e] = hist[e];
    }
}

template <int RG, int NI, int STAGES, bool RAGGED>
static int launch_gate_topk_wide_k(const GateTopkParams &p, hipStream_t s)
{
    const size_t smem = (size_t)STAGES * (RG + NI) * 32 * 64 * sizeof(uint16_t);
    static_assert((size_t)STAGES * (RG + NI) * 4096 >= 32u * RG * (NI * 32 + 4) * 4 + 128 * 4, "logits and histogram reuse the stages");
    auto kern = gate_topk_wide_kernel<RG, NI, STAGES, RAGGED>;
    static std::once_flag once;  // per instantiation
    static hipError_t attr_rc = hipSuccess;
    std::call_once(once, [&]() {
        attr_rc = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    });
    MOE_HIP_CHECK(attr_rc);
    ProfScope ps("gate_topk", s);
    hipLaunchKernelGGL(kern, dim3((unsigned)ceil_div(p.T, 32 * RG)), dim3(RG * NI * 64), smem, s, p);
    MOE_LAUNCH_CHECK("gate_topk_wide_kernel");
    return MOE_OK;
}

template <int RG, int NI, int STAGES>
static int launch_gate_topk_wide(const GateTopkParams &p, hipStream_t s)
{
    // four waves of 32 rows and 128 columns: as scheduled here the loop with the question in it is the faster one (4096 tokens, 128 experts,
    // without / with: 1024 dimensions 9.5 / 9.2 us, 4096 dimensions 21.1 / 19.8)
    if constexpr (RG == 1 && NI == 4) return launch_gate_topk_wide_k<RG, NI, STAGES, true>(p, s);
    return p.K % 64 != 0 ? launch_gate_topk_wide_k<RG, NI, STAGES, true>(p, s) : launch_gate_topk_wide_k<RG, NI, STAGES, false>(p, s);
}

template <int WAVES, int NI, int STAGES, bool RAGGED>
static int launch_gate_topk_k(const GateTopkParams &p, hipStream_t s)
{
    constexpr int BM = 32 * WAVES, BN = 32 * NI;
    const size_t smem = (size_t)STAGES * (BM + BN) * 64 * sizeof(uint16_t);
    auto kern = gate_topk_kernel<WAVES, NI, STAGES, RAGGED>;
    static std::once_flag once;  // per instantiation
    static hipError_t attr_rc = hipSuccess;
    std::call_once(once, [&]() {
        attr_rc = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                      (int)smem);
    });
    MOE_HIP_CHECK(attr_rc);
    ProfScope ps("gate_topk", s);
    hipLaunchKernelGGL(kern, dim3((unsigned)ceil_div(p.T, BM)), dim3(WAVES * 64), smem, s, p);
    MOE_LAUNCH_CHECK("gate_topk_kernel");
    return MOE_OK;
}

template <int WAVES, int NI, int STAGES>
static int launch_gate_topk_t(const GateTopkParams &p, hipStream_t s)
{
    return p.K % 64 != 0 ? launch_gate_topk_k<WAVES, NI, STAGES, true>(p, s) : launch_gate_topk_k<WAVES, NI, STAGES, false>(p, s);
}

bool gate_topk_fused_ok(int dtype, int T, int E, int K)
{
    return dtype == MOE_DTYPE_BF16 && T > 0 && E >= 1 && E <= 128 && K >= 64 && K % 8 == 0;
}

// Groups of 32 rows in a tile of gate_topk_wide_kernel's, 0: not for this kernel
static int gate_topk_wide(int T, int E, int K, int num_cus)
{
    // One column block and a short K loop: the selection by two lanes a token costs more than the loop gains.  us, a wave per 32 rows / this: 4096
    // tokens, 32 experts, 64 dimensions 4.8 / 5.6, 256 5.5 / 6.1, 512 6.5 / 6.7, 768 7.5 / 7.3; 16 experts, 256 dimensions 5.5 / 5.8, 512 6.5 /
    // 6.5; 12000 tokens, 32 experts, 64 dimensions 5.0 / 5.4, 256 5.8 / 5.9
    if (E <= 32 && K <= (T <= 32 * num_cus ? 512 : 256)) return 0;
    // 128 rows: 20000 tokens, 2048 dimensions, 128 experts 35.9 / 23.2 us, 24576 36.6 / 25.8; with 64 experts and fewer they are no faster
    return T <= 32 * num_cus ? 1 : T <= 64 * num_cus ? 2 : T <= 96 * num_cus && E > 64 ? 4 : 0;
}

// Tokens per tile (= tokens per histogram row) the fused kernel uses for T tokens, E experts and K dimensions: the wide kernel's where it
// runs, else the tallest of 256, 128, 64, 32 rows that still gives every CU a tile and whose wave count divides the weight
// tile's load instructions (32 rows: only where the wide kernel leaves small batches to it).
int gate_topk_tile_tokens(int T, int E, int K, int num_cus)
{
    const int ni = ceil_div(E, 32);
    if (gate_topk_wide(T, E, K, num_cus)) return 32 * gate_topk_wide(T, E, K, num_cus);
    for (int waves = 8; waves > 1; waves >>= 1) {
        if ((ni * 4) % waves != 0) continue;
        if (ceil_div(T, 32 * waves) >= num_cus) return 32 * waves;
    }
    return 32;
}

int launch_gate_topk(const void *x, const void *wg, const float *gate_bias, int T, int E, int K, int k, int renorm,
                     float *logits, int32_t *idx, float *w, int32_t *hist, int num_cus, hipStream_t s)
{
    GateTopkParams p;
    p.x = static_cast<const uint16_t *>(x);
    p.wg = static_cast<const uint16_t *>(wg);
    p.bias = gate_bias;
    p.logits = logits;
    p.idx = idx;
    p.w = w;
    p.hist = hist;
    p.T = T;
    p.E = E;
    p.K = K;
    p.k = k;
    p.renorm = renorm;
    const int ni = ceil_div(E, 32);
    const int waves = gate_topk_tile_tokens(T, E, K, num_cus) / 32;
    // stages: more of them make the start longer and the loop no shorter (4096 tokens over 128 experts, 4 / 8: 13.5 / 14.2 us; 64 rows, 3 / 6: 22.1 / 20.9)
    if (const int rg = gate_topk_wide(T, E, K, num_cus)) {
        switch (rg * 10 + ni) {
        case 11: return launch_gate_topk_wide<1, 1, 9>(p, s);
        case 12: return launch_gate_topk_wide<1, 2, 6>(p, s);
        case 13: return launch_gate_topk_wide<1, 3, 5>(p, s);
        case 14: return launch_gate_topk_wide<1, 4, 4>(p, s);
        case 21: return launch_gate_topk_wide<2, 1, 6>(p, s);
        case 22: return launch_gate_topk_wide<2, 2, 5>(p, s);
        case 23: return launch_gate_topk_wide<2, 3, 5>(p, s);
        case 24: return launch_gate_topk_wide<2, 4, 6>(p, s);
        case 43: return launch_gate_topk_wide<4, 3, 5>(p, s);
        case 44: return launch_gate_topk_wide<4, 4, 5>(p, s);
        default: break;
        }
    }
#define MOE_GT(W, N, S) return launch_gate_topk_t<W, N, S>(p, s)
    switch (waves * 10 + ni) {
    case 84: MOE_GT(8, 4, 3);
    case 82: MOE_GT(8, 2, 3);
    case 44: MOE_GT(4, 4, 3);
    case 43: MOE_GT(4, 3, 3);
    case 42: MOE_GT(4, 2, 3);
    case 41: MOE_GT(4, 1, 3);
    case 24: MOE_GT(2, 4, 3);
    case 23: MOE_GT(2, 3, 3);
    case 22: MOE_GT(2, 2, 3);
    case 21: MOE_GT(2, 1, 3);
    case 11: MOE_GT(1, 1, 4);
    default: break;
    }
#undef MOE_GT
    set_error("gate_topk: no kernel for %d waves and %d column blocks", waves, ni);
    return MOE_ERR_UNSUPPORTED;
}

}  // namespace moe355
