// Routing kernels: softmax + top-k over the gate logits, per-expert counts with a prefix
// scan, the stable permutation of the assignments, and the M-tile map of the grouped GEMM.
//
// Paper: top-1 / top-2 gating (Sec. 2.3); dynamic gating sorts the expert assignments and counts
// the occurrences of each expert (Sec. 5.1).  The sort here is a counting sort: its result is the
// stable argsort (ascending token inside each expert) and costs O(N) instead of O(N log N).
// Nothing uses atomics on global memory, so the permutation is the same on every run.
#include <type_traits>

#include "moe_internal.h"
#include "ring_schedule.h"

namespace moe355 {

static constexpr int kThreads = 256;
static constexpr int kWave = 64;
static constexpr int kMaxLogitParts = 16;  // slices the top-k kernel can add up (the gate GEMM's split K)

typedef __attribute__((ext_vector_type(4))) float f32x4_t;

// A word (one or four logits) that arrives as n_parts partial sums (the gate GEMM's split K), slice 0 at `at`, slice i > 0 at parts +
// (i - 1) * part_stride: added in slice order, the sum is also written back to `at`.  What bounds it is the latency of a slice another
// XCD wrote, so all slices are requested before the first is added.
template <typename W>
__device__ __forceinline__ W add_slices(float *at, int n_parts, const float *parts, int64_t part_stride)
{
    W f = *reinterpret_cast<const W *>(at);
    if (n_parts > 1) {  // uniform over the grid
        W g[kMaxLogitParts - 1];
#pragma unroll
        for (int sp = 1; sp < kMaxLogitParts; ++sp) g[sp - 1] = sp < n_parts ? *reinterpret_cast<const W *>(parts + (sp - 1) * part_stride) : W{};
#pragma unroll
        for (int sp = 1; sp < kMaxLogitParts; ++sp)
            if (sp < n_parts) f += g[sp - 1];
        *reinterpret_cast<W *>(at) = f;
    }
    return f;
}

// n logits (whole rows) to LDS, by the whole block, a word per thread and round.  VEC: n, the slices' distance and the pointers allow
// 16-byte accesses.
template <bool VEC>
__device__ __forceinline__ void stage_logits(float *__restrict__ s_row, float *logits, int n, int n_parts, const float *parts,
                                             int64_t part_stride)
{
    typedef std::conditional_t<VEC, f32x4_t, float> W;
    constexpr int N = sizeof(W) / sizeof(float);
    for (int i = threadIdx.x * N; i < n; i += blockDim.x * N)
        *reinterpret_cast<W *>(s_row + i) = add_slices<W>(logits + i, n_parts, parts + i, part_stride);
}

// ------------------------------------------------------------------------------------------------
// softmax + top-k.  G lanes (a power of two <= 64) share one token; lane `sub` holds logits
// sub, sub+G, sub+2G, ...  Each of the k rounds takes the largest remaining logit; equal logits
// go to the lower expert index (inside a lane indices ascend with the register slot, across
// lanes the butterfly compares (value, index)).
// ------------------------------------------------------------------------------------------------
// VEC: lane `sub` instead holds the 16-byte groups sub, sub+G, ... of the row (4 logits each, E a
// multiple of 4), so every lane has V/4 float4 loads in flight; slot i of the lane is expert
// (i/4)*4G + 4*sub + i%4, still ascending with i.
// One token per group of G lanes: token t, lane sub of the group, its logits at `row`.  s_idx (may be NULL): the selection goes
// there too.  SLICES: the lane adds the slices of its words itself; parts: the token's.
template <int G, int V, bool VEC, bool SLICES = false>
__device__ __forceinline__ void topk_token(int t, bool live, int sub, std::conditional_t<SLICES, float, const float> *row, int E, int k,
                                           int renorm, int32_t *__restrict__ idx, float *__restrict__ w, int *s_idx, int n_parts = 1,
                                           const float *__restrict__ parts = nullptr, int64_t part_stride = 0)
{
    const float NEG_INF = -__builtin_huge_valf();
    auto expert_of = [&](int i) { return VEC ? (i >> 2) * (4 * G) + 4 * sub + (i & 3) : sub + i * G; };

    float v[V];
    if (VEC) {
#pragma unroll
        for (int q = 0; q < V / 4; ++q) {
            const int e0 = (q * G + sub) * 4;
            f32x4_t f = {NEG_INF, NEG_INF, NEG_INF, NEG_INF};
            if (live && e0 < E) {
                if constexpr (SLICES)
                    f = add_slices<f32x4_t>(row + e0, n_parts, parts + e0, part_stride);
                else
                    f = *reinterpret_cast<const f32x4_t *>(row + e0);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) v[(4 * q + i) % V] = f[i];
        }
    } else {
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const int e = sub + i * G;
            v[i] = NEG_INF;
            if (live && e < E) {
                if constexpr (SLICES)
                    v[i] = add_slices<float>(row + e, n_parts, parts + e, part_stride);
                else
                    v[i] = row[e];
            }
        }
    }
    uint32_t taken = 0;  // bit i: register slot i already selected (or beyond E)
#pragma unroll
    for (int i = 0; i < V; ++i)
        if (expert_of(i) >= E) taken |= 1u << i;

    float sel_v[MOE_MAX_K];
    int sel_e[MOE_MAX_K];
#pragma unroll
    for (int j = 0; j < MOE_MAX_K; ++j) {
        sel_v[j] = NEG_INF;
        sel_e[j] = 0;
        if (j >= k) continue;  // uniform over the block
        float bv = NEG_INF;
        int be = 0x7fffffff;  // "none"
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const bool free_slot = !((taken >> i) & 1u);
            if (free_slot && (be == 0x7fffffff || v[i] > bv)) {
                bv = v[i];
                be = expert_of(i);
            }
        }
#pragma unroll
        for (int off = G / 2; off >= 1; off >>= 1) {
            const float ov = __shfl_xor(bv, off, kWave);
            const int oe = __shfl_xor(be, off, kWave);
            const bool other_wins = (oe != 0x7fffffff) && (be == 0x7fffffff || ov > bv || (ov == bv && oe < be));
            if (other_wins) {
                bv = ov;
                be = oe;
            }
        }
        // every lane of the group agrees for finite inputs; take lane 0's view so that the
        // "taken" bookkeeping stays consistent whatever the inputs are
        const int base = (threadIdx.x % kWave) - sub;
        bv = __shfl(bv, base, kWave);
        be = __shfl(be, base, kWave);
        sel_v[j] = bv;
        sel_e[j] = be;
        if (be != 0x7fffffff) {
            const int owner = VEC ? (be % (4 * G)) >> 2 : be % G;
            const int slot = VEC ? (be / (4 * G)) * 4 + (be & 3) : be / G;
            if (owner == sub) taken |= 1u << slot;
        }
    }

    // gate weights in fp32: exp(l - max) over the selected (renorm) or over all experts
    const float m = sel_v[0];
    float denom = 0.f;
    if (renorm) {
#pragma unroll
        for (int j = 0; j < MOE_MAX_K; ++j)
            if (j < k) denom += expf(sel_v[j] - m);
    } else {
        float part = 0.f;
#pragma unroll
        for (int i = 0; i < V; ++i)
            if (expert_of(i) < E) part += expf(v[i] - m);
#pragma unroll
        for (int off = G / 2; off >= 1; off >>= 1) part += __shfl_xor(part, off, kWave);
        denom = part;
    }
    if (live && sub == 0) {
#pragma unroll
        for (int j = 0; j < MOE_MAX_K; ++j) {
            if (j < k) {
                idx[(int64_t)t * k + j] = sel_e[j];
                if (s_idx) s_idx[t * k + j] = sel_e[j];
                w[(int64_t)t * k + j] = expf(sel_v[j] - m) / denom;
            }
        }
    }
}

// Where the logits are the gate GEMM's slices, who adds them: all threads into LDS, or the lanes of the selection.
// Staged, the slices of a word are one thread's; the lanes have the loads of all their words under way at once, and no barrier.
// Gate and top-k in us, lanes / staged: 200 tokens, 127 experts, 4 slices 9.2 / 9.7, 8 slices 9.7 / 10.1, 16 slices 11.8 / 10.7; 250 experts 10.6 / 11.1,
// 11.5 / 11.9, 14.5 / 13.7 (one token 21.7 / 21.1 a layer call); 32 experts 7.6 / 7.9, 7.9 / 8.2, 8.2 / 8.4; 256 experts 11.8 / 11.7, 12.9 / 12.7, 15.2 / 14.7.
enum { PARTS_NONE, PARTS_LANES, PARTS_STAGED };
template <int G, int V, bool VEC>
static bool topk_stages(int T, int n_parts) { return n_parts > 8 || (VEC && V >= 8) || T <= 2; }

template <int G, int V, bool VEC, int PARTS>
__global__ __launch_bounds__(kThreads) void topk_kernel(float *logits, int T, int E, int k, int renorm,
                                                        int32_t *__restrict__ idx, float *__restrict__ w,
                                                        int n_parts, const float *__restrict__ parts,
                                                        int64_t part_stride)
{
    constexpr int TPB = kThreads / G;
    const int t0 = blockIdx.x * TPB, local = threadIdx.x / G, t = t0 + local;
    if constexpr (PARTS == PARTS_STAGED) {
        __shared__ __align__(16) float s_logits[TPB * G * V];
        const int64_t at = (int64_t)t0 * E;
        stage_logits<VEC>(s_logits, logits + at, min(TPB, T - t0) * E, n_parts, parts + at, part_stride);
        __syncthreads();
        topk_token<G, V, VEC>(t, t < T, threadIdx.x % G, s_logits + local * E, E, k, renorm, idx, w, nullptr);
    } else if constexpr (PARTS == PARTS_LANES) {
        const int64_t at = (int64_t)t * E;
        topk_token<G, V, VEC, true>(t, t < T, threadIdx.x % G, logits + at, E, k, renorm, idx, w, nullptr, n_parts, parts + at, part_stride);
    } else {
        topk_token<G, V, VEC>(t, t < T, threadIdx.x % G, logits + (int64_t)t * E, E, k, renorm, idx, w, nullptr);
    }
}

template <int G, int V, bool VEC>
static int launch_topk_t(float *logits, int T, int E, int k, int renorm, int32_t *idx, float *w, hipStream_t s,
                         int n_parts, const float *parts, int64_t part_stride)
{
    const int tpb = kThreads / G;
    ProfScope ps("topk", s);
    const auto kern = n_parts <= 1 ? topk_kernel<G, V, VEC, PARTS_NONE>
                      : topk_stages<G, V, VEC>(T, n_parts) ? topk_kernel<G, V, VEC, PARTS_STAGED> : topk_kernel<G, V, VEC, PARTS_LANES>;
    hipLaunchKernelGGL(kern, dim3(ceil_div(T, tpb)), dim3(kThreads), 0, s, logits, T, E, k, renorm, idx, w, n_parts, parts, part_stride);
    MOE_LAUNCH_CHECK("topk_kernel");
    return MOE_OK;
}

int launch_topk(float *logits, int T, int E, int k, int renorm, int32_t *idx, float *w, hipStream_t s, int n_parts,
                const float *parts, int64_t part_stride)
{
    if (T == 0) return MOE_OK;
    if (n_parts > kMaxLogitParts) {
        set_error("top-k: %d logit slices, at most %d", n_parts, kMaxLogitParts);
        return MOE_ERR_INVALID_ARG;
    }
    if (E % 4 == 0) {  // rows are 16-byte aligned: vector loads, fewer lanes per token
        if (E <= 8) return launch_topk_t<2, 4, true>(logits, T, E, k, renorm, idx, w, s, n_parts, parts, part_stride);
        if (E <= 16) return launch_topk_t<4, 4, true>(logits, T, E, k, renorm, idx, w, s, n_parts, parts, part_stride);
        if (E <= 32) return launch_topk_t<8, 4, true>(logits, T, E, k, renorm, idx, w, s, n_parts, parts, part_stride);
        if (E <= 64) return launch_topk_t<16, 4, true>(logits, T, E, k, renorm, idx, w, s, n_parts, parts, part_stride);
        if (E <= 128) return launch_topk_t<16, 8, true>(logits, T, E, k, renorm, idx, w, s, n_parts, parts, part_stride);
        if (E <= 256) return launch_topk_t<16, 16, true>(logits, T, E, k, renorm, idx, w, s, n_parts, parts, part_stride);
        if (E <= 512) return launch_topk_t<32, 16, true>(logits, T, E, k, renorm, idx, w, s, n_parts, parts, part_stride);
        return launch_topk_t<64, 16, true>(logits, T, E, k, renorm, idx, w, s, n_parts, parts, part_stride);
    }
    if (E <= 4) return launch_topk_t<4, 1, false>(logits, T, E, k, renorm, idx, w, s, n_parts, parts, part_stride);
    if (E <= 8) return launch_topk_t<8, 1, false>(logits, T, E, k, renorm, idx, w, s, n_parts, parts, part_stride);
    if (E <= 16) return launch_topk_t<16, 1, false>(logits, T, E, k, renorm, idx, w, s, n_parts, parts, part_stride);
    if (E <= 32) return launch_topk_t<32, 1, false>(logits, T, E, k, renorm, idx, w, s, n_parts, parts, part_stride);
    if (E <= 64) return launch_topk_t<64, 1, false>(logits, T, E, k, renorm, idx, w, s, n_parts, parts, part_stride);
    if (E <= 128) return launch_topk_t<64, 2, false>(logits, T, E, k, renorm, idx, w, s, n_parts, parts, part_stride);
    if (E <= 256) return launch_topk_t<64, 4, false>(logits, T, E, k, renorm, idx, w, s, n_parts, parts, part_stride);
    if (E <= 512) return launch_topk_t<64, 8, false>(logits, T, E, k, renorm, idx, w, s, n_parts, parts, part_stride);
    return launch_topk_t<64, 16, false>(logits, T, E, k, renorm, idx, w, s, n_parts, parts, part_stride);
}

// ------------------------------------------------------------------------------------------------
// counts / offsets / stable permutation.
//   K1 route_hist : block b histograms its 256 tokens into LDS -> block_hist[b][e]
//                   (the fused gate kernel writes these rows itself, one per tile of its own)
//   K2 route_prefix: per expert (one wave each), exclusive prefix over the rows (block_hist becomes
//                   the base of row b inside expert e) and counts[e]
//   K3 route_rank : every block scans the counts into offsets[] (wave-shuffle scan), then ranks its
//                   tokens: bit-wise ballots find equal experts inside a wave, an LDS prefix runs over
//                   the 4 waves, plus the row base and the expert offset
// ------------------------------------------------------------------------------------------------
int route_blocks(int T) { return T > 0 ? ceil_div(T, kThreads) : 1; }

__device__ __forceinline__ int clamp_expert(int e, int E) { return e < 0 ? 0 : (e >= E ? E - 1 : e); }

__global__ __launch_bounds__(kThreads) void route_hist_kernel(const int32_t *__restrict__ idx, int T, int E, int k,
                                                              int32_t *__restrict__ block_hist)
{
    __shared__ int hist[MOE_MAX_E];
    for (int e = threadIdx.x; e < E; e += kThreads) hist[e] = 0;
    __syncthreads();
    const int t = blockIdx.x * kThreads + threadIdx.x;
    if (t < T) {
        for (int j = 0; j < k; ++j) atomicAdd(&hist[clamp_expert(idx[(int64_t)t * k + j], E)], 1);
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += kThreads) block_hist[(int64_t)blockIdx.x * E + e] = hist[e];
}

// Per expert, the exclusive prefix of its histogram column over the rows (blocks of tokens) and its total.
// One wave per expert, 64 rows per step: the column is walked with a wave-shuffle scan and a running carry.
// hist[b][e] becomes the number of assignments to expert e in the rows before b.
__global__ __launch_bounds__(kThreads) void route_prefix_kernel(int32_t *__restrict__ hist, int nrows, int E,
                                                                int32_t *__restrict__ counts)
{
    const int lane = threadIdx.x % kWave;
    const int e = blockIdx.x * (kThreads / kWave) + threadIdx.x / kWave;
    if (e >= E) return;  // whole waves leave together
    int carry = 0;
    for (int b0 = 0; b0 < nrows; b0 += kWave) {
        const int b = b0 + lane;
        const int v = b < nrows ? hist[(int64_t)b * E + e] : 0;
        int incl = v;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int up = __shfl_up(incl, off, kWave);
            if (lane >= off) incl += up;
        }
        if (b < nrows) hist[(int64_t)b * E + e] = carry + incl - v;
        carry += __shfl(incl, kWave - 1, kWave);
    }
    if (lane == 0) counts[e] = carry;
}

// Exclusive scan of n <= 4 * blockDim values in LDS (in place), one block; returns nothing, `total` receives
// the sum.  Thread t owns elements 4 t .. 4 t + 3.
__device__ __forceinline__ void block_exclusive_scan4(int *vals, int n, int *wave_tot, int &total)
{
    const int lane = threadIdx.x % kWave;
    const int wave = threadIdx.x / kWave;
    const int nw = blockDim.x / kWave;
    int loc[4];
    int sum = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int at = 4 * threadIdx.x + i;
        loc[i] = at < n ? vals[at] : 0;
        sum += loc[i];
    }
    int incl = sum;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int up = __shfl_up(incl, off, kWave);
        if (lane >= off) incl += up;
    }
    if (lane == kWave - 1) wave_tot[wave] = incl;
    __syncthreads();
    int run = incl - sum;
    int all = 0;
    for (int w2 = 0; w2 < nw; ++w2) {
        const int t = wave_tot[w2];
        if (w2 < wave) run += t;
        all += t;
    }
    total = all;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int at = 4 * threadIdx.x + i;
        if (at < n) vals[at] = run;
        run += loc[i];
    }
    __syncthreads();
}

// Schedule of the grouped GEMM's ring kernel (layout: moe_internal.h), by one whole block.  rows_of(e), e < E.
// What it balances: an expert's rows come in tiles of up to eight 32-row units, and a tile costs about six units whatever
// its height, and one of less than four units as much as one of four: its time is that of the weights' way into the CU
// (fitted to K tiles of 0.8 us at one unit, 1.05 at four and 1.6 at eight; where all CUs stream weights of their own from HBM, 8
// experts 8192 -> 8192, they take 1.54, 1.70 and 2.10; counted as less, a low tile made 128 experts of one or two units fall to the XCDs by
// 15 to 17 instead of 16, a round more for some: 1473 against 1610 us for 34 rows).  The choice of a height leaves that floor out: it
// compares heights for the same rows, and with the floor no round would be spread over idle blocks.
// The experts' rows, in order, are cut in eight parts of equal cost, one per XCD, between two tiles of an expert at most
// (an XCD's blocks share weights and rows in its L2, so what one expert needs stays together).  Inside a part every expert's tiles
// get the same height, at most the one that makes the part's rounds of 32 blocks cheapest, and the experts with the taller tiles
// come first, so that a round's tiles cost about the same.  (Places among experts of one height are handed out by LDS atomics:
// their order differs between runs, the sums do not.)
//
// Where parts of whole row tiles do not come out, the XCDs share one list of experts and each takes an eighth of its output tiles:
// if a window of the kernel's holds the experts and the eighths' rounds are estimated at less than kRingSharedGain of the slowest
// part's, with up to kRingSharedTiles row tiles kRingSharedFewGain.  The list is in the experts' order: sorted by height the first
// eighth would cost the most.
// FFN in us, parts / shared: 128 experts 2048 -> 8192, 1024 rows on one expert 151 / 137, on four 189 / 158; 8 experts 4096 -> 14336, 1024
// rows on four 477 / 374, on one 401 / 288; 4 experts 8192 -> 28672, 400 rows on two 1238 / 661.  With more than kRingSharedTiles row
// tiles the time's ratio is the estimated one plus a twentieth, because an eighth's heights are mixed: 42 experts 768 -> 1536, 372 rows
// each 0.65, measured 0.73; 25 experts 1280 -> 1280, 857 rows 0.74, 0.78; 32 experts 1024 -> 4096, 256 rows 0.84, 0.91; 64 experts
// 1024 -> 4096, 256 rows, more and less skewed 0.90, 0.99 and 0.95, 1.03; 16 experts 2048 -> 8192, 500 rows 1.00, 1.06.  With fewer it
// is spread about the estimate: 92 batches of 8 and 16 experts, 1024 -> 4096, 2048 -> 8192 and 4096 -> 14336, with 245 to 340 rows each
// measured 0.81 to 0.98 where it is below 0.92, 0.95 to 1.03 up to 0.95, 0.96 to 1.04 up to 0.98 and 0.98 to 1.14 above (8 experts 4096 ->
// 14336, parts / shared: 245 rows 764 / 620 at 0.69, 273 rows 615 / 694 at 0.98 and 616 / 702 at 1.02).
// (Dealing the rounds of the whole chip over the XCDs instead, 32 neighbours on the list each, cost 32 even experts 10 %.)

struct RingScratch {
    int cost[MOE_MAX_E];         // then its prefix
    int wave_tot[16];
    int tiles[8][9];             // of every part, cut to a height of at most h; [0]: its units
    int cap[2][8];
    int shared;
    int bin[2][64];              // experts by GEMM, part and height (8 first), then the first place of each
};

template <typename Rows>
__device__ __forceinline__ void ring_schedule(const Rows &rows_of, int E, int n1, int n2, int32_t *__restrict__ list1,
                                              int32_t *__restrict__ list2, int max_list, int32_t *__restrict__ words, RingScratch &sm)
{
    const int tid = threadIdx.x, nthreads = blockDim.x, lane = tid % kWave, wave = tid / kWave;
    for (int e = tid; e < E; e += nthreads) sm.cost[e] = ring_cost(ring_units(rows_of(e)));
    if (tid < 72) sm.tiles[tid / 9][tid % 9] = 0;
    if (tid < 128) sm.bin[tid / 64][tid % 64] = 0;
    if (tid < 9) words[kRingCut + tid] = MOE_MAX_E << kRingCutShift;  // no expert
    __syncthreads();
    int total = 0;
    block_exclusive_scan4(sm.cost, E, sm.wave_tot, total);
    for (int e = tid; e < E; e += nthreads)
        ring_pieces(
            ring_units(rows_of(e)), sm.cost[e], total,
            [&](int x, int, int units) {
                atomicAdd(&sm.tiles[x][0], units);
                for (int h = 1; h <= 8; ++h) atomicAdd(&sm.tiles[x][h], (units + h - 1) / h);
            },
            [&](int x, int first) { words[kRingCut + x] = e << kRingCutShift | first; });
    __syncthreads();
    if (wave == 0) {
        // lanes 0 .. 7 and 8 .. 15: the parts of the first and of the second GEMM; 16 and 17: the GEMMs with one list for all XCDs
        int all = 0;  // lane h: row tiles of all parts cut to a height of at most h; lane 0: units
        if (lane < 9)
#pragma unroll
            for (int x = 0; x < 8; ++x) all += sm.tiles[x][lane];
        const int row_tiles = __shfl(all, 8, kWave);
        const bool one_list = lane >= 16;
        const int x = lane & 7, n = (one_list ? lane & 1 : lane >> 3) == 0 ? n1 : n2, log_blocks = one_list ? 8 : 5;
        // read at once: each read where one_list says so is a branch and a wait of its own (layer of 24 experts 1000 -> 4000, 3001
        // tokens, 197.0 us that way, 196.0 this way)
        int tiles[9];
#pragma unroll
        for (int h = 0; h <= 8; ++h) tiles[h] = sm.tiles[x][h];
#pragma unroll
        for (int h = 0; h <= 8; ++h) {
            const int all_h = __shfl(all, h, kWave);
            tiles[h] = one_list ? all_h : tiles[h];
        }
        const float units = (float)tiles[0];
        RingRounds rounds;
#pragma unroll
        for (int h = 8; h >= 1; --h) ring_try_height(rounds, h, tiles[h], units, n, log_blocks);
        float slowest = rounds.cost;  // of the GEMM's parts
#pragma unroll
        for (int m = 1; m < 8; m <<= 1) slowest = fmaxf(slowest, __shfl_xor(slowest, m, kWave));
        // a GEMM's K loop is as long as the other one has columns
        const float parts = __shfl(slowest, 0, kWave) * (float)n2 + __shfl(slowest, 8, kWave) * (float)n1;
        const float eighths = __shfl(rounds.cost, 16, kWave) * (float)n2 + __shfl(rounds.cost, 17, kWave) * (float)n1;
        const bool share = ring_shares_pay(E, row_tiles, eighths, parts);
        const int cap_all = __shfl(rounds.height, 16 + (lane >> 3 & 1), kWave);
        if (lane < 16) sm.cap[lane >> 3][x] = share ? cap_all : rounds.height;
        if (lane == 0) sm.shared = share;
    }
    __syncthreads();
    const bool shared = sm.shared;
    auto pieces = [&](int e, auto piece) {
        if (!shared) ring_pieces(ring_units(rows_of(e)), sm.cost[e], total, piece, [](int, int) {});
        else if (ring_units(rows_of(e)) > 0) piece(0, 0, ring_units(rows_of(e)));
    };
    if (tid < 8) words[kRingCap + tid] = sm.cap[0][tid] | sm.cap[1][tid] << 8 | (int)shared << kRingShared;
    if (shared && tid < 9) words[kRingCut + tid] = MOE_MAX_E << kRingCutShift;
    auto bin_of = [&](int g, int x, int units) {
        const int k = (units + sm.cap[g][x] - 1) / sm.cap[g][x];
        return &sm.bin[g][shared ? 0 : 8 * x + 8 - (units + k - 1) / k];
    };
    for (int e = tid; e < E; e += nthreads)
        pieces(e, [&](int x, int, int units) {
            for (int g = 0; g < 2; ++g) atomicAdd(bin_of(g, x, units), 1);
        });
    __syncthreads();
    if (wave < 2) {
        const int v = sm.bin[wave][lane];
        int incl = v;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const int up = __shfl_up(incl, off, kWave);
            if (lane >= off) incl += up;
        }
        sm.bin[wave][lane] = incl - v;
        // the parts' places, the same for both GEMMs (shared: all experts are in the first bin)
        if (wave == 0 && (lane & 7) == 0) words[kRingFirst + (lane >> 3)] = shared ? 0 : incl - v;
        const int part_end = __shfl(incl, shared ? kWave - 1 : lane, kWave);
        if (wave == 0 && (lane & 7) == 7) words[kRingLast + (lane >> 3)] = part_end;
    }
    __syncthreads();
    for (int e = tid; e < E; e += nthreads)
        pieces(e, [&](int x, int, int units) {
            for (int g = 0; g < 2; ++g) {
                const int at = atomicAdd(bin_of(g, x, units), 1);
                if (at < max_list) (g == 0 ? list1 : list2)[at] = e;  // at most E + 7 places are needed
            }
        });
}

// Stable position of every assignment.  Block b ranks its 256 tokens:
//   row(t, j) = offsets[e] + (assignments to e in the blocks before b) + (in the waves before this one)
//               + (in the lanes before this one, or in earlier slots of this lane)
// Every block scans the E counts into the offsets itself (E <= 1024 integers out of L2), so no launch stands
// between the per-expert prefix and the ranking; block 0 also writes offsets[] and, when asked, the grouped
// GEMM's M-tile map.
// Equal experts inside a wave are found with one ballot per BIT of the expert index (ceil(log2 E) of them
// per slot) instead of one per expert: the lanes whose slot j' holds this lane's expert are the AND over the
// bits b of (bit b of my expert set ? ballot(bit b set) : its complement).
// hist_row_step: histogram rows per block of 256 tokens (the fused gate kernel's tiles may be shorter).
template <int KMAX>
__global__ __launch_bounds__(kThreads) void route_rank_kernel(const int32_t *__restrict__ idx, int T, int E, int k,
                                                              int nbits, const int32_t *__restrict__ counts,
                                                              const int32_t *__restrict__ block_base,
                                                              int hist_row_step, int32_t *__restrict__ offsets,
                                                              int32_t *__restrict__ dst_row,
                                                              int32_t *__restrict__ src_tok, int tile_bm,
                                                              int32_t *__restrict__ tile_expert,
                                                              int32_t *__restrict__ tile_row,
                                                              int32_t *__restrict__ num_tiles, int max_m_tiles,
                                                              int ring_n1, int ring_n2)
{
    constexpr int NW = kThreads / kWave;
    __shared__ int offs[MOE_MAX_E];
    __shared__ int wave_cnt[NW][MOE_MAX_E];
    __shared__ int wave_tot[NW];
    const int lane = threadIdx.x % kWave;
    const int wave = threadIdx.x / kWave;
    const int t = blockIdx.x * kThreads + threadIdx.x;

    for (int e = threadIdx.x; e < E; e += kThreads) {
        offs[e] = counts[e];
#pragma unroll
        for (int w2 = 0; w2 < NW; ++w2) wave_cnt[w2][e] = 0;
    }
    __syncthreads();
    int total = 0;
    block_exclusive_scan4(offs, E, wave_tot, total);  // offs[e] = first row of expert e
    if (tile_bm == kRingMap && blockIdx.x == gridDim.x - 1) {  // a block of its own, next to the ranking ones
        __shared__ RingScratch ring;
        ring_schedule([&](int e) { return (e + 1 < E ? offs[e + 1] : total) - offs[e]; }, E, ring_n1, ring_n2, tile_expert, tile_row,
                      max_m_tiles, num_tiles, ring);
        return;
    }
    if (blockIdx.x == 0) {
        for (int e = threadIdx.x; e < E; e += kThreads) offsets[e] = offs[e];
        if (threadIdx.x == 0) offsets[E] = total;
    }

    int ej[KMAX];
    int below[KMAX];  // assignments to the same expert earlier in this wave
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
        ej[j] = (t < T && j < k) ? clamp_expert(idx[(int64_t)t * k + j], E) : -1;
        below[j] = 0;
    }
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
    const uint64_t gt_mask = (lane == kWave - 1) ? 0ull : (~0ull << (lane + 1));
    int after[KMAX];  // ... later in this wave
#pragma unroll
    for (int j = 0; j < KMAX; ++j) after[j] = 0;
#pragma unroll
    for (int jp = 0; jp < KMAX; ++jp) {
        if (jp >= k) continue;  // uniform
        uint64_t same[KMAX];
        const uint64_t valid = __ballot(ej[jp] >= 0);
#pragma unroll
        for (int j = 0; j < KMAX; ++j) same[j] = valid;
        for (int b = 0; b < nbits; ++b) {
            const uint64_t bal = __ballot(ej[jp] >= 0 && ((ej[jp] >> b) & 1));
#pragma unroll
            for (int j = 0; j < KMAX; ++j) same[j] &= ((ej[j] >> b) & 1) ? bal : ~bal;
        }
#pragma unroll
        for (int j = 0; j < KMAX; ++j) {
            if (ej[j] < 0) continue;
            below[j] += __popcll(same[j] & lt_mask);
            after[j] += __popcll(same[j] & gt_mask);
            // the lane's own other slots (only a caller's duplicate experts make these match)
            if (jp < j && ej[jp] == ej[j]) below[j] += 1;
            if (jp > j && ej[jp] == ej[j]) after[j] += 1;
        }
    }
    // the last assignment of every expert present in the wave publishes the wave's count of it
#pragma unroll
    for (int j = 0; j < KMAX; ++j)
        if (ej[j] >= 0 && after[j] == 0) wave_cnt[wave][ej[j]] = below[j] + 1;
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += kThreads) {
        int run = 0;
#pragma unroll
        for (int w2 = 0; w2 < NW; ++w2) {
            const int c = wave_cnt[w2][e];
            wave_cnt[w2][e] = run;
            run += c;
        }
    }
    __syncthreads();
    if (t < T) {
        const int32_t *base = block_base + (int64_t)blockIdx.x * hist_row_step * E;
#pragma unroll
        for (int j = 0; j < KMAX; ++j) {
            if (j < k) {
                const int e = ej[j];
                const int r = offs[e] + base[e] + wave_cnt[wave][e] + below[j];
                dst_row[(int64_t)t * k + j] = r;
                src_tok[r] = t;
            }
        }
    }
    if (tile_bm > 0 && tile_bm != kRingMap && blockIdx.x == 0) {  // the grouped GEMM's M-tile map: expert e owns ceil(count / tile_bm) tiles
        __syncthreads();
        int *first = &wave_cnt[0][0];  // reused: first tile of every expert
        for (int e = threadIdx.x; e < E; e += kThreads) first[e] = (counts[e] + tile_bm - 1) / tile_bm;
        __syncthreads();
        int n_tiles = 0;
        block_exclusive_scan4(first, E, wave_tot, n_tiles);
        for (int e = threadIdx.x; e < E; e += kThreads) {
            const int nt = (counts[e] + tile_bm - 1) / tile_bm;
            for (int i = 0; i < nt; ++i) {
                const int ti = first[e] + i;
                if (ti < max_m_tiles) {
                    tile_expert[ti] = e;
                    tile_row[ti] = offs[e] + i * tile_bm;
                }
            }
        }
        if (threadIdx.x == 0) num_tiles[0] = min(n_tiles, max_m_tiles);
    }
}

// ------------------------------------------------------------------------------------------------
// Small batches (decoder steps: a few hundred assignments): the three kernels above are then all
// launch latency, so one block of 256 to 1024 threads does the whole job in LDS -- histogram, scan,
// tile map and ranks -- with one thread per assignment a = t*k + j, in chunks of its size.  The rank
// of a inside its expert is (assignments of that expert in earlier chunks and waves) + (lanes
// below it in its wave with the same expert); waves add their counts to the running per-expert
// totals one after the other, so the order is that of a, as in the kernels above.
// ------------------------------------------------------------------------------------------------
static constexpr int kSmallRouteMax = 1024;  // assignments: one round of the block

// Assignments up to which that block also beats the three launches, us by 1024, 1536, 2048, 3072 assignments against 8.2 ... 9.7
// for the three launches: 8 experts 5.0, 6.3, 7.4, 9.8; 16 experts 5.1, 6.5, 7.5, 9.9; 32 experts 5.2, 6.6, 8.1.
static constexpr int kRouteBlockMax = 2 * kSmallRouteMax;
static_assert(kRouteBlockMax < 1 << 15 && MOE_MAX_E <= 1024, "the block's scan keeps rows and tiles in halves of a word, an expert per thread");

__device__ __forceinline__ void route_small(const int32_t *idx, int n_assign, int E, int k, int32_t *__restrict__ counts,
                                            int32_t *__restrict__ offsets, int32_t *__restrict__ dst_row,
                                            int32_t *__restrict__ src_tok, int tile_bm, int32_t *__restrict__ tile_expert,
                                            int32_t *__restrict__ tile_row, int32_t *__restrict__ num_tiles, int max_m_tiles,
                                            int ring_n1, int ring_n2)
{
    __shared__ int hist[MOE_MAX_E];   // counts
    __shared__ int seen[MOE_MAX_E];   // running totals of the ranking pass
    __shared__ int start[MOE_MAX_E];  // first row of every expert
    __shared__ int wave_tot[16];
    const int lane = threadIdx.x % kWave;
    const int wave = threadIdx.x / kWave;
    const int threads = blockDim.x;
    hist[threadIdx.x] = 0;  // at least as many threads as experts
    seen[threadIdx.x] = 0;
    __syncthreads();
    for (int a = threadIdx.x; a < n_assign; a += threads) atomicAdd(&hist[clamp_expert(idx[a], E)], 1);
    __syncthreads();
    // exclusive scan over the experts, thread e owns expert e: rows in the low half of a word, tiles of the grouped GEMM's M-tile
    // map in the high half (at most kRouteBlockMax of either)
    const bool map = tile_bm > 0 && tile_bm != kRingMap;  // uniform over the block
    const int cnt = threadIdx.x < E ? hist[threadIdx.x] : 0;
    const int nt = map ? (cnt + tile_bm - 1) / tile_bm : 0;
    const int both = cnt | nt << 16;
    int incl = both;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int up = __shfl_up(incl, off, kWave);
        if (lane >= off) incl += up;
    }
    if (lane == kWave - 1) wave_tot[wave] = incl;
    __syncthreads();
    int before = incl - both;
    for (int w2 = 0; w2 < wave; ++w2) before += wave_tot[w2];
    const int my_off = before & 0xffff;
    if (threadIdx.x < E) {
        counts[threadIdx.x] = cnt;
        offsets[threadIdx.x] = my_off;
        start[threadIdx.x] = my_off;
    }
    if (threadIdx.x == 0) offsets[E] = n_assign;
    if (map) {  // as route_rank_kernel's block 0 writes it
        const int first = before >> 16;
        for (int i = 0; i < nt; ++i) {
            const int ti = first + i;
            if (ti < max_m_tiles) {
                tile_expert[ti] = threadIdx.x;
                tile_row[ti] = my_off + i * tile_bm;
            }
        }
        if (threadIdx.x == threads - 1) num_tiles[0] = min(first + nt, max_m_tiles);
    } else if (tile_bm > 0) {
        __shared__ RingScratch ring;
        ring_schedule([&](int e) { return hist[e]; }, E, ring_n1, ring_n2, tile_expert, tile_row, max_m_tiles, num_tiles, ring);
    }
    __syncthreads();
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
    int nbits = 0;
    while ((1 << nbits) < E) ++nbits;
    for (int a0 = 0; a0 < n_assign; a0 += threads) {  // trip count uniform over the block
        const int a = a0 + threadIdx.x;
        const bool live = a < n_assign;
        const int e = live ? clamp_expert(idx[a], E) : -1;
        // lanes of the wave with the same expert, by one ballot per bit of the index (see route_rank_kernel).  One per expert
        // present, as here before, made this loop the block's time: 64 tokens over 128 experts 18.6 us with their top-k, now 12.4.
        uint64_t mask = __ballot(live);
        for (int b = 0; b < nbits; ++b) {
            const uint64_t bal = __ballot(live && ((e >> b) & 1));
            mask &= ((e >> b) & 1) ? bal : ~bal;
        }
        const int below = __popcll(mask & lt_mask), same = __popcll(mask);
        const int first = live ? __ffsll((unsigned long long)mask) - 1 : lane;  // the group's first lane
        const bool leader = live && first == lane;
        // the waves take their turns in order; the first lane of every expert group moves the total
        int base = 0;
        const int live_waves = min(threads / kWave, (n_assign - a0 + kWave - 1) / kWave);  // uniform over the block
        for (int w2 = 0; w2 < live_waves; ++w2) {
            if (wave == w2 && leader) {
                base = seen[e];
                seen[e] = base + same;
            }
            __syncthreads();
        }
        base = __shfl(base, first, kWave);  // to the group's other lanes
        if (live) {
            const int r = start[e] + base + below;
            dst_row[a] = r;
            src_tok[r] = a / k;
        }
    }
}

__global__ __launch_bounds__(1024) void route_small_kernel(const int32_t *__restrict__ idx, int n_assign, int E, int k, RouteOut o)
{
    route_small(idx, n_assign, E, k, o.counts, o.offsets, o.dst_row, o.src_tok, o.tile_bm, o.tile_expert, o.tile_row, o.num_tiles,
                o.max_m_tiles, o.ring_n1, o.ring_n2);
}

// Threads of the block that routes: as many as it has experts, assignments and other items (at most 1024, in rounds then).
// Fewer waves start and meet sooner: with it and the logits staged by all threads the launch takes, alone, 8.5 -> 6.2 us for one
// token over 128 experts (16 slices), 6.5 -> 5.9 over 64.
static int route_block_threads(int64_t items, int E, int64_t n_assign)
{
    const int64_t most = items > n_assign ? (items > E ? items : E) : (n_assign > E ? n_assign : E);
    return most <= 256 ? 256 : most <= 512 ? 512 : 1024;
}

// Top-k of a decoder step and its routing in one launch: 1024 / G tokens fit the block, their logits and selection stay in LDS.
// Bound by latency: a dependent launch costs about 4.5 us here whatever it does.
// STAGED: lanes with several words each (V > 4), and batches of at most a word per thread.  Else the lanes add their own slices, whose
// loads the compiler has in flight together.  Layer in us, lanes / staged: 512 experts 512 -> 2048, 32 tokens 71.0 / 73.5; 128 experts 1024 ->
// 4096, 52 tokens 59.2 / 60.3; 64 experts 1024 -> 64, 64 tokens 24.2 / 25.0, 2048 -> 64 28.6 / 29.4.
template <int G, int V, bool VEC, bool STAGED>
__global__ __launch_bounds__(1024) void route_topk_kernel(float *logits, int T, int E, int k, int renorm, int32_t *__restrict__ idx,
                                                          float *__restrict__ w, int n_parts, const float *__restrict__ parts,
                                                          int64_t part_stride, RouteOut o)
{
    __shared__ int s_idx[kSmallRouteMax];
    const int t = threadIdx.x / G;
    if constexpr (STAGED) {
        __shared__ __align__(16) float s_logits[1024 * (VEC ? 4 : V)];
        stage_logits<VEC>(s_logits, logits, T * E, n_parts, parts, part_stride);
        __syncthreads();
        topk_token<G, V, VEC>(t, t < T, threadIdx.x % G, s_logits + t * E, E, k, renorm, idx, w, s_idx);
    } else {
        const int64_t at = (int64_t)t * E;
        topk_token<G, V, VEC, true>(t, t < T, threadIdx.x % G, logits + at, E, k, renorm, idx, w, s_idx, n_parts, parts + at, part_stride);
    }
    __syncthreads();
    route_small(s_idx, T * k, E, k, o.counts, o.offsets, o.dst_row, o.src_tok, o.tile_bm, o.tile_expert, o.tile_row, o.num_tiles,
                o.max_m_tiles, o.ring_n1, o.ring_n2);
}

template <int G, int V, bool VEC>
static int launch_route_topk_t(float *logits, int T, int E, int k, int renorm, int32_t *idx, float *w, hipStream_t s, int n_parts,
                               const float *parts, int64_t part_stride, const RouteOut &o, bool *taken)
{
    // (without vector loads a full block is no faster than two launches: layer of 31 experts 1000 -> 1136, 31 tokens 48.4 / 48.8 us, 16
    // tokens 46.1 / 45.2; 15 experts, 30 tokens 32.7 / 31.6)
    if (T > (VEC ? 1024 : 512) / G) return MOE_OK;
    *taken = true;
    ProfScope ps("route", s);
    const int64_t words = (int64_t)T * E / (VEC ? 4 : 1), lanes = (int64_t)T * G;
    const int threads = route_block_threads(words > lanes ? words : lanes, E, (int64_t)T * k);
    if constexpr (VEC) {
        if (V <= 4 || words > 1024) {
            hipLaunchKernelGGL((route_topk_kernel<G, V, VEC, false>), dim3(1), dim3(threads), 0, s, logits, T, E, k, renorm, idx, w, n_parts,
                               parts, part_stride, o);
            MOE_LAUNCH_CHECK("route_topk_kernel");
            return MOE_OK;
        }
    }
    if constexpr (!VEC || V > 4) {
        hipLaunchKernelGGL((route_topk_kernel<G, V, VEC, true>), dim3(1), dim3(threads), 0, s, logits, T, E, k, renorm, idx, w, n_parts, parts,
                           part_stride, o);
        MOE_LAUNCH_CHECK("route_topk_kernel");
    }
    return MOE_OK;
}

// *taken = false: not a batch for the single block (nothing was launched).  Few tokens only, so that the block's one
// compute unit is no slower than the top-k kernel's blocks; the lane groups are the top-k kernel's.
int launch_route_topk(float *logits, int T, int E, int k, int renorm, int32_t *idx, float *w, hipStream_t s, int n_parts,
                      const float *parts, int64_t part_stride, const RouteOut &o, bool *taken)
{
    *taken = false;
    if (T < 1 || T > 64 || (int64_t)T * k > kSmallRouteMax || n_parts > kMaxLogitParts) return MOE_OK;
#define MOE_ROUTE_TOPK(G, V, VEC) launch_route_topk_t<G, V, VEC>(logits, T, E, k, renorm, idx, w, s, n_parts, parts, part_stride, o, taken)
    if (E % 4 == 0) {
        if (E <= 8) return MOE_ROUTE_TOPK(2, 4, true);
        if (E <= 16) return MOE_ROUTE_TOPK(4, 4, true);
        if (E <= 32) return MOE_ROUTE_TOPK(8, 4, true);
        if (E <= 64) return MOE_ROUTE_TOPK(16, 4, true);
        if (E <= 128) return MOE_ROUTE_TOPK(16, 8, true);
        if (E <= 256) return MOE_ROUTE_TOPK(16, 16, true);
        if (E <= 512) return MOE_ROUTE_TOPK(32, 16, true);
        return MOE_ROUTE_TOPK(64, 16, true);
    }
    if (E <= 4) return MOE_ROUTE_TOPK(4, 1, false);
    if (E <= 8) return MOE_ROUTE_TOPK(8, 1, false);
    if (E <= 16) return MOE_ROUTE_TOPK(16, 1, false);
    if (E <= 32) return MOE_ROUTE_TOPK(32, 1, false);
    if (E <= 64) return MOE_ROUTE_TOPK(64, 1, false);
    if (E <= 128) return MOE_ROUTE_TOPK(64, 2, false);
    return MOE_OK;
#undef MOE_ROUTE_TOPK
}

bool route_uses_hist(int T, int k) { return (int64_t)T * k > kSmallRouteMax; }

int launch_route(const int32_t *idx, int T, int E, int k, const RouteOut &o, int32_t *block_hist, hipStream_t s, int hist_tokens)
{
    ProfScope ps("route", s);  // histogram + prefix + rank together
    if ((int64_t)T * k <= (hist_tokens > 0 ? kSmallRouteMax : kRouteBlockMax)) {  // a histogram that is there saves a launch
        hipLaunchKernelGGL(route_small_kernel, dim3(1), dim3(route_block_threads(0, E, (int64_t)T * k)), 0, s, idx, T * k, E, k, o);
        MOE_LAUNCH_CHECK("route_small_kernel");
        return MOE_OK;
    }
    // hist_tokens > 0: block_hist already holds one histogram row per hist_tokens tokens (the fused gate kernel
    // wrote it); else it is made here, one row per block of 256 tokens
    if (hist_tokens > 0 && (kThreads % hist_tokens != 0)) {
        set_error("route: %d tokens per histogram row do not divide %d", hist_tokens, kThreads);
        return MOE_ERR_INVALID_ARG;
    }
    const int nblk = route_blocks(T);
    int nrows = nblk, row_step = 1;
    if (hist_tokens > 0) {
        nrows = ceil_div(T, hist_tokens);
        row_step = kThreads / hist_tokens;
    } else {
        hipLaunchKernelGGL(route_hist_kernel, dim3(nblk), dim3(kThreads), 0, s, idx, T, E, k, block_hist);
        MOE_LAUNCH_CHECK("route_hist_kernel");
    }
    hipLaunchKernelGGL(route_prefix_kernel, dim3(ceil_div(E, kThreads / kWave)), dim3(kThreads), 0, s, block_hist,
                       nrows, E, o.counts);
    MOE_LAUNCH_CHECK("route_prefix_kernel");
    int nbits = 0;
    while ((1 << nbits) < E) ++nbits;
#define MOE_RANK(KM)                                                                                              \
    hipLaunchKernelGGL(route_rank_kernel<KM>, dim3(nblk + (o.tile_bm == kRingMap)), dim3(kThreads), 0, s, idx, T, E, k, nbits, o.counts, \
                       block_hist, row_step, o.offsets, o.dst_row, o.src_tok, o.tile_bm, o.tile_expert, o.tile_row, \
                       o.num_tiles, o.max_m_tiles, o.ring_n1, o.ring_n2)
    // KMAX = slots a lane holds: the smallest instantiation that holds k
    if (k <= 1) MOE_RANK(1);
    else if (k <= 2) MOE_RANK(2);
    else if (k <= 4) MOE_RANK(4);
    else MOE_RANK(MOE_MAX_K);
#undef MOE_RANK
    MOE_LAUNCH_CHECK("route_rank_kernel");
    return MOE_OK;
}

// ------------------------------------------------------------------------------------------------
// M-tile map of the grouped GEMM: expert e owns ceil(count_e / BM) tiles; tile i of the flat list
// starts at row tile_row[i] of expert tile_expert[i].  Experts with no rows own no tile, so their
// weights are never touched.  One block of 1024 threads, thread e handles expert e, e + 1024, ...
// (E <= 1024 here, so one expert per thread).
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void tile_map_kernel(const int32_t *__restrict__ offsets, int E, int BM,
                                                        int32_t *__restrict__ tile_expert,
                                                        int32_t *__restrict__ tile_row,
                                                        int32_t *__restrict__ num_tiles, int max_m_tiles,
                                                        const int32_t *__restrict__ stage_of, int stage, int ring_n1, int ring_n2)
{
    if (BM == kRingMap) {
        __shared__ RingScratch ring;
        __shared__ int rows[MOE_MAX_E];
        if (threadIdx.x < E)
            rows[threadIdx.x] = stage_of && stage_of[threadIdx.x] != stage ? 0 : max(0, offsets[threadIdx.x + 1] - offsets[threadIdx.x]);
        __syncthreads();
        ring_schedule([&](int e) { return rows[e]; }, E, ring_n1, ring_n2, tile_expert, tile_row, max_m_tiles, num_tiles, ring);
        return;
    }
    __shared__ int wave_tot[16];
    const int e = threadIdx.x;
    int row0 = 0, row1 = 0;
    if (e < E && (!stage_of || stage_of[e] == stage)) {
        row0 = offsets[e];
        row1 = offsets[e + 1];
    }
    const int nt = (row1 > row0) ? (row1 - row0 + BM - 1) / BM : 0;
    int incl = nt;
    const int lane = threadIdx.x % kWave;
    const int wave = threadIdx.x / kWave;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int up = __shfl_up(incl, off, kWave);
        if (lane >= off) incl += up;
    }
    if (lane == kWave - 1) wave_tot[wave] = incl;
    __syncthreads();
    int wbase = 0;
    for (int w2 = 0; w2 < wave; ++w2) wbase += wave_tot[w2];
    const int first = wbase + incl - nt;
    for (int i = 0; i < nt; ++i) {
        const int ti = first + i;
        if (ti < max_m_tiles) {  // cannot fail when offsets are consistent with the host's bound
            tile_expert[ti] = e;
            tile_row[ti] = row0 + i * BM;
        }
    }
    if (threadIdx.x == 1023) num_tiles[0] = min(first + nt, max_m_tiles);
}

int launch_tile_map(const int32_t *offsets, int E, int block_m, int32_t *tile_expert, int32_t *tile_row,
                    int32_t *num_tiles, int max_m_tiles, const int32_t *stage_of, int stage, hipStream_t s, int ring_n1, int ring_n2)
{
    ProfScope ps("tile_map", s);
    hipLaunchKernelGGL(tile_map_kernel, dim3(1), dim3(1024), 0, s, offsets, E, block_m, tile_expert, tile_row,
                       num_tiles, max_m_tiles, stage_of, stage, ring_n1, ring_n2);
    MOE_LAUNCH_CHECK("tile_map_kernel");
    return MOE_OK;
}

}  // namespace moe355
