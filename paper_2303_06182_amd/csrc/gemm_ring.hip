// Grouped bf16 expert GEMM on one persistent block per CU:  C = A * B^T (+ bias, ReLU), fp32 accumulation, tiles of
// 32 .. 256 rows (in steps of 32) by 256 columns.
//
// What bounds it: the matrix cores where an expert has rows enough, the stream of the weights where it has few.
// Dynamic gating gives every expert its own number of rows, so the last tile of an expert is rarely full; a tile here
// costs what its rows cost: its 16-row blocks are dealt to the two rows of waves in turn (block 2 i + wm is wave row
// wm's i-th) and the K loop exists once per block count, so a tile of 97 rows runs half the MFMAs of one of 256.
//
// 8 waves, 2 x 4; each owns up to 8 blocks of 16 rows and 4 of 16 columns (v_mfma_f32_16x16x32_bf16, the weights as
// first operand).  Why 16x16x32: it contracts 32 k per accumulator read and write where v_mfma_f32_32x32x16_bf16
// contracts 16; a register-only loop on live data sustains 2.14 PFLOP/s with the former against 1.93 with the latter
// under the chip's power limit.  Why direct-to-LDS: ds_write_b128 moves 64 bytes per clock per CU (measured) where
// ds_read_b128 moves 256, so writing a K tile's 64 KB from registers costs the LDS more time than reading its 192 KB
// of fragments.  Why a ring: a CU takes 64 KB per K tile through a 64-byte-per-clock path -- half the time the MFMAs of
// a full tile need -- so the loads must flow evenly, not in a burst per K tile, and they come from HBM or a remote L2
// slice.  With two 64 KB buffers a load can only be issued in the first half of a K tile to land by its end (measured:
// MFMA pipes 56 % busy; 68 % when every load hits the L2).  Five slots of ONE K step (32 k: 256 + 256 rows of 64 bytes
// = 32 KB; 160 KB in all) let a wave spread its loads over the step, each with two to three steps to land.
//
// Step u multiplies the fragments of slot u mod 5, which were read into registers during step u - 1:
//   1. the MFMAs of row block 0 (their operands landed long ago);
//   2. wait for this wave's LDS reads (all of step u's fragments), on odd steps also for its loads of the next K tile;
//      barrier.  Behind it every wave's fragments of slot u are in registers, so slots u - 1 and u are free, and the
//      next K tile has landed for everybody;
//   3. the other MFMAs; behind them the reads of step u + 1's fragments from slot u + 1 (the four weight fragments into
//      the other register set and block 0 at once, block i in place behind its last MFMA) and the loads of the K tile
//      two ahead, both halves of a 16-row group back to back (the second request finds the line in the L1 or merges
//      with the first), the first half into slot u + 4, the second into slot u + 5 = u: the weights in the even step,
//      the rows in the odd one behind its wait, so that the weights, which come from further away, have longer to land;
//      the other way round in tiles of up to 128 rows, where HBM sets the pace.
//      "At most as many outstanding as the even step issued" is the wait of point 2.
// A slot row is 64 bytes: 16-byte chunk c of row r sits at position c ^ ((r >> 2) & 3), which keeps the 16 lanes x 16
// bytes of a fragment read on 16 different bank groups; the permutation is applied on the global side of the load,
// inside one 64-byte segment.
// Weight row (output column) permutation inside a wave's columns: LDS row 16 * ni + r holds column
// 32 * (ni / 2) + 8 * (r / 4) + 4 * (ni % 2) + r % 4, so that the accumulators of blocks 2p and 2p + 1 of a lane are the
// 8 consecutive columns 32 p + 8 * (lane / 16) ... of token row lane % 16 and leave as one 16-byte store, without a
// trip through LDS (all of which the ring holds).
//
// Weights of 8 or 4 bits (BQ) go to LDS as they are stored and are widened to bf16 in registers, 8 per lane and fragment by
// four v_cvt_scalef32_pk_bf16_* (mxfp4: with the block's scale; e4m3: the expert's scale multiplies the sums), behind the MFMAs
// of the step before theirs, where vector instructions are free; both wave rows widen the same fragments.  A K tile of 256 columns is 16 or 8 KB
// instead of 32, so the rows get seven slots and everything is loaded three K tiles ahead instead of two: what then bounds tiles
// of few rows is the latency of the loads (with two K tiles ahead 128 experts 2048 -> 8192, 64 rows per expert, FFN: e4m3 930 us, now
// 869, mxfp4 861, now 788; with the weights alone, by four waves of their own, four and six ahead 888 and 878: the CU's loads return in
// order).  Full tiles run at 1.35 (e4m3) and 1.40 PFLOP/s (same layer, 512 rows), where bf16 weights reach 1.15: there is half as much to load.
//
// Launch: PERSISTENT, one block per CU.  Workgroups are handed to the 8 XCDs round-robin and each XCD has its own L2,
// so the schedule (ring_schedule, route.hip) gives each a part of the experts' rows of equal cost, or, where that does not
// come out, an eighth of all output tiles.
// The load cursor walks the block's whole sequence of (tile, K tile) pairs, so the first K tiles of the NEXT tile are
// loaded during the last steps of the current one and the epilogue's stores overlap the next tile.
#include <mutex>
#include <type_traits>

#include "gemm_bf16_dev.h"
#include "moe_internal.h"
#include "ring_schedule.h"

namespace moe355 {

namespace {

typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int BM = 256, BN = 256, BK = 64, WN = 4, WTN = BN / WN;
constexpr int NWAVE = 8, THREADS = NWAVE * 64;
constexpr int NSLOT = 5, SLOT_BYTES = (BM + BN) * 64;
constexpr int MI = 8, NI = 4;                              // 16-row and 16-column blocks of a wave, at most
constexpr int AG = BM / 16 / NWAVE, BG = BN / 16 / NWAVE;  // 16-row groups a wave loads per K tile
constexpr int GROUP_M = 4;
// Byte offset past the end of every operand, which stays past it, and below 2^32, when a K tile's offset is added (64 MiB: an
// operand with 65 rows has less a row).  Not closer to 2^32: the loads of rows past a tile's end take longer there (128 experts 2048 ->
// 8192, 1024 skewed rows, FFN in us, 0xf0000000 7135, 0xf8000000 7142, 0xfc000000 7152, 0xfe000000 7201, 0xffe00000 7208; 16 experts, 2048 rows
// 1845, 1847, 1835, 1859, 1860).
constexpr uint32_t kNowhere = 0xfc000000u;

// Quantised weights: seven slots of rows; behind them the weights' K tiles, three or four (a K tile's last read is in its even step, so
// that three do for loads issued in the odd one); behind them mxfp4's block scales in groups of 16 bytes a column (8 K tiles'
// worth, fewer at a tile's end).  Three K tiles lie in three groups at most, as two short groups are never neighbours.
constexpr int Q_SLOTS = 7, Q_AHEAD = 3, Q_SCALES = BN * 16, Q_SCALE_BUFS = 3;
constexpr int q_ring(int bq) { return bq == 8 ? 3 : bq == 4 ? 4 : 0; }
constexpr int q_tile_bytes(int bq) { return bq == 8 ? BN * 64 : bq == 4 ? BN * 32 : 0; }
template <int BQ> struct QuantRaw { typedef u32x2 type; };   // a lane's 8 weights
template <> struct QuantRaw<4> { typedef u32_lds type; };

constexpr int kTurnedRows = 512, kTurnedRowsHeavy = 320, kTurnedExperts = 256;  // see first_k

struct RingTile {
    int row0, row_end, expert, n0;
};

// acc += w * a.  In place, by hand: an accumulator that lives across basic blocks gets a second set of registers from the
// compiler, and 64 copies a step to go with it.  What its hazard handling then no longer sees: the accumulators are
// written by vector instructions at the head of a tile only and read at its end, both padded there; the operands come
// from LDS reads; a register the compiler copies where two blocks of code join is covered by the padding of a step's FIRST.
template <bool FIRST>
__device__ __forceinline__ void mfma_in_place(f32x4 &acc, const bf16x8 &w, const bf16x8 &a)
{
    if constexpr (FIRST)
        asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(w), "v"(a));
    else
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(w), "v"(a));
}
// The same value, in a scalar register, of which the optimiser knows nothing: a chain of tests on such values stays a chain.
__device__ __forceinline__ int opaque(int v)
{
    asm volatile("" : "+s"(v));
    return __builtin_amdgcn_readfirstlane(v);
}

}  // namespace

template <bool RELU, bool RAGGED, int BQ = 0, bool TURNED = false>
__global__ __launch_bounds__(THREADS, 1) void gemm_ring_kernel(GemmParams p)
{
    constexpr bool Q = BQ != 0, B4 = BQ == 4;
    static_assert(!TURNED || (!Q && !RAGGED), "turned: bf16 rows of whole K tiles");
    static_assert(!Q || !RAGGED, "8- and 4-bit weights come in whole K tiles");
    constexpr int SLOT = Q ? BM * 64 : SLOT_BYTES;
    constexpr int SLOTS = Q ? Q_SLOTS : NSLOT, AHEAD = Q ? Q_AHEAD : 2;
    constexpr int QT = q_tile_bytes(BQ), Q_RING = q_ring(BQ), QB = SLOTS * SLOT, QS = QB + Q_RING * QT;  // quantised weights: size of a K tile, LDS offsets of the first and of the block scales
    constexpr int NBL = Q ? QT / 1024 / NWAVE : 0;  // a wave's loads of a K tile of weights
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem_raw[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int K = p.K, KT = (K + BK - 1) / BK;

    // ---- the block's tiles.  XCD x has blocks x, x + 8, ...; its part of the schedule is a list of experts, those with
    // the taller tiles first.  Of one expert, GROUP_M row tiles at a time are walked across all column tiles, the rows fastest,
    // so the tiles an XCD works on together share rows and weights.  A block takes one of every 32 of these tiles, the other
    // way round in every second round, so that the blocks that begin with the taller tiles of a round end with the shorter
    // ones of the next.
    const int n_tiles = (p.N + BN - 1) / BN;
    int x_first, x_last, cut_first, cut_last, x_cap, shared;
    {
        const int32_t *const w = p.ring_words + (blockIdx.x & 7);
        uniform_load2(w + kRingFirst, w + kRingLast, x_first, x_last);
        uniform_load2(w + kRingCut, w + kRingCut + 1, cut_first, cut_last);
        const int caps = uniform_load(w + kRingCap);
        x_cap = (caps >> p.ring_cap_shift) & 15;
        shared = caps >> kRingShared & 1;
    }
    // the experts, 64 at a time, one per lane: row range, tiles along the rows, tiles before it
    int w_base = __builtin_amdgcn_readfirstlane(x_first), w_pos = 0, w_total = 0;
    int w_expert, w_row0, w_row_end, w_cuts, w_excl;
    auto load_window = [&]() __attribute__((always_inline)) {
        w_cuts = 0, w_expert = 0, w_row0 = 0, w_row_end = 0;
        if (w_base + lane < x_last) {
            w_expert = p.ring_list[w_base + lane];
            w_row0 = p.offsets[w_expert], w_row_end = p.offsets[w_expert + 1];
            ring_clip(w_expert, cut_first, cut_last, w_row0, w_row_end);
            w_cuts = (int)((uint32_t)(ring_units(w_row_end - w_row0) + x_cap - 1) / (uint32_t)x_cap);
        }
        int incl = w_cuts;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int up = __shfl_up(incl, off, 64);
            if (lane >= off) incl += up;
        }
        w_excl = (incl - w_cuts) * n_tiles;
        w_total = __builtin_amdgcn_readlane(incl, 63) * n_tiles;
    };
    load_window();
    const int s_blk = blockIdx.x >> 3;
    int pos = s_blk, pos_next = 63 - s_blk;
    if (shared) {  // the one list of all XCDs, at most 64 experts and so one window: an eighth of its tiles each
        const int first = ring_share(w_total, blockIdx.x & 7);
        w_total = ring_share(w_total, (blockIdx.x & 7) + 1);
        pos += first;
        pos_next += first;
    }
    RingTile nx;  // the stream's next tile
    auto next_tile_pos = [&]() __attribute__((always_inline)) -> bool {
        while (pos - w_pos >= w_total) {
            if (w_base + 64 >= x_last) return false;
            w_pos += w_total;
            w_base += 64;
            load_window();
        }
        const int at = pos - w_pos;
        const int src = 63 - __builtin_clzll(__ballot(w_excl <= at && w_cuts > 0));
        nx.expert = __builtin_amdgcn_readlane(w_expert, src);
        const int row0 = __builtin_amdgcn_readlane(w_row0, src), row_end = __builtin_amdgcn_readlane(w_row_end, src);
        const int cuts = __builtin_amdgcn_readlane(w_cuts, src), units = (row_end - row0 + 31) >> 5;
        const int in = at - __builtin_amdgcn_readlane(w_excl, src);
        const int grp = in / (GROUP_M * n_tiles), within = in - grp * (GROUP_M * n_tiles);
        const int gsz = min(GROUP_M, cuts - grp * GROUP_M);
        const int nt = within / gsz, mt = grp * GROUP_M + within - nt * gsz;
        nx.n0 = __builtin_amdgcn_readfirstlane(nt * BN);
        nx.row0 = __builtin_amdgcn_readfirstlane(row0 + 32 * (int)((uint32_t)(units * mt) / (uint32_t)cuts));
        nx.row_end = __builtin_amdgcn_readfirstlane(min(row_end, row0 + 32 * (int)((uint32_t)(units * (mt + 1)) / (uint32_t)cuts)));
        const int after = pos + 64;
        pos = pos_next;
        pos_next = after;
        return true;
    };
    // The K tile a tile begins with: see turned_k.
    // FFN in us, from 0 / turned: 64 experts 1024 -> 4096, 32 even rows 239 / 211, 128 rows 281 / 254, 256 rows 340 / 313, skewed (0.5) 373 / 362;
    // 16 experts 2048 -> 8192, 128 rows 304 / 257; 128 experts, 32 rows 1498 / 1450, 128 rows 1684 / 1648, skewed 1878 / 1823; 128 experts 512 ->
    // 2048, 128 rows 174 / 159; 12 experts 4096 -> 14336, 256 skewed rows 968 / 939.  Other ways to turn (by a hash of expert and column, two or five
    // K tiles a column, the expert alone) are behind by up to 9 %.  Rows of other lengths spread by themselves (1536, 3072, 4000, 6144:
    // within 1 % either way), as do the blocks of quantised weights.  From 512 rows per expert on, 320 with 2^30 weights, the weights'
    // time hides behind the MFMAs and what is left is the rows' lost sharing (128 experts 2048 -> 8192: 384 rows 3005 / 3009, skewed 3123 / 3098, 768 rows 5255 / 5250,
    // skewed 5574 / 5613, 1024 skewed 7288 / 7317; 464 rows, layer 3663 / 3691; 64 experts 1024 -> 4096, 384 rows 443 / 433, 512 rows 519 / 515).  With 256 experts and more the blocks' tiles lie far enough
    // apart (1024 -> 4096, 16 even rows: 192 experts 586 / 557, 256 experts 733 / 733, 400 experts 1210 / 1184, 512 experts 1496 / 1477, skewed 1506 /
    // 1497; 256 experts 2048 -> 2048 712 / 738; 512 experts 512 -> 2048 409 / 416).  An instance of its own: with the place along K in all of them
    // full tiles are 0.7 % slower.
    auto first_k = [&]() __attribute__((always_inline)) -> int {
        if constexpr (!TURNED) return 0;
        return turned_k(nx.expert, nx.n0 / BN & 31, KT);
    };
    if (p.c_zero_row >= 0 && blockIdx.x == 0) {
        // one all-zero row behind the output rows, for the GEMM that reads C as its A (N is a multiple of 8)
        uint16_t *z = static_cast<uint16_t *>(p.C) + (int64_t)p.c_zero_row * p.ldc;
        for (int i = tid * 8; i < p.N; i += THREADS * 8) *reinterpret_cast<uint4 *>(z + i) = make_uint4(0, 0, 0, 0);
    }
    if (!next_tile_pos()) return;

    f32x4 acc[MI][NI];
    const int row16 = lane & 15, kq = lane >> 4;
    // fragment reads: row (block base + row16), chunk position kq ^ ((row16 >> 2) & 3); row block i of wave row wm is
    // block 2 i + wm of the tile
    const int frag_off = row16 * 64 + ((kq ^ ((row16 >> 2) & 3)) << 4);
    const uint8_t *fragA = smem_raw + wm * 1024 + frag_off;
    const uint8_t *fragB = smem_raw + BM * 64 + (wn * WTN) * 64 + frag_off;
    auto read_a = [&](int slot, int block) __attribute__((always_inline)) { return *reinterpret_cast<const bf16x8 *>(fragA + slot * SLOT + block * 2048); };
    auto read_b = [&](int slot, int block) __attribute__((always_inline)) { return *reinterpret_cast<const bf16x8 *>(fragB + slot * SLOT_BYTES + block * 1024); };

    // ---- load stream
    int l_kt = 0, l_k = 0;  // the stream's K tile, and where along K it lies
    bool l_more = true;
    int l_groups = 0;  // row groups of the stream's tile that this wave loads
    int w_slot = 0;    // slot of the first half of the K tile the stream is at
    // Both operands through buffer loads: an offset past the buffer's end costs no memory traffic and fills zeros, which is
    // what rows past a tile's end, columns past N and the chunks past K of the last K tile need.
    const __amdgpu_buffer_rsrc_t bufA = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p.A), 0, (int)kNowhere, 0x00020000);
    __amdgpu_buffer_rsrc_t bufB = bufA;  // the expert's weights
    const __amdgpu_buffer_rsrc_t bufC = __builtin_amdgcn_make_buffer_rsrc(p.C, 0, (int)kNowhere, 0x00020000);
    uint32_t a_voff[AG], b_voff[BG], s_voff = 0;
    const int ld_row = lane >> 2;                         // row inside the 16-row group
    const int ld_chunk = (lane & 3) ^ ((lane >> 4) & 3);  // K chunk this lane fetches for its LDS position
    int b_col[BG];                                        // column of the tile this lane fetches in group g
#pragma unroll
    for (int g = 0; g < BG; ++g) {
        const int rho = (wave * BG + g) * 16 + ld_row;  // LDS row of the tile
        const int x = rho % WTN, xi = x >> 4, xr = x & 15;
        b_col[g] = (rho / WTN) * WTN + 32 * (xi >> 1) + 8 * (xr >> 2) + 4 * (xi & 1) + (xr & 3);
    }
    uint32_t q_lane[BG];  // quantised weights: the lane's 16 bytes of a 1 KB block, rows of 64 / 32 bytes (see read_q)
#pragma unroll
    for (int g = 0; g < BG; ++g)
        q_lane[g] = B4 ? (lane >> 1) * 32 + (((lane & 1) ^ (lane >> 4 & 1)) << 4) : (lane >> 2) * 64 + (((lane & 3) ^ ((2 * g + (lane >> 5)) & 3)) << 4);
    __amdgpu_buffer_rsrc_t bufS = bufA;  // the expert's block scales
    int w_q = 0, w_s = 0;                // the stream's K tile of weights, and its group of block scales, in LDS
    (void)q_lane, (void)bufS, (void)w_q, (void)w_s, (void)s_voff;
    auto set_ptrs = [&]() __attribute__((always_inline)) {
        const RingTile &ti = nx;
        const int slot = p.b_slot ? __builtin_amdgcn_readfirstlane(uniform_load(p.b_slot + ti.expert)) : ti.expert;
        const int rows = __builtin_amdgcn_readfirstlane(ti.row_end - ti.row0);
        l_groups = rows > (8 + wave) * 16 ? 2 : rows > wave * 16 ? 1 : 0;
        bufB = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(static_cast<const uint8_t *>(p.B) + (int64_t)slot * p.strideB * (Q ? 1 : 2)), 0, (int)kNowhere, 0x00020000);
#pragma unroll
        for (int g = 0; g < AG; ++g) {
            const int r = (g * NWAVE + wave) * 16 + ld_row;
            const bool live = ti.row0 + r < ti.row_end;
            int gr = min(ti.row0 + r, ti.row_end - 1);
            if (p.a_rows) gr = p.a_rows[gr];
            a_voff[g] = live ? (uint32_t)gr * (uint32_t)p.lda * 2u + ld_chunk * 16 : kNowhere;
        }
        if constexpr (Q) {
            constexpr int ROWS = B4 ? 32 : 16;  // of a block; N is a multiple of it
#pragma unroll
            for (int g = 0; g < NBL; ++g) {
                const int col = ti.n0 + (wave * NBL + g) * ROWS;
                b_voff[g] = col < p.N ? (uint32_t)(col / ROWS) * (uint32_t)(KT * 1024) + q_lane[g] : kNowhere;
            }
            if constexpr (B4) {
                const int col = ti.n0 + (wave & 3) * 64 + (lane >> 5) * 32;
                bufS = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(p.b_blk_scale + (int64_t)ti.expert * p.stride_blk_scale), 0, (int)kNowhere, 0x00020000);
                s_voff = col < p.N ? (uint32_t)(col >> 5) * (uint32_t)((KT + 7) >> 3) * 512u + (lane & 31) * 16 : kNowhere;
            }
            return;
        }
#pragma unroll
        for (int g = 0; g < BG; ++g)
            b_voff[g] = ti.n0 + b_col[g] < p.N ? (uint32_t)(ti.n0 + b_col[g]) * (uint32_t)p.ldb * 2u + ld_chunk * 16 : kNowhere;
    };
    auto issue = [&](__amdgpu_buffer_rsrc_t buf, uint32_t voff, int h, int lds_off) __attribute__((always_inline)) {
        int slot = w_slot + h;
        if (slot >= SLOTS) slot -= SLOTS;
        if (RAGGED && l_kt * BK + h * 32 + ld_chunk * 8 >= K) voff = kNowhere;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(buf, (lds_void *)(smem_raw + slot * SLOT + lds_off), 16, voff, (TURNED ? l_k : l_kt) * 128 + h * 64, 0, 0);
    };
    auto issue_a = [&](int g, int h) __attribute__((always_inline)) { issue(bufA, a_voff[g], h, (g * NWAVE + wave) * 1024); };
    auto issue_b = [&](int g, int h) __attribute__((always_inline)) { issue(bufB, b_voff[g], h, BM * 64 + (wave * BG + g) * 1024); };
    auto issue_q = [&](int g) __attribute__((always_inline)) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(bufB, (lds_void *)(smem_raw + QB + w_q * QT + (wave * NBL + g) * 1024), 16, b_voff[g], l_kt * 1024, 0, 0);
    };
    auto issue_s = [&]() __attribute__((always_inline)) {  // the block scales of 8 K tiles, with the first of them
        if ((l_kt & 7) == 0) {
            if (wave < 4)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(bufS, (lds_void *)(smem_raw + QS + w_s * Q_SCALES + wave * 1024), 16, s_voff, l_kt * 64, 0, 0);
            w_s = w_s + 1 == Q_SCALE_BUFS ? 0 : w_s + 1;
        }
    };
    auto next_k = [&]() __attribute__((always_inline)) {
        ++l_kt;
        if constexpr (TURNED) l_k = l_k + 1 == KT ? 0 : l_k + 1;
        if constexpr (Q) w_q = w_q + 1 == Q_RING ? 0 : w_q + 1;
        w_slot += 2;
        if (w_slot >= SLOTS) w_slot -= SLOTS;
    };
    auto next_tile = [&]() __attribute__((always_inline)) {  // of the stream: the block's next one
        l_more = next_tile_pos();
        if (l_more) {
            l_kt = 0;
            l_k = first_k();
            set_ptrs();
        } else {
            l_kt = KT - AHEAD;  // past the end: K tiles again, into slots nobody reads
        }
        // lgkmcnt(0): no scalar load is in flight where this joins the K loop, whose waits then count LDS reads only
        __builtin_amdgcn_s_waitcnt(0xc07f);
    };

    // a16[M - 1 + P]: the last row block has a register set per step parity, so that its read for the next step goes
    // out with the first ones and the step's last LDS read is four MFMAs from the step's end
    bf16x8 a16[MI + 1], w16[2][NI];
    int r_slot = 0;  // slot of the step being multiplied
    // Quantised weights: read as they are, widened behind the MFMAs of the step before theirs.
    typename QuantRaw<BQ>::type raw[NI];
    uint32_t sc[NI];                 // a K tile's two scale bytes
    int r_q = 0, r_s = Q_SCALE_BUFS - 1, r_kt = 0;  // the K tile being multiplied
    (void)raw, (void)sc, (void)r_q, (void)r_s, (void)r_kt;
    const int q_row = wn * WTN + 8 * (row16 >> 2) + (row16 & 3);  // column of the lane's operand in block 0; in block ni 32 (ni / 2) + 4 (ni % 2) further
    auto read_q = [&](int tile, int half) __attribute__((always_inline)) {
        // chunk c of row r: e4m3 at c ^ ((r >> 3) & 3) of four, mxfp4 at c ^ ((r >> 3) & 1) of two
        const int at = B4 ? q_row * 32 + ((half ^ (row16 >> 2 & 1)) << 4) + kq * 4 : q_row * 64 + (((2 * half + (kq >> 1)) ^ (row16 >> 2)) << 4) + (kq & 1) * 8;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
            raw[ni] = *reinterpret_cast<const typename QuantRaw<BQ>::type *>(smem_raw + QB + tile * QT + at + (32 * (ni >> 1) + 4 * (ni & 1)) * (B4 ? 32 : 64));
    };
    auto read_scales = [&](int kt) __attribute__((always_inline)) {
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
            sc[ni] = *reinterpret_cast<const u16_lds *>(smem_raw + QS + r_s * Q_SCALES + (q_row + 32 * (ni >> 1) + 4 * (ni & 1)) * 16 + ((kt & 7) << 1));
    };
    auto widen = [&](int set, int ni, int half) __attribute__((always_inline)) {
        u32x4 w = {};
        if constexpr (BQ == 8) {  // every e4m3 value is a bf16 value
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                w[2 * i] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[ni][i], 1.f, false));
                w[2 * i + 1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(raw[ni][i], 1.f, true));
            }
        } else if constexpr (B4) {
            const float scale = __uint_as_float((half ? sc[ni] << 15 : sc[ni] << 23) & 0x7f800000u);  // 2^(byte - 127)
            w[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(raw[ni], scale, 0));
            w[1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(raw[ni], scale, 1));
            w[2] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(raw[ni], scale, 2));
            w[3] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(raw[ni], scale, 3));
        }
        asm volatile("" : "+v"(w));  // here, and not in front of the MFMA that reads it
        w16[set][ni] = __builtin_bit_cast(bf16x8, w);
    };
    // One step of a tile with M row blocks per wave; P: parity.
    auto step = [&](auto parity, auto blocks) __attribute__((always_inline)) {
        constexpr int P = decltype(parity)::value, M = decltype(blocks)::value;
        constexpr int POST = (M - 1) * NI;  // MFMAs behind the barrier
        auto mfma = [&](auto first, int mi, int ni) __attribute__((always_inline)) {
            mfma_in_place<decltype(first)::value>(acc[mi][ni], w16[P][ni], a16[mi == M - 1 ? mi + P : mi]);
        };
        mfma(std::true_type{}, 0, 0);
#pragma unroll
        for (int ni = 1; ni < NI; ++ni) mfma(std::false_type{}, 0, ni);
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        // lgkmcnt(0); odd steps: at most the loads of the even step before may be outstanding, three K tiles ahead also those of
        // the K tile before it
        static_assert(AG == BG, "either operand's loads are as many");
        if (P == 1)
            __builtin_amdgcn_s_waitcnt(0x0070 | (Q ? (BQ == 8 ? 6 + 2 : 5 + 3) : 2 * BG));
        else
            __builtin_amdgcn_s_waitcnt(0xc07f);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        const int nslot = r_slot + 1 == SLOTS ? 0 : r_slot + 1;
        if constexpr (Q) {
            if constexpr (P == 1) {
                r_q = r_q + 1 == Q_RING ? 0 : r_q + 1;
                ++r_kt;
                if constexpr (B4) {
                    if ((r_kt & 7) == 0 && r_kt < KT) r_s = r_s + 1 == Q_SCALE_BUFS ? 0 : r_s + 1;  // behind the last K tile the next tile's group is run_tile's
                    read_scales(r_kt);
                }
            }
            read_q(r_q, P ^ 1);
        } else {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) w16[P ^ 1][ni] = read_b(nslot, ni);
        }
        a16[0] = read_a(nslot, 0);
        a16[M - 1 + (P ^ 1)] = read_a(nslot, M - 1);
        __builtin_amdgcn_sched_barrier(0);
        // the step's loads, the j-th behind MFMA j * POST / 4 of those behind the barrier
        auto loads_at = [&](int at) __attribute__((always_inline)) {
            if constexpr (Q) {
                // one row group of the K tile three ahead; e4m3: the weights in the odd step (three K tiles of them, see above)
                constexpr int LOADS = BQ == 8 ? (P ? 4 : 2) : P ? 2 : 3;
                if constexpr (B4 && P == 0)
                    if (at == 0) issue_s();
#pragma unroll
                for (int j = 0; j < LOADS; ++j)
                    if (j * POST / LOADS == at) {
                        if (j < 2) issue_a(P, j);
                        else issue_q(j - 2);
                    }
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
                    if ((POST > 4 ? POST / 2 + ni * POST / 8 : POST - 1) == at) widen(P ^ 1, ni, P ^ 1);
                return;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (j * POST / 4 == at) {
                    // Up to four blocks a K tile takes as long as HBM takes for its weights, and asking for them in the odd step, one
                    // K tile ahead instead of one and a half, is the faster order (one pair in each step is between).  us per GEMM, 128
                    // experts 2048 -> 8192, before / after: 25 rows per expert 795 / 743 and 771 / 717, 39 rows 780 / 774 and 771 /
                    // 728, 39 skewed 790 / 792 and 773 / 757, 78 rows 826 / 824 and 796 / 773.  With full tiles the same or 1 % slower.
                    if constexpr (M <= 4) {
                        if constexpr (P == 0) issue_a(j >> 1, j & 1);
                        else issue_b(j >> 1, j & 1);
                    } else if constexpr (P == 0) {
                        issue_b(j >> 1, j & 1);
                    } else {
                        // A group past the tile's end would only fill zeros.  Stepping over it pays where the steps are short: the
                        // CU's address unit takes 16 clocks a load, whatever it fetches.
                        if (M > 5 || (j >> 1) < l_groups) issue_a(j >> 1, j & 1);
                    }
                }
        };
#pragma unroll
        for (int mi = 1; mi < M; ++mi) {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
                mfma(std::false_type{}, mi, ni);
                if (ni == NI - 1 && mi < M - 1) a16[mi] = read_a(nslot, mi);
                loads_at((mi - 1) * NI + ni);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        r_slot = nslot;
        __builtin_amdgcn_sched_barrier(0);
    };
    auto epilogue = [&](const RingTile &ti, auto blocks) __attribute__((always_inline)) {
        constexpr int M = decltype(blocks)::value;
        const uint16_t *bias = static_cast<const uint16_t *>(p.bias);
        if (bias) bias += (int64_t)ti.expert * p.strideBias;
        const float b_scale = BQ == 8 && p.b_scale ? __int_as_float(uniform_load(reinterpret_cast<const int32_t *>(p.b_scale) + ti.expert)) : 1.f;
        (void)b_scale;
        const int col_base = ti.n0 + wn * WTN + 8 * kq;
        const uint32_t row_step = 32u * (uint32_t)p.ldc * 2u;  // bytes between two row blocks
        asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");  // see mfma_in_place
#pragma unroll
        for (int mi = 0; mi < M; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) asm volatile("" : "+v"(acc[mi][ni]));  // no accumulator is read before the padding
        auto store_all = [&](auto with_bias) __attribute__((always_inline)) {
            constexpr bool BIAS = decltype(with_bias)::value;
            uint32_t bw[NI / 2][4] = {};
            if constexpr (BIAS) {
#pragma unroll
                for (int pp = 0; pp < NI / 2; ++pp)
                    if (col_base + 32 * pp < p.N) {  // N is a multiple of 8
                        const uint4 bb = *reinterpret_cast<const uint4 *>(bias + col_base + 32 * pp);
                        bw[pp][0] = bb.x, bw[pp][1] = bb.y, bw[pp][2] = bb.z, bw[pp][3] = bb.w;
                    }
            }
            const int row0 = ti.row0 + wm * 16 + row16;
            uint32_t off = (uint32_t)row0 * (uint32_t)p.ldc * 2u + (uint32_t)col_base * 2u;  // the launcher checked that C fits 32 bits
#pragma unroll
            for (int mi = 0; mi < M; ++mi) {
                // the column pairs of a row block back to back: together they fill whole 128-byte lines
#pragma unroll
                for (int pp = 0; pp < NI / 2; ++pp) {
                    uint32_t o[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {  // columns 2q, 2q + 1 of the 8: block 2pp + q / 2, registers 2 (q % 2), + 1
                        float v0 = acc[mi][2 * pp + (q >> 1)][2 * (q & 1)], v1 = acc[mi][2 * pp + (q >> 1)][2 * (q & 1) + 1];
                        if constexpr (BQ == 8) {
                            v0 *= b_scale;
                            v1 *= b_scale;
                        }
                        if constexpr (BIAS) {
                            v0 += __uint_as_float(bw[pp][q] << 16);
                            v1 += __uint_as_float(bw[pp][q] & 0xffff0000u);
                        }
                        o[q] = pack_bf16(v0, v1);
                        if (RELU) o[q] = relu_bf16x2(o[q]);
                    }
                    const bool live = row0 + mi * 32 < ti.row_end && col_base + 32 * pp < p.N;
                    __builtin_amdgcn_raw_buffer_store_b128(u32x4{o[0], o[1], o[2], o[3]}, bufC, live ? off + 64 * pp : kNowhere, 0, 0);
                }
                off += row_step;
            }
        };
        if (bias)
            store_all(std::true_type{});
        else
            store_all(std::false_type{});
    };
    // a tile with M row blocks per wave
    auto run_tile = [&](const RingTile &ti, auto blocks) __attribute__((always_inline)) {
        constexpr int M = decltype(blocks)::value;
#pragma unroll
        for (int mi = 0; mi < M; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[mi][ni][r] = 0.f;
#pragma unroll
        for (int mi = 0; mi < M; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) asm volatile("" : "+v"(acc[mi][ni]));
        asm volatile("s_nop 7");
        // fragments of step 0, an even one (its slot has landed: the barrier before saw to it)
        if constexpr (Q) {
            r_kt = 0;
            r_s = r_s + 1 == Q_SCALE_BUFS ? 0 : r_s + 1;  // a tile begins with a group of block scales of its own
            if constexpr (B4) read_scales(0);
            read_q(r_q, 0);
        } else {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) w16[0][ni] = read_b(r_slot, ni);
        }
#pragma unroll
        for (int mi = 0; mi < M; ++mi) a16[mi] = read_a(r_slot, mi);
        if constexpr (Q) {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) widen(0, ni, 0);
        }
        for (int kt = 0; kt < KT; ++kt) {
            if (kt == KT - AHEAD) next_tile();
            step(std::integral_constant<int, 0>{}, blocks);
            step(std::integral_constant<int, 1>{}, blocks);
            next_k();
        }
        epilogue(ti, blocks);
    };

    // prologue: the stream's first K tiles
    RingTile t = nx;
    l_k = first_k();
    set_ptrs();
#pragma unroll 1
    for (int rep = 0; rep < AHEAD; ++rep) {
        if constexpr (Q) {
            if constexpr (B4) issue_s();
#pragma unroll
            for (int g = 0; g < NBL; ++g) issue_q(g);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) issue_b(j >> 1, j & 1);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            issue_a(j >> 1, j & 1);
        next_k();
    }
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0f70 | (Q ? 2 * (4 + NBL) : 2 * AG + 2 * BG));  // the first K tile has landed: the others' loads are younger
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    while (true) {
        // One block per wave runs as two: with one, a step's loads leave in a burst behind the barrier (25 rows per expert, 128 experts
        // 2048 -> 8192: 768 and 744 us where two blocks take 758 and 740).
        const int blocks = max(2, (t.row_end - t.row0 + 31) >> 5);
#define MOE_RING_CASE(M) if (opaque(blocks) == M) run_tile(t, std::integral_constant<int, M>{})
        MOE_RING_CASE(8);
        MOE_RING_CASE(7);
        MOE_RING_CASE(6);
        MOE_RING_CASE(5);
        MOE_RING_CASE(4);
        MOE_RING_CASE(3);
        MOE_RING_CASE(2);
#undef MOE_RING_CASE
        if (!l_more) break;  // the stream has moved on already
        t = nx;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no LDS write may outlive the block
}

template <bool RELU, bool RAGGED, int BQ = 0, bool TURNED = false>
static int launch_ring_t(const GemmParams &p, hipStream_t s)
{
    const size_t smem = BQ == 0 ? NSLOT * SLOT_BYTES : Q_SLOTS * BM * 64 + q_ring(BQ) * q_tile_bytes(BQ) + (BQ == 4 ? Q_SCALE_BUFS * Q_SCALES : 0);
    auto kern = gemm_ring_kernel<RELU, RAGGED, BQ, TURNED>;
    static std::once_flag once;  // per instantiation, whichever host thread comes first
    static hipError_t setup_rc = hipSuccess;
    std::call_once(once, [&]() {
        setup_rc = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    });
    MOE_HIP_CHECK(setup_rc);
    // the schedule's 8 XCDs of 32 blocks; with fewer CUs the blocks take turns, which is right and not balanced
    hipLaunchKernelGGL(kern, dim3(256), dim3(THREADS), smem, s, p);
    MOE_LAUNCH_CHECK("gemm_ring_kernel");
    return MOE_OK;
}

// For both GEMMs of a layer (N and K swap places): the kernel addresses its operands and C with 32-bit byte offsets from
// one base, ...
bool gemm_ring_addresses(int64_t n_rows, int N, int K)
{
    const int64_t wide = N > K ? N : K;
    return (n_rows + 1) * wide * 2 <= (int64_t)kNowhere && (int64_t)N * K * 2 <= (int64_t)kNowhere;
}
// ... and its load stream is two K tiles ahead.
bool gemm_ring_ok(int64_t n_rows, int N, int K) { return N > BK && K > BK && gemm_ring_addresses(n_rows, N, K); }

// Quantised weights: the load stream is three K tiles ahead and never in the tile after next.
static constexpr int kRingQuantK = 256;
bool gemm_ring_quant_ok(int64_t n_rows, int N, int K)
{
    return N >= kRingQuantK && K >= kRingQuantK && N <= 1 << 22 && K <= 1 << 22 && gemm_ring_ok(n_rows, N, K);  // 16 K is added to kNowhere
}

// wbits: storage of the weights, 8 or 4, else bf16
int launch_gemm_ring(const GemmParams &p, int wbits, bool relu, hipStream_t s)
{
    if (p.chosen) {
        *p.chosen = kChosenRing;
        return MOE_OK;
    }
    if (wbits && p.K < kRingQuantK) {
        set_error("cut tiles over quantised weights need K (%d) of %d at least", p.K, kRingQuantK);
        return MOE_ERR_UNSUPPORTED;
    }
    if (wbits == 8) return relu ? launch_ring_t<true, false, 8>(p, s) : launch_ring_t<false, false, 8>(p, s);
    if (wbits == 4) return relu ? launch_ring_t<true, false, 4>(p, s) : launch_ring_t<false, false, 4>(p, s);
    if (p.K % BK != 0) return relu ? launch_ring_t<true, true>(p, s) : launch_ring_t<false, true>(p, s);
    const int64_t turned_rows = (int64_t)p.num_experts * p.N * p.K >= 1ll << 30 ? kTurnedRowsHeavy : kTurnedRows;
    if (p.K % kTurnedK == 0 && p.M < turned_rows * p.num_experts && p.num_experts < kTurnedExperts)
        return relu ? launch_ring_t<true, false, 0, true>(p, s) : launch_ring_t<false, false, 0, true>(p, s);
    return relu ? launch_ring_t<true, false>(p, s) : launch_ring_t<false, false>(p, s);
}

}  // namespace moe355
