// bf16 MFMA GEMM  C = A * B^T (+ bias, ReLU)  with fp32 accumulation, plain or grouped.
//
// Serves the three dense contractions of the layer: the gate (x * Wg^T, fp32 logits out), and the
// two grouped expert GEMMs (Xp * W1[e]^T with ReLU, H * W2[e]^T), where every expert multiplies
// exactly the rows dynamic gating gave it (paper Sec. 5.1) -- no capacity padding.
//
// Both operands are K-contiguous, so every MFMA operand fragment (8 consecutive bf16 along K for
// one row) is one 16-byte LDS read.  Tile: BM x BN x 64, WM x WN waves of 64 lanes, each wave owns
// a (BM/WM) x (BN/WN) sub-tile made of 32x32 MFMA blocks (v_mfma_f32_32x32x16_bf16).  The weight
// fragment is the MFMA's first operand and the activation fragment the second, so a lane ends up
// with 4 CONSECUTIVE output columns of one output row per group of 4 accumulator registers and
// stores them as one 8-byte (bf16) or 16-byte (fp32) access.
//
// LDS layout: tile rows of 64 bf16 = 128 B = 8 chunks of 16 B; chunk c of row r is stored at
// chunk position c ^ ((r >> 1) & 7).  gfx950's LDS serves a 16-byte-per-lane read 16 consecutive
// lanes (256 B, 64 banks) per clock: the 16 rows such a group reads at one K chunk are 8 even rows
// (first half of the banks) and 8 odd rows (second half), and the swizzle gives each half 8
// different chunk positions, so fragment reads are conflict free (measured: 4 clk per
// ds_read_b128 against 6 clk with an (r & 7) swizzle).
//
// Two K pipelines, chosen per tile shape (template argument STAGES); tiles cut to an expert's rows are gemm_ring.hip's:
//  * direct-to-LDS (small tiles; the gate's with whole K tiles): STAGES LDS stages; K tiles go straight from global
//    memory into LDS (global_load_lds_dwordx4, no register staging; zeros for what lies past K), the loads run STAGES-1 K
//    tiles ahead of the MFMAs and are waited for (vmcnt) only at the barrier that ends an
//    iteration.  Several such blocks share a CU, so one block's load burst and barrier hide
//    behind another block's MFMAs.
//  * register-staged (256- and 128-row tiles, one or two blocks per CU; 32-row tiles where K ends inside a K tile, but for few tiles): measured on gfx950, a
//    vector-memory instruction costs the issuing wave 20-30 clocks of MFMA issue and the CU's
//    address unit 16 clocks, so a K tile's loads issued as one burst stall every wave while the
//    matrix units idle, and with only two 64 KB stages in LDS they cannot be issued late either.
//    Here the loads of K tile i+2 go into registers one by one between the MFMAs of iteration i,
//    are written to the other LDS buffer at the same slot of iteration i+1 and the register is
//    refilled at once: every load has a full iteration to land and the address unit sees an
//    even stream.
// In both, the fragments of K-step ks+1 are read while the MFMAs of K-step ks issue (the
// instruction order is pinned with sched_group_barrier / sched_barrier, otherwise the compiler
// sinks the reads next to their use).
//
// Epilogue (bf16 output): each wave converts a 32-row strip of its tile, parks it in the LDS rows
// only this wave's loads ever fill, and writes it out with 16 bytes per lane, i.e. whole
// contiguous row segments per store instruction; the scattered form (16 bytes per row per
// instruction) cost up to a fifth of a tile's time.
//
// Launch: PERSISTENT.  The grid is (CUs x resident blocks per CU); workgroups are handed to the 8
// XCDs round-robin and each XCD has its own L2, so XCD x walks the contiguous range
// [x*chunk, (x+1)*chunk) of the logical tile list, its blocks taking consecutive entries.  The
// list orders tiles GROUP_M M-tiles at a time across all N-tiles, so the tiles an XCD works on
// together share A rows and B (weight) rows.  The load cursor walks the block's whole sequence of (tile, K tile)
// pairs, so the first K tiles of the NEXT tile are loaded during the last iterations of the current
// one: the pipeline never drains between tiles and the epilogue's stores overlap the next tile.
#include <mutex>

#include "gemm_bf16_dev.h"
#include "moe_internal.h"

namespace moe355 {

bool gemm_ring_ok(int64_t n_rows, int N, int K);
bool gemm_ring_addresses(int64_t n_rows, int N, int K);
bool gemm_ring_quant_ok(int64_t n_rows, int N, int K);
int launch_gemm_ring(const GemmParams &p, int wbits, bool relu, hipStream_t s);

static constexpr int BK = 64;
static constexpr int GROUP_M = 4;
static constexpr int REG_STAGED = 0;  // value of the STAGES template argument that selects the register-staged pipeline
// cache policy of the direct-to-LDS weight loads (template argument NT): plain, non-temporal, or non-temporal for the tiles
// that are their expert's only one
static constexpr int NT_NONE = 0, NT_ALL = 1, NT_SOLE = 2;

// 4-bit weights: whether the block scales of a group of 8 K tiles may still be in flight when it begins, so that the K loop has
// to wait for them.  They are requested as the group before begins, in front of that K tile's operand loads, and the wait
// that ends a K tile leaves those of the newest stages - 2 K tiles in flight: stages - 2 K tiles have to pass.  The shortest group
// is a tile's last one.
__host__ __device__ constexpr bool scales_in_flight(int KT, int stages) { return ((KT - 1) & 7) + 1 < stages - 2; }
bool gemm_bf16_scales_in_flight(int KT, int stages) { return scales_in_flight(KT, stages); }

struct TileInfo {
    int row0, row_end, expert, n0;
    int row_begin;  // the expert's first row (NT_SOLE only)
    int kt0, split;  // plain mode with split K: first K tile and index of this block's K range
};

// BQ: storage of the B operand (the weights).  0: bf16.  8: 8-bit floats (OCP e4m3, one byte per
// element, a tile row of 64 elements = 64 bytes) with one fp32 scale per expert; a fragment is
// widened to bf16 in registers after the LDS read (every e4m3 value is a bf16 value, so the products
// are exact) and the scale multiplies the fp32 accumulators in the epilogue.  4: 4-bit floats (OCP
// e2m1, two per byte, a tile row = 32 bytes) with one power-of-two scale byte (e8m0) per 32
// elements along K; the scale is applied while widening (v_cvt_scalef32_pk_bf16_fp4), the result is
// again exactly a bf16 value.  8 and 4: direct-to-LDS pipeline only.
template <int BM, int BN, int WM, int WN, bool OUT_F32, bool RELU, bool GROUPED, bool KFULL, int MINB, int STAGES,
          int NT = 0, int BQ = 0>
__global__ __launch_bounds__(WM *WN * 64, MINB) void gemm_bf16_kernel(GemmParams p)
{
    constexpr int THREADS = WM * WN * 64;
    constexpr int WTM = BM / WM, WTN = BN / WN;
    constexpr int MI = WTM / 32, NI = WTN / 32;
    constexpr bool B8 = BQ == 8, B4 = BQ == 4;
    static_assert(BQ == 0 || B8 || B4, "B storage: bf16, e4m3 or e2m1");
    constexpr int A_IT = BM * 8 / THREADS, B_IT = (B8 ? BN * 4 : B4 ? BN * 2 : BN * 8) / THREADS;
    constexpr int BROW = B8 ? BK / 2 : B4 ? BK / 4 : BK;  // one B tile row in 16-bit units
    constexpr int BTILE = BN * BROW;                       // one B stage in 16-bit units
    static_assert(!B8 || (BN * 4) % THREADS == 0, "8-bit B tile rows must split evenly over threads");
    static_assert(!B4 || (BN * 2) % THREADS == 0, "4-bit B tile rows must split evenly over threads");
    // bf16 and e4m3 experts: the K loop may go round K from another place (turned_k)
    constexpr bool TURNED = GROUPED && KFULL && !B4 && BM < 256;
    static_assert(WTM % 32 == 0 && WTN % 32 == 0, "wave tile must be made of 32x32 blocks");
    static_assert((BM * 8) % THREADS == 0 && (BN * 8) % THREADS == 0, "tile rows must split evenly over threads");

    extern __shared__ __attribute__((aligned(1024))) uint8_t smem_raw[];
    // STAGES == REG_STAGED selects the register-staged pipeline (two LDS buffers)
    constexpr bool RSTAGE = STAGES == REG_STAGED;
    constexpr int NSTAGE = RSTAGE ? 2 : STAGES;
    uint16_t *sA = reinterpret_cast<uint16_t *>(smem_raw);  // [NSTAGE][BM*64]
    uint16_t *sB = sA + NSTAGE * BM * BK;                   // [NSTAGE][BN*64]
    static_assert(NSTAGE >= 2, "at least two LDS stages");
    static_assert(KFULL || GROUPED || RSTAGE || STAGES == 2, "K that ends inside a K tile: the gate has a two-stage loop of its own");
    static_assert(BQ == 0 || (KFULL && !RSTAGE && GROUPED), "8- and 4-bit weights: grouped direct-to-LDS pipeline, K a multiple of the K tile");

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int K = p.K;
    // Split K (plain mode, skinny problems: the gate GEMM of a decoder step has a tile or two and a long K
    // loop): the K tiles are cut into k_split equal ranges, each a tile of its own whose fp32 result goes to
    // its own slice (range 0 to C, range i > 0 to c_parts + (i - 1) * split_stride); whoever reads C adds the
    // slices in order.
    const int S = (!GROUPED && p.k_split > 1) ? p.k_split : 1;
    const int KT = (K + BK - 1) / BK / S;  // the launcher made sure that S divides the K tile count

    // ---- the block's sequence of tiles -----------------------------------------------------------
    // Tail splitting (grouped GEMM over 256x256 tiles): a persistent launch of G blocks runs
    // ceil(tiles / G) rounds, and when the last round is mostly empty the chip idles for a whole
    // tile time.  So the launch with tail_mode 1 stops at the last whole round, and a second launch
    // (tail_mode 2, a smaller tile shape, more blocks per CU) runs the L leftover tiles as SUB
    // sub-tiles each.  Both compute the same cut from the device-side tile count; the split is taken
    // when the sub-tiles' lower rate still beats one more whole round (measured: a tail of L tiles
    // costs 1.5 to 1.7 x L / G rounds, so it is taken for L < G / 1.8).
    constexpr int PT = 256;                             // parent tile edge
    constexpr int SUB_N = PT / BN > 0 ? PT / BN : 1;    // sub-tiles per parent along N
    constexpr int SUB = (PT / BM > 0 ? PT / BM : 1) * SUB_N;
    const bool tail_sub = GROUPED && p.tail_mode == 2;
    const int n_tiles = (p.N + (tail_sub ? PT : BN) - 1) / (tail_sub ? PT : BN);  // of the tile list's geometry
    const int m_tiles = GROUPED ? p.num_tiles[0] : (p.M + BM - 1) / BM;
    int live = m_tiles * n_tiles * S;          // logical tiles
    int cut = 0;                               // first parent tile of the tail
    if (GROUPED && (p.tail_mode == 1 || p.tail_mode == 2)) {
        const int left = live % p.main_slots;
        cut = (left > 0 && left * 9 < p.main_slots * 5) ? live - left : live;
        live = tail_sub ? (live - cut) * SUB : cut;
    }
    const int chunk = (live + 7) >> 3;         // per XCD
    const int xcd = blockIdx.x & 7;
    const int slots = gridDim.x >> 3;          // blocks per XCD (grid is a multiple of 8)
    int seq = blockIdx.x >> 3;                 // position inside the XCD's chunk
    auto seq_ok = [&](int sq) { return sq < chunk && xcd * chunk + sq < live; };
    // logical tile -> (M tile, N tile): groups of GROUP_M M-tiles (the last group may be narrower),
    // inside a group the M index runs fastest
    auto tile_info = [&](int sq) {
        int lid = xcd * chunk + sq;
        int sub = 0, split = 0;
        if (S > 1) {
            split = lid % S;
            lid /= S;
        }
        if (tail_sub) {
            sub = lid % SUB;
            lid = cut + lid / SUB;
        }
        const int per_group = GROUP_M * n_tiles;
        const int grp = lid / per_group;
        const int within = lid - grp * per_group;
        const int gsz = min(GROUP_M, m_tiles - grp * GROUP_M);
        const int mt = grp * GROUP_M + within % gsz;
        const int nt = within / gsz;
        TileInfo t;
        if (GROUPED) {
            uniform_load2(p.tile_expert + mt, p.tile_row + mt, t.expert, t.row0);
            if constexpr (NT == NT_SOLE)
                uniform_load2(p.offsets + t.expert, p.offsets + t.expert + 1, t.row_begin, t.row_end);
            else
                t.row_end = uniform_load(p.offsets + t.expert + 1);
        } else {
            t.expert = 0;
            t.row0 = mt * BM;
            t.row_end = p.M;
        }
        t.n0 = nt * BN;
        t.kt0 = split * KT;
        t.split = split;
        if (tail_sub) {  // sub-tile (sub / SUB_N, sub % SUB_N) of the 256x256 parent
            t.row0 += (sub / SUB_N) * BM;
            t.n0 = nt * PT + (sub % SUB_N) * BN;
        }
        return t;
    };
    if (GROUPED && !OUT_F32 && p.c_zero_row >= 0 && blockIdx.x == 0 && p.tail_mode != 2) {
        // one all-zero row behind the output rows, for the GEMM that reads C as its A (N is a multiple of 8)
        uint16_t *z = static_cast<uint16_t *>(p.C) + (int64_t)p.c_zero_row * p.ldc;
        for (int i = tid * 8; i < p.N; i += THREADS * 8) *reinterpret_cast<uint4 *>(z + i) = make_uint4(0, 0, 0, 0);
    }
    if (!seq_ok(seq)) return;

    const uint16_t *Ag = static_cast<const uint16_t *>(p.A);
    const uint16_t *Bg0 = static_cast<const uint16_t *>(p.B);

    f32x16 acc[MI][NI];
    auto zero_acc = [&]() {
#pragma unroll
        for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;
    };

    // fragment read offsets: row = (wave tile) + mi*32 + (lane & 31), K chunk = ks*2 + (lane >> 5)
    const int frag_row = lane & 31;
    const int frag_half = lane >> 5;
    const int swz = (lane >> 1) & 7;  // == (row >> 1) & 7 for every row this lane reads

    // MFMAs of one K tile out of LDS stage `cur`.
    // 4-bit weights: the block scales are staged in LDS too, behind the operand stages: two buffers of
    // 16 bytes per weight row of the tile (the scales of 8 consecutive K tiles, two 32-element blocks per K
    // tile), one for the 8 K tiles being computed (c_buf) and one being filled for the 8 after them.
    // (Kept in registers instead, the refill every 8th K tile made the compiler wait for the load it had
    // just issued -- a full memory latency with the whole operand pipeline drained.)
    uint8_t *sS = reinterpret_cast<uint8_t *>(sB + NSTAGE * BTILE);
    static_assert(!B4 || (BN % 64 == 0 && BN / 64 <= THREADS / 64), "a 1 KB scale load of a wave covers 64 of the tile's columns");
    int c_buf = 0;
    auto compute = [&](int cur, int kt) {
        const uint16_t *cA = sA + cur * BM * BK + (wm * WTM + frag_row) * BK;
        const uint16_t *cB = sB + cur * BTILE + (wn * WTN + frag_row) * BROW;
        (void)kt;
        uint32_t sc2[B4 ? NI : 1];
        if constexpr (B4) {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
                sc2[ni] = *reinterpret_cast<const u16_lds *>(sS + c_buf * (BN * 16) + (wn * WTN + ni * 32 + frag_row) * 16 +
                                                             ((kt & 7) << 1));
        }
        (void)sc2;
        bf16x8 af[2][MI], bfr[2][NI];
        auto load_frags = [&](int ks, int set) {
            const int chunkpos = ((ks * 2 + frag_half) ^ swz) << 3;
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
                af[set][mi] = *reinterpret_cast<const bf16x8 *>(cA + mi * 32 * BK + chunkpos);
            if constexpr (B8) {
                // 64-byte rows, 16-byte chunk c of row r at chunk position c ^ ((r >> 2) & 3); the 8
                // bytes of this lane's fragment: chunk ks, half frag_half
                const int bytepos = ((ks ^ ((lane >> 2) & 3)) << 4) + (frag_half << 3);
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) {
                    const u32x2 raw = *reinterpret_cast<const u32x2 *>(reinterpret_cast<const uint8_t *>(cB) +
                                                                       ni * 32 * (BK) + bytepos);
                    const f32x2 f0 = __builtin_amdgcn_cvt_pk_f32_fp8(raw.x, false);
                    const f32x2 f1 = __builtin_amdgcn_cvt_pk_f32_fp8(raw.x, true);
                    const f32x2 f2 = __builtin_amdgcn_cvt_pk_f32_fp8(raw.y, false);
                    const f32x2 f3 = __builtin_amdgcn_cvt_pk_f32_fp8(raw.y, true);
                    const uint4 packed = make_uint4(pack_bf16(f0[0], f0[1]), pack_bf16(f1[0], f1[1]),
                                                    pack_bf16(f2[0], f2[1]), pack_bf16(f3[0], f3[1]));
                    bfr[set][ni] = *reinterpret_cast<const bf16x8 *>(&packed);
                }
            } else if constexpr (B4) {
                // 32-byte rows; this lane's 8 elements of K-step ks are the 4 bytes at ks*8 + half*4, their
                // block scale is byte (kt mod 8)*2 + ks/2 of the row's 16 scale bytes (sc2: the K tile's two)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni) {
                    const uint32_t raw = *reinterpret_cast<const u32_lds *>(reinterpret_cast<const uint8_t *>(cB) +
                                                                            ni * 32 * (BK / 2) + ks * 8 + frag_half * 4);
                    const float scale = __uint_as_float(((sc2[ni] >> ((ks >> 1) << 3)) & 0xffu) << 23);  // 2^(byte - 127)
                    const bf16x2 d0 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(raw, scale, 0);
                    const bf16x2 d1 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(raw, scale, 1);
                    const bf16x2 d2 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(raw, scale, 2);
                    const bf16x2 d3 = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp4(raw, scale, 3);
                    const uint4 packed = make_uint4(*reinterpret_cast<const uint32_t *>(&d0),
                                                    *reinterpret_cast<const uint32_t *>(&d1),
                                                    *reinterpret_cast<const uint32_t *>(&d2),
                                                    *reinterpret_cast<const uint32_t *>(&d3));
                    bfr[set][ni] = *reinterpret_cast<const bf16x8 *>(&packed);
                }
            } else {
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
                    bfr[set][ni] = *reinterpret_cast<const bf16x8 *>(cB + ni * 32 * BK + chunkpos);
            }
        };
        load_frags(0, 0);
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            if (ks + 1 < BK / 16) load_frags(ks + 1, (ks + 1) & 1);
#pragma unroll
            for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[ks & 1][ni], af[ks & 1][mi], acc[mi][ni],
                                                                          0, 0, 0);
            // issue order: one LDS read behind each of the first MFMAs, then the remaining MFMAs
            if (ks + 1 < BK / 16) {
                constexpr int NR = MI + NI, NM = MI * NI;
#pragma unroll
                for (int i = 0; i < (NR < NM ? NR : NM); ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                }
                if (NR > NM) __builtin_amdgcn_sched_group_barrier(0x100, NR - NM, 0);
                if (NM > NR) __builtin_amdgcn_sched_group_barrier(0x008, NM - NR, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // ---- epilogue: acc[mi][ni] holds D[column][row]: lane -> row (lane & 31) of block mi, registers
    // 4g..4g+3 -> columns 8g + 4*(lane >> 5) + 0..3 of block ni
    // A wave tile of 256 accumulator registers lives in the accumulation registers (AGPRs); left to
    // itself the compiler copies all of them to VGPRs at the loop exit and spills.  Reading them one
    // by one where they are used keeps the epilogue at a handful of VGPRs.  The reads are opaque to
    // the compiler's hazard handling, so the MFMA -> accumulator-read distance is padded by hand.
    constexpr bool ACC_IN_AGPR = MI * NI * 16 > 128;
    auto epilogue = [&](const TileInfo &t) {
        if constexpr (ACC_IN_AGPR) {
            asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
        }
        const uint16_t *bias = static_cast<const uint16_t *>(p.bias);
        if (bias) bias += (int64_t)t.expert * p.strideBias;
        const float b_scale = (B8 && p.b_scale) ? __int_as_float(uniform_load(reinterpret_cast<const int32_t *>(p.b_scale) + t.expert)) : 1.f;
        (void)b_scale;
        const bool vec_ok = !OUT_F32 || ((p.ldc & 3) == 0 && (p.N & 3) == 0);
        // The fp32 offsets of this lane's columns are fetched before the first store: a load
        // issued between stores would have to wait for every store before it (memory operations
        // of a wave complete in order), once per group of four columns.
        float bias32[NI][4][4];
        const bool add_bias32 = p.bias_f32 && t.split == 0;
        if (add_bias32) {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int col = t.n0 + wn * WTN + ni * 32 + 8 * g + 4 * (lane >> 5);
#pragma unroll
                    for (int i = 0; i < 4; ++i) bias32[ni][g][i] = (col + i < p.N) ? p.bias_f32[col + i] : 0.f;
                }
            // Added here, under the same condition as the loads and for every row block, not inside the
            // row / column predicates below: a loaded register whose use sits behind a branch that a wave may
            // skip counts as "load still in flight" for the rest of the kernel, and the compiler then waits
            // for ALL loads (vmcnt(0)) before it reuses that register -- at the top of every K iteration.
            if constexpr (!ACC_IN_AGPR) {
#pragma unroll
                for (int mi = 0; mi < MI; ++mi)
#pragma unroll
                    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[mi][ni][r] += bias32[ni][r >> 2][r & 3];
            }
        }
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
            const int row = t.row0 + wm * WTM + mi * 32 + (lane & 31);
            if (row >= t.row_end) continue;
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int col = t.n0 + wn * WTN + ni * 32 + 8 * g + 4 * (lane >> 5);
                    if (col >= p.N) continue;
                    float v[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if constexpr (ACC_IN_AGPR)
                            asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v[i]) : "a"(acc[mi][ni][4 * g + i]));
                        else
                            v[i] = acc[mi][ni][4 * g + i];
                    }
                    if constexpr (B8) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] *= b_scale;
                    }
                    if (bias) {
                        if (col + 3 < p.N) {
                            const uint2 bb = *reinterpret_cast<const uint2 *>(bias + col);
                            v[0] += __uint_as_float(bb.x << 16);
                            v[1] += __uint_as_float(bb.x & 0xffff0000u);
                            v[2] += __uint_as_float(bb.y << 16);
                            v[3] += __uint_as_float(bb.y & 0xffff0000u);
                        } else {
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                if (col + i < p.N) v[i] += from_bf16(bias[col + i]);
                        }
                    }
                    if constexpr (ACC_IN_AGPR) {
                        if (add_bias32) {
#pragma unroll
                            for (int i = 0; i < 4; ++i) v[i] += bias32[ni][g][i];
                        }
                    }
                    if (RELU && OUT_F32) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] = v[i] > 0.f ? v[i] : 0.f;
                    }
                    if (OUT_F32) {
                        float *c = (t.split == 0 ? static_cast<float *>(p.C) : p.c_parts + (int64_t)(t.split - 1) * p.split_stride) +
                                   (int64_t)row * p.ldc + col;
                        if (vec_ok) {
                            *reinterpret_cast<float4 *>(c) = make_float4(v[0], v[1], v[2], v[3]);
                        } else {
#pragma unroll
                            for (int i = 0; i < 4; ++i)
                                if (col + i < p.N) c[i] = v[i];
                        }
                    } else {
                        // bf16 output: N and ldc are multiples of 8 here, so the 4 columns exist
                        uint2 o;
                        o.x = pack_bf16(v[0], v[1]);
                        o.y = pack_bf16(v[2], v[3]);
                        if (RELU) {
                            o.x = relu_bf16x2(o.x);
                            o.y = relu_bf16x2(o.y);
                        }
                        *reinterpret_cast<uint2 *>(static_cast<uint16_t *>(p.C) + (int64_t)row * p.ldc + col) = o;
                    }
                }
            }
        }
    };

    // ---- bf16 epilogue through LDS: a wave turns one 32-row strip of its tile (32 x WTN outputs)
    // into bf16, parks it in LDS and stores it back out with 16 bytes per lane, so a store
    // instruction writes whole contiguous row segments instead of 32 scattered 16-byte pieces.
    // The strip lives in the rows of the just-consumed LDS stage that THIS wave's own loads fill
    // (rows (wave*IT + i)*8..+7), so no other wave ever writes there and no barrier is needed: the
    // wave's own LDS accesses execute in order, all waves finished reading that stage before the
    // last barrier, and the wave's next load into it is issued after the strip's last read returned.
    // 16-byte chunk c of strip row r sits at chunk position c ^ (r mod chunks-per-row).
    constexpr int STRIP_ROW_BYTES = WTN * 2;
    constexpr int STRIP_BYTES = 32 * STRIP_ROW_BYTES;
    constexpr bool STRIP_IN_A = A_IT * 1024 >= STRIP_BYTES;
    constexpr bool STRIP_IN_B = !STRIP_IN_A && B_IT * 1024 >= STRIP_BYTES;
    constexpr bool LDS_EPILOGUE = !OUT_F32 && (KFULL || RSTAGE || GROUPED) && (STRIP_IN_A || STRIP_IN_B);
    auto epilogue_lds = [&](const TileInfo &t, int free_stage) {
        constexpr int CPRW = STRIP_ROW_BYTES / 16;  // chunks per strip row
        constexpr int RPI = 64 / CPRW;              // strip rows one 64-lane access covers
        if constexpr (ACC_IN_AGPR) asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
        uint8_t *stg = reinterpret_cast<uint8_t *>(STRIP_IN_A ? sA + free_stage * BM * BK + wave * A_IT * 8 * BK
                                                             : sB + free_stage * BTILE + wave * B_IT * 8 * BK);
        const uint16_t *bias = static_cast<const uint16_t *>(p.bias);
        if (bias) bias += (int64_t)t.expert * p.strideBias;
        const float b_scale = (B8 && p.b_scale) ? __int_as_float(uniform_load(reinterpret_cast<const int32_t *>(p.b_scale) + t.expert)) : 1.f;
        (void)b_scale;
        const int r = lane & 31;
        const int col_base = t.n0 + wn * WTN;
#pragma unroll
        for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int cl = ni * 32 + 8 * g + 4 * (lane >> 5);  // column inside the strip
                    const int col = col_base + cl;
                    float v[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if constexpr (ACC_IN_AGPR)
                            asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v[i]) : "a"(acc[mi][ni][4 * g + i]));
                        else
                            v[i] = acc[mi][ni][4 * g + i];
                    }
                    if constexpr (B8) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] *= b_scale;
                    }
                    if (bias && col < p.N) {  // N is a multiple of 8 for bf16 output: the 4 columns exist together
                        const uint2 bb = *reinterpret_cast<const uint2 *>(bias + col);
                        v[0] += __uint_as_float(bb.x << 16);
                        v[1] += __uint_as_float(bb.x & 0xffff0000u);
                        v[2] += __uint_as_float(bb.y << 16);
                        v[3] += __uint_as_float(bb.y & 0xffff0000u);
                    }
                    if (p.bias_f32 && col < p.N) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[i] += p.bias_f32[col + i];
                    }
                    uint2 o;
                    o.x = pack_bf16(v[0], v[1]);
                    o.y = pack_bf16(v[2], v[3]);
                    if (RELU) {
                        o.x = relu_bf16x2(o.x);
                        o.y = relu_bf16x2(o.y);
                    }
                    const int pos = (cl >> 3) ^ (r & (CPRW - 1));
                    *reinterpret_cast<uint2 *>(stg + r * STRIP_ROW_BYTES + pos * 16 + ((cl >> 2) & 1) * 8) = o;
                }
            }
#pragma unroll
            for (int j = 0; j < 32 / RPI; ++j) {
                const int rr = j * RPI + lane / CPRW;
                const int ch = lane % CPRW;
                const uint4 val =
                    *reinterpret_cast<const uint4 *>(stg + rr * STRIP_ROW_BYTES + ((ch ^ (rr & (CPRW - 1))) * 16));
                const int row = t.row0 + wm * WTM + mi * 32 + rr;
                const int col = col_base + ch * 8;
                if (row < t.row_end && col < p.N)
                    *reinterpret_cast<uint4 *>(static_cast<uint16_t *>(p.C) + (int64_t)row * p.ldc + col) = val;
            }
        }
    };

    TileInfo t = tile_info(seq);

    if constexpr (KFULL || RSTAGE || GROUPED) {
        // ---- global -> LDS without registers: one global_load_lds_dwordx4 moves 64 lanes x 16 B =
        // 1 KB = 8 tile rows into LDS, lane L landing at byte 16*L of the instruction's LDS base.
        // The base is fixed per instruction, so the swizzle is applied on the global side: the lane
        // that lands in chunk slot (L & 7) of row r fetches K chunk (L & 7) ^ ((r >> 1) & 7).
        // Instruction i of wave w fills rows (w*IT + i)*8 .. +7.
        // Per lane: one 64-bit base per operand (row of instruction 0) plus a 32-bit element offset per
        // instruction -- 64-bit pointers per instruction would not fit the register file next to
        // the accumulators of the largest tile.
        const uint16_t *a_base, *b_base;
        int a_off[A_IT], b_off[B_IT];
        int k_turn = 0;  // the K tile the loads' tile begins with
        int b_rows = 0;  // NT_SOLE: rows of the expert the loads are at
        auto set_ptrs = [&](const TileInfo &ti) {
            if constexpr (TURNED) k_turn = p.turned ? __builtin_amdgcn_readfirstlane(turned_k(ti.expert, B8 ? ti.n0 / BN & 15 : ti.n0 >> 8 & 31, KT)) : 0;
            if constexpr (NT == NT_SOLE) b_rows = __builtin_amdgcn_readfirstlane(ti.row_end - ti.row_begin);
            // weights of expert e sit in slot b_slot[e] of the weight array when experts are buffered
            const uint16_t *Bg = Bg0 + (int64_t)((GROUPED && p.b_slot) ? uniform_load(p.b_slot + ti.expert) : ti.expert) * p.strideB;
            int gr0 = 0, gn0 = 0;
#pragma unroll
            for (int i = 0; i < A_IT; ++i) {
                const int r = (wave * A_IT + i) * 8 + (lane >> 3);
                const int kc = (lane & 7) ^ ((r >> 1) & 7);
                int gr = min(ti.row0 + r, ti.row_end - 1);  // rows past the end repeat the last one ...
                if (GROUPED && p.a_zero_row >= 0 && ti.row0 + r >= ti.row_end) gr = p.a_zero_row;  // ... or read zeros
                // dispatch fused into the load: the rows of the expert's batch are gathered straight
                // from the token array (the launcher checked that rows * lda fits 31 bits)
                if (GROUPED && p.a_rows) gr = p.a_rows[gr];
                if (i == 0) {
                    gr0 = gr;
                    a_base = Ag + (int64_t)gr * p.lda + ti.kt0 * BK;
                }
                a_off[i] = (gr - gr0) * (int)p.lda + kc * 8;
            }
            if constexpr (B8) {
                // one instruction = 1 KB = 16 rows of 64 bytes: lane L lands in row (L >> 2), chunk slot
                // (L & 3) and fetches K chunk (L & 3) ^ ((row >> 2) & 3).  In memory that 1 KB block is
                // contiguous and the blocks of a 16-row group follow each other along K (the
                // quantiser's layout), so the offsets are those of the group; they are in bytes,
                // carried as half as many 16-bit units.
                const uint8_t *Bg8 = reinterpret_cast<const uint8_t *>(Bg0) +
                                     (int64_t)((GROUPED && p.b_slot) ? uniform_load(p.b_slot + ti.expert) : ti.expert) * p.strideB;
                const int group_bytes = (K / BK) * 1024;  // one 16-row group over the whole of K
                const int last_group = p.N / 16 - 1;       // groups past the end repeat the last one
#pragma unroll
                for (int i = 0; i < B_IT; ++i) {
                    const int r = (wave * B_IT + i) * 16 + (lane >> 2);
                    const int kc = (lane & 3) ^ ((r >> 2) & 3);
                    const int grp = min((ti.n0 + r) >> 4, last_group);
                    if (i == 0) {
                        gn0 = grp;
                        b_base = reinterpret_cast<const uint16_t *>(Bg8 + (int64_t)grp * group_bytes);
                    }
                    b_off[i] = ((grp - gn0) * group_bytes + (r & 15) * 64 + kc * 16) / 2;
                }
            } else if constexpr (B4) {
                // one instruction = 1 KB = 32 rows of 32 bytes: lane L lands in row (L >> 1), 16-byte half
                // (L & 1); in memory that 1 KB block is contiguous and the blocks of a 32-row group follow
                // each other along K (the quantiser's layout)
                const uint8_t *Bg4 = reinterpret_cast<const uint8_t *>(Bg0) +
                                     (int64_t)((GROUPED && p.b_slot) ? uniform_load(p.b_slot + ti.expert) : ti.expert) * p.strideB;
                const int group_bytes = (K / BK) * 1024;
                const int last_group = p.N / 32 - 1;
#pragma unroll
                for (int i = 0; i < B_IT; ++i) {
                    const int r = (wave * B_IT + i) * 32 + (lane >> 1);
                    const int grp = min((ti.n0 + r) >> 5, last_group);
                    if (i == 0) {
                        gn0 = grp;
                        b_base = reinterpret_cast<const uint16_t *>(Bg4 + (int64_t)grp * group_bytes);
                    }
                    b_off[i] = ((grp - gn0) * group_bytes + (r & 31) * 32 + (lane & 1) * 16) / 2;
                }
            } else {
#pragma unroll
                for (int i = 0; i < B_IT; ++i) {
                    const int r = (wave * B_IT + i) * 8 + (lane >> 3);
                    const int kc = (lane & 7) ^ ((r >> 1) & 7);
                    const int gn = min(ti.n0 + r, p.N - 1);
                    if (i == 0) {
                        gn0 = gn;
                        b_base = Bg + (int64_t)gn * p.ldb + ti.kt0 * BK;
                    }
                    b_off[i] = (gn - gn0) * p.ldb + kc * 8;
                }
            }
        };
        auto turn = [&](int kt) {
            if constexpr (!TURNED) return kt;
            kt += k_turn;
            return kt >= KT ? kt - KT : kt;
        };
        auto issue = [&](int tile, int buf) {
            const int kt = turn(tile);
            if constexpr (!KFULL) {
                if (kt == KT - 1) {  // uniform: K ends inside this K tile, the lanes whose chunk lies past it load zeros
                    auto inside = [&](const uint16_t *at, int row) {
                        return kt * BK + (((lane & 7) ^ (((row + (lane >> 3)) >> 1) & 7)) << 3) < K ? at : chunk_of_zeros;
                    };
#pragma unroll
                    for (int i = 0; i < A_IT; ++i) {
                        const int r = (wave * A_IT + i) * 8;
                        __builtin_amdgcn_global_load_lds((const glb_void *)inside(a_base + (a_off[i] + kt * BK), r),
                                                         (lds_void *)(sA + (buf * BM + r) * BK), 16, 0, 0);
                    }
#pragma unroll
                    for (int i = 0; i < B_IT; ++i) {
                        const int r = (wave * B_IT + i) * 8;
                        __builtin_amdgcn_global_load_lds((const glb_void *)inside(b_base + (b_off[i] + kt * BK), r),
                                                         (lds_void *)(sB + (buf * BN + r) * BK), 16, 0, 0);
                    }
                    return;
                }
            }
#pragma unroll
            for (int i = 0; i < A_IT; ++i)
                __builtin_amdgcn_global_load_lds((const glb_void *)(a_base + (a_off[i] + kt * BK)),
                                                 (lds_void *)(sA + buf * BM * BK + (wave * A_IT + i) * 8 * BK), 16, 0, 0);
            if (NT == NT_ALL || (NT == NT_SOLE && b_rows <= BM)) {
#pragma unroll
                for (int i = 0; i < B_IT; ++i)
                    __builtin_amdgcn_global_load_lds((const glb_void *)(b_base + (b_off[i] + kt * (BQ != 0 ? 512 : BK))),
                                                     (lds_void *)(sB + buf * BTILE + (wave * B_IT + i) * 8 * BK), 16, 0, 2);
            } else {
#pragma unroll
                for (int i = 0; i < B_IT; ++i)
                    __builtin_amdgcn_global_load_lds((const glb_void *)(b_base + (b_off[i] + kt * (BQ != 0 ? 512 : BK))),
                                                     (lds_void *)(sB + buf * BTILE + (wave * B_IT + i) * 8 * BK), 16, 0, 0);
            }
        };
        // The loads run STAGES-1 K tiles ahead of the MFMAs along the block's whole sequence of
        // (tile, K tile) pairs, so the pipeline never drains between tiles and an epilogue's stores
        // overlap the next tile's first iterations.  Every call issues the same number of loads
        // (past the end of the sequence it re-reads the last K tile into a stage nobody will use),
        // which keeps the vmcnt arithmetic fixed: "at most (STAGES-2) stages' loads outstanding"
        // means the K tile needed next has landed.
        // The barrier between iterations is the bare s_barrier: __syncthreads() would add a full
        // vmcnt(0) wait (it fences the outstanding LDS-bound loads), which serialises the stages.
        // What the barrier must order is covered explicitly: (1) this wave's own global->LDS loads
        // of the stage read next have landed -- the s_waitcnt vmcnt just before it; (2) this
        // wave's LDS reads of the stage overwritten next have returned -- every fragment read is
        // consumed by an MFMA issued before the barrier, and an MFMA does not issue before its
        // operands arrived.
        auto stage_barrier = [&]() {
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            __builtin_amdgcn_sched_barrier(0);
        };
        constexpr int LPS = A_IT + B_IT;             // load instructions per wave per stage
        if constexpr (RSTAGE) {
            // ---- register-staged pipeline.  A vector-memory instruction costs the issuing wave
            // about one MFMA slot and the CU's address unit 16 clocks, so the loads of a K tile
            // must neither come as one burst (every wave stalls in the queue while the matrix
            // units idle) nor late (two LDS buffers leave no slack for their latency).  Here the
            // LPS loads of K tile i+2 go into registers, one behind every (MFMAs per K tile / LPS)-th
            // MFMA of iteration i; one iteration later, at the same slot, the register is written
            // to the LDS buffer of tile i+1 (ds_write_b128, 1 KB contiguous per wave instruction)
            // and immediately refilled.  Every load has a whole iteration to land, the address unit
            // sees an even stream, and the LDS buffer written in an iteration is the one nobody
            // reads until the barrier that ends it.
            constexpr int KS = BK / 16, NM = MI * NI, NR = MI + NI, TM = KS * NM;
            int l_seq = seq, l_kt = 0;
            bool l_more = true;
            set_ptrs(t);
            uint4 R[LPS];
            // K that ends inside the last K tile (KFULL false; K is a multiple of 8): there a lane whose chunk lies past the
            // end loads the K tile's first chunk instead and writes zeros, for both operands, so that not even a NaN of
            // the neighbouring row can reach a sum.
            const int tail_chunks = (K & (BK - 1)) / 8;  // valid chunks of the last K tile
            bool put_tail = false;                       // R holds the last K tile
            auto chunk_of = [&](int i) {                 // the K chunk this lane fetches with load i (see set_ptrs)
                const int g = i < A_IT ? wave * A_IT + i : wave * B_IT + (i - A_IT);
                return (lane & 7) ^ ((g * 4 + (lane >> 4)) & 7);
            };
            auto gload = [&](int i) -> uint4 {
                int ko = turn(l_kt) * BK;
                if (!KFULL && l_kt == KT - 1 && chunk_of(i) >= tail_chunks) ko -= chunk_of(i) * 8;
                const uint16_t *g = i < A_IT ? a_base + (a_off[i] + ko) : b_base + (b_off[i - A_IT] + ko);
                return *reinterpret_cast<const uint4 *>(g);
            };
            auto lds_put = [&](int buf, int i, uint4 v) {
                if (!KFULL && put_tail && chunk_of(i) >= tail_chunks) v = make_uint4(0, 0, 0, 0);
                uint16_t *d = i < A_IT ? sA + buf * BM * BK + (wave * A_IT + i) * 8 * BK
                                       : sB + buf * BTILE + (wave * B_IT + (i - A_IT)) * 8 * BK;
                *reinterpret_cast<uint4 *>(d + lane * 8) = v;
            };
            auto advance = [&]() {
                if (!KFULL) put_tail = l_kt == KT - 1;
                if (l_more && ++l_kt == KT) {
                    if (seq_ok(l_seq + slots)) {
                        l_seq += slots;
                        l_kt = 0;
                        set_ptrs(tile_info(l_seq));
                    } else {
                        l_more = false;
                        l_kt = KT - 1;  // past the end: re-read the last K tile, never used
                    }
                }
            };
            bf16x8 af[2][MI], bfr[2][NI];
            auto read_one = [&](int buf, int ks, int set, int m) {
                const int chunkpos = ((ks * 2 + frag_half) ^ swz) << 3;
                if (m < MI)
                    af[set][m] = *reinterpret_cast<const bf16x8 *>(sA + buf * BM * BK + (wm * WTM + frag_row + m * 32) * BK +
                                                                   chunkpos);
                else
                    bfr[set][m - MI] = *reinterpret_cast<const bf16x8 *>(
                        sB + buf * BTILE + (wn * WTN + frag_row + (m - MI) * 32) * BK + chunkpos);
            };
            // the ds_writes of this iteration must be complete before anyone reads the buffer
            auto rs_sync = [&]() {
                __builtin_amdgcn_sched_barrier(0);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
            };
            // One K tile out of LDS buffer cur; the instruction order is pinned MFMA by MFMA.
            auto compute_rs = [&](int cur) {
                const int nxt = cur ^ 1;
#pragma unroll
                for (int m = 0; m < NR; ++m) read_one(cur, 0, 0, m);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
                    for (int m = 0; m < NM; ++m) {
                        if (ks + 1 < KS) {  // fragment f of the next K-step is read behind MFMA f * NM / NR
#pragma unroll
                            for (int f = 0; f < NR; ++f)
                                if (f * NM / NR == m) read_one(cur, ks + 1, (ks + 1) & 1, f);
                        }
                        const int mi = m / NI, ni = m % NI;
                        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[ks & 1][ni], af[ks & 1][mi],
                                                                              acc[mi][ni], 0, 0, 0);
                        const int gm = ks * NM + m;
#pragma unroll
                        for (int i = 0; i < LPS; ++i) {
                            if ((i * TM + TM / 2) / LPS == gm) {  // slot i sits behind MFMA number (i + 1/2) * TM / LPS
                                lds_put(nxt, i, R[i]);
                                R[i] = gload(i);
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                advance();
                rs_sync();
            };
            // prologue: K tile 0 -> LDS buffer 0, K tile 1 -> registers
#pragma unroll
            for (int i = 0; i < LPS; ++i) R[i] = gload(i);
            advance();
#pragma unroll
            for (int i = 0; i < LPS; ++i) lds_put(0, i, R[i]);
#pragma unroll
            for (int i = 0; i < LPS; ++i) R[i] = gload(i);
            advance();
            rs_sync();
            // (Letting the waves whose rows all lie past the end of an expert's batch skip their MFMAs
            // makes such a tile 13 % shorter, but the CUs of an XCD then drift apart, share less of the
            // weight panels in L2, and the launch fetches 45 % more from HBM: slower overall.)
            int cur = 0;
            while (true) {
                zero_acc();
                for (int kt = 0; kt < KT; ++kt) {
                    compute_rs(cur);
                    cur ^= 1;
                }
                if constexpr (LDS_EPILOGUE)
                    epilogue_lds(t, cur ^ 1);  // the buffer the last K tile was read from
                else
                    epilogue(t);
                seq += slots;
                if (!seq_ok(seq)) break;
                t = tile_info(seq);
            }
            return;
        }
        constexpr int WAITN = STAGES >= 2 ? (STAGES - 2) * LPS : 0;
        // s_waitcnt vmcnt(WAITN), through the builtin and not as inline assembly: the compiler's own wait-count
        // bookkeeping reads the builtin and then knows that every older load has landed.  It cannot see into
        // inline assembly; with that, a register load left over from an epilogue counted as still in flight
        // and the compiler drained the whole load pipeline (vmcnt(0)) at the top of every K iteration.
        // Encoding: vmcnt in bits 3:0 and 15:14, expcnt (bits 6:4) and lgkmcnt (bits 11:8) left at "no wait".
        auto wait_loads = [&]() {
            static_assert(WAITN >= 0 && WAITN < 64, "vmcnt is a 6-bit counter");
            constexpr int kWaitImm = (WAITN & 15) | ((WAITN >> 4) << 14) | (7 << 4) | (15 << 8);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_waitcnt(kWaitImm);
            asm volatile("" ::: "memory");
        };
        int l_seq = seq, l_kt = 0, l_stage = 0;
        bool l_more = true;
        set_ptrs(t);
        auto issue_next = [&]() {
            issue(l_kt, l_stage);
            l_stage = (l_stage + 1 == STAGES) ? 0 : l_stage + 1;
            if (l_more && ++l_kt == KT) {
                if (seq_ok(l_seq + slots)) {
                    l_seq += slots;
                    l_kt = 0;
                    set_ptrs(tile_info(l_seq));
                } else {
                    l_more = false;
                    l_kt = KT - 1;
                }
            }
        };
        // 4-bit weights: the scale bytes run one group of 8 K tiles ahead of the MFMAs, across tile borders.
        // One load instruction per wave fills 64 rows x 16 bytes of the buffer: lane L fetches the 16 bytes
        // of row 64 * wave + L (row group 2 * wave + L / 32 of the tile, row L % 32 of that group's 512-byte
        // block).  These loads are older than the operand loads issued after them, and loads complete in
        // order, so the per-iteration vmcnt wait covers them once enough iterations have passed (scales_in_flight).
        int s_seq = seq, s_grp = 0, s_buf = 0;
        const uint8_t *s_lane = nullptr;
        const int s_groups = (KT + 7) >> 3;  // 16-byte scale groups per weight row
        const bool s_drain = scales_in_flight(KT, STAGES);
        (void)s_drain;
        auto scale_tile = [&]() {
            const TileInfo ts = tile_info(s_seq);
            const int rg = min((ts.n0 + wave * 64 + (lane >> 5) * 32) >> 5, p.N / 32 - 1);
            s_lane = p.b_blk_scale + (int64_t)ts.expert * p.stride_blk_scale + (int64_t)rg * s_groups * 512 + (lane & 31) * 16;
        };
        auto issue_scales = [&]() {
            if constexpr (B4) {
                if (BN / 64 == THREADS / 64 || __builtin_amdgcn_readfirstlane(wave) < BN / 64)
                    __builtin_amdgcn_global_load_lds((const glb_void *)(s_lane + s_grp * 512),
                                                     (lds_void *)(sS + s_buf * (BN * 16) + wave * 1024), 16, 0, 0);
                s_buf ^= 1;
                if (++s_grp == s_groups) {  // on to the next tile of this block, if there is one
                    s_grp = 0;
                    if (seq_ok(s_seq + slots)) {
                        s_seq += slots;
                        scale_tile();
                    }
                }
            }
        };
        if constexpr (B4) {
            scale_tile();
            issue_scales();
            issue_scales();
        }
#pragma unroll
        for (int i = 0; i < STAGES - 1; ++i) issue_next();
        wait_loads();
        stage_barrier();
        int stage = 0;
        while (true) {
            zero_acc();
            for (int kt = 0; kt < KT; ++kt) {
                if constexpr (B4) {
                    if ((kt & 7) == 0 && (kt > 0 || seq != (int)(blockIdx.x >> 3))) {  // a new group of 8 K tiles
                        if (s_drain) {
                            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                            stage_barrier();
                        }
                        c_buf ^= 1;
                        issue_scales();  // into the buffer of the group just finished
                    }
                }
                issue_next();  // into the stage the previous iteration computed from
                compute(stage, kt);
                wait_loads();
                stage_barrier();
                stage = (stage + 1 == STAGES) ? 0 : stage + 1;
            }
            if constexpr (LDS_EPILOGUE)
                epilogue_lds(t, stage == 0 ? STAGES - 1 : stage - 1);  // the stage the last K tile was read from
            else
                epilogue(t);
            seq += slots;
            if (!seq_ok(seq)) break;
            t = tile_info(seq);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no LDS write may outlive the block
    } else {
        // ---- the gate with K no multiple of the K tile: stage through registers so the tail can be zero filled.
        // chunk c = tid + i*THREADS; row = c >> 3, kc = c & 7
        const int kc = tid & 7;
        while (true) {
            const uint16_t *a_ptr[A_IT];
            const uint16_t *b_ptr[B_IT];
            int a_lds[A_IT], b_lds[B_IT];
#pragma unroll
            for (int i = 0; i < A_IT; ++i) {
                const int r = (tid + i * THREADS) >> 3;
                const int gr = min(t.row0 + r, t.row_end - 1);
                a_ptr[i] = Ag + (int64_t)gr * p.lda + kc * 8;
                a_lds[i] = r * BK + ((kc ^ ((r >> 1) & 7)) << 3);
            }
#pragma unroll
            for (int i = 0; i < B_IT; ++i) {
                const int r = (tid + i * THREADS) >> 3;
                const int gn = min(t.n0 + r, p.N - 1);
                b_ptr[i] = Bg0 + (int64_t)gn * p.ldb + kc * 8;
                b_lds[i] = r * BK + ((kc ^ ((r >> 1) & 7)) << 3);
            }
            uint4 a_reg[A_IT], b_reg[B_IT];
            auto load_global = [&](int kt) {
                const int k0 = (t.kt0 + kt) * BK;
                const bool ok = k0 + kc * 8 < K;
#pragma unroll
                for (int i = 0; i < A_IT; ++i)
                    a_reg[i] = ok ? *reinterpret_cast<const uint4 *>(a_ptr[i] + k0) : make_uint4(0, 0, 0, 0);
#pragma unroll
                for (int i = 0; i < B_IT; ++i)
                    b_reg[i] = ok ? *reinterpret_cast<const uint4 *>(b_ptr[i] + k0) : make_uint4(0, 0, 0, 0);
            };
            auto store_lds = [&](int buf) {
#pragma unroll
                for (int i = 0; i < A_IT; ++i) *reinterpret_cast<uint4 *>(sA + buf * BM * BK + a_lds[i]) = a_reg[i];
#pragma unroll
                for (int i = 0; i < B_IT; ++i) *reinterpret_cast<uint4 *>(sB + buf * BN * BK + b_lds[i]) = b_reg[i];
            };
            zero_acc();
            load_global(0);
            store_lds(0);
            __syncthreads();
            for (int kt = 0; kt < KT; ++kt) {
                const int cur = kt & 1;
                if (kt + 1 < KT) load_global(kt + 1);
                compute(cur, kt);
                if (kt + 1 < KT) store_lds(cur ^ 1);
                __syncthreads();
            }
            epilogue(t);
            seq += slots;
            if (!seq_ok(seq)) break;
            t = tile_info(seq);
        }
    }
}

template <int BM, int BN, int WM, int WN, bool OUT_F32, bool RELU, bool GROUPED, bool KFULL, int MINB, int STAGES,
          int NT = 0, int BQ = 0>
static int launch_k(const GemmParams &p_in, int num_cus, hipStream_t s, int *main_grid)
{
    GemmParams p = p_in;
    if (p.chosen) {
        *p.chosen = BM * 10000 + BN * 10 + STAGES;
        return MOE_OK;
    }
    const int n_tiles = ceil_div(p.N, BN);
    const int m_tiles = GROUPED ? p.max_m_tiles : ceil_div(p.M, BM);
    if (m_tiles <= 0 || n_tiles <= 0) return MOE_OK;
    const size_t smem = (size_t)(STAGES == REG_STAGED ? 2 : STAGES) * (BM + (BQ == 8 ? BN / 2 : BQ == 4 ? BN / 4 : BN)) * BK * sizeof(uint16_t) +
                        (BQ == 4 ? 2 * BN * 16 : 0);  // 4-bit weights: two buffers of block scales
    // FFN in us, K loops from 0 / turned, 32x128 tiles: 128 experts 2048 -> 8192, 2 rows per expert 1357 / 1282, skewed (0.8) 974 / 946; 64
    // experts 1024 -> 4096, 4 rows 200 / 162, half idle 112 / 103; 16 experts 2048 -> 8192, 8 rows 233 / 196; 256 experts 512 -> 2048, 16 rows
    // 235 / 203; 64x128: 64 experts 1024 -> 4096, 40 rows 234 / 203; 128x128: 16 experts 2048 -> 8192, 40 rows 266 / 202, 100 rows 276 / 221, 8
    // experts, 192 rows 195 / 178; from some 256 rows on either way (8 experts, 400 rows 302 / 306, skewed 309 / 304).  With 512 experts 1024 -> 4096
    // 1385 / 1381, 512 -> 2048 331 / 334.
    // e4m3, 32x128 tiles: 128 experts 2048 -> 8192, 2 rows 697 / 669, skewed 499 / 489; 64 experts 1024 -> 4096, 4 rows 104 / 92, 16 rows 119 / 105;
    // 16 experts 2048 -> 8192, 8 rows 125 / 111, 32 rows 138 / 117; 512 experts 1024 -> 4096, 4 rows 718 / 686; 64 rows within 1 %.  Not with few columns
    // (64 experts 512 -> 2048, whose second GEMM has 512, 4 rows 35.2 / 36.3; 48 experts 1024 -> 1024 27.2 / 27.8).
    p.turned = GROUPED && (BQ == 8 ? p.K % kTurnedK8 == 0 && p.N >= 2048
                                   : p.K % kTurnedK == 0 && p.M < 256ll * p.num_experts && p.num_experts < 384);
    auto kern = gemm_bf16_kernel<BM, BN, WM, WN, OUT_F32, RELU, GROUPED, KFULL, MINB, STAGES, NT, BQ>;
    // per instantiation, once, whichever host thread comes first: the LDS size attribute and the occupancy
    static std::once_flag once;
    static int blocks_per_cu = 0;
    static hipError_t setup_rc = hipSuccess;
    std::call_once(once, [&]() {
        setup_rc = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)smem);
        int occ = 0;
        if (setup_rc == hipSuccess) setup_rc = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kern, WM * WN * 64, smem);
        blocks_per_cu = occ < 1 ? 1 : (occ > 8 ? 8 : occ);
    });
    MOE_HIP_CHECK(setup_rc);
    // persistent grid: every resident slot of the chip, but never more blocks than upper-bound tiles
    int64_t grid = (int64_t)num_cus * blocks_per_cu;
    int64_t tiles = (int64_t)m_tiles * n_tiles;
    if (!GROUPED && p.k_split > 1) {
        if (ceil_div(p.K, BK) % p.k_split != 0) {
            set_error("split K: %d does not divide the %d K tiles", p.k_split, ceil_div(p.K, BK));
            return MOE_ERR_INVALID_ARG;
        }
        tiles *= p.k_split;
    }
    if (p.tail_mode == 2) {
        // max_m_tiles counts 256-row parents; at most (main_slots * 5 - 1) / 9 of the parent tiles are left over
        p.main_slots = *main_grid;
        const int64_t parents = (int64_t)m_tiles * ceil_div(p.N, 256);
        const int64_t left_max = ((int64_t)p.main_slots * 5 - 1) / 9;
        tiles = (parents < left_max ? parents : left_max) * ((256 / BM) * (256 / BN));
        if (tiles <= 0) return MOE_OK;
    }
    if (p.tail_mode == 1) {  // a round is the whole chip, also where the grid is smaller
        p.main_slots = (int)grid;
        *main_grid = (int)grid;
    }
    if (grid > tiles) grid = tiles;
    grid = align_up(grid, 8);
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(WM * WN * 64), smem, s, p);
    MOE_LAUNCH_CHECK("gemm_bf16_kernel");
    return MOE_OK;
}

template <int BM, int BN, int WM, int WN, bool OUT_F32, bool RELU, bool GROUPED, int MINB, int STAGES = 2>
static int launch_one(const GemmParams &p, int num_cus, hipStream_t s, int *main_grid = nullptr)
{
    // K a multiple of the K tile: pipelined main loop without a tail predicate; else the register-staged
    // pipeline zero-fills the last K tile, and the gate's shapes run a plain two-stage loop
    return (p.K % BK == 0)
               ? launch_k<BM, BN, WM, WN, OUT_F32, RELU, GROUPED, true, MINB, STAGES>(p, num_cus, s, main_grid)
               : launch_k<BM, BN, WM, WN, OUT_F32, RELU, GROUPED, false, MINB, STAGES == REG_STAGED ? REG_STAGED : 2>(p, num_cus, s, main_grid);
}

// grouped GEMM on the direct-to-LDS pipeline, bf16 (BQ = 0), 8-bit (8) or 4-bit (4) weights.  K that ends inside a K tile: bf16 only, and
// not for 32-row tiles in two stages, which are register-staged there.
template <int BM, int BN, int WM, int WN, int MINB, int STAGES, int NT, int BQ>
static int launch_grouped_dtl(const GemmParams &p, bool relu, int num_cus, hipStream_t s)
{
    if (p.K % BK != 0) {
        if constexpr (BQ == 0 && (BM > 32 || STAGES > 2))
            return relu ? launch_k<BM, BN, WM, WN, false, true, true, false, MINB, STAGES, NT>(p, num_cus, s, nullptr)
                        : launch_k<BM, BN, WM, WN, false, false, true, false, MINB, STAGES, NT>(p, num_cus, s, nullptr);
        set_error("%dx%d tiles need K (%d) to be a multiple of %d", BM, BN, p.K, BK);
        return MOE_ERR_UNSUPPORTED;
    }
    return relu ? launch_k<BM, BN, WM, WN, false, true, true, true, MINB, STAGES, NT, BQ>(p, num_cus, s, nullptr)
                : launch_k<BM, BN, WM, WN, false, false, true, true, MINB, STAGES, NT, BQ>(p, num_cus, s, nullptr);
}

// Below kNtRows rows per expert on average the 32-row tiles read the weights with the non-temporal policy: an expert with
// one row tile uses them once, and such a stream gets 6.3 TB/s out of HBM where the plain one gets 5.7.  128 experts
// 2048 -> 8192, layer in ms, plain / non-temporal, 1, 2, 4, 7 rows per expert: 0.95 / 0.87, 1.28 / 1.18, 1.50 / 1.37, 1.53 / 1.41;
// e4m3 0.50 / 0.47, 0.67 / 0.62, 0.77 / 0.71, 0.80 / 0.75.  A hot expert's row tiles share its weights through the caches; from
// kNtSoleRows on (variants 5, 25) its tiles read plainly: 512 experts 1024 -> 4096, 1792 skewed tokens 676 us, with all tiles
// non-temporal 788, with none 745.  Below it (3, 23) the choice costs the 0.5 % it gains.  4-bit weights (43): all, there
// the choice costs 1 % and gains nothing.  From kNtRows on the plain variants (4, 24, 44) run: with 16 skewed rows over 512
// experts of 1024 -> 4096 the policy, taken for all tiles, gained 2 % on repeated passes (1.645 -> 1.612) and lost 6 % on a first one
// (1.732 -> 1.837), and 64-row tiles of 4-bit weights over 256 rows 0.402 -> 0.412.
static constexpr int kNtRows = 8, kNtSoleRows = 2;
// Weights of one GEMM (all experts) from which on its time is that of streaming them
static constexpr int64_t kHeavyWeights = 1ll << 29;
// ... and below which it is that of its launch and of one tile
static constexpr int64_t kLightWeights = 3ll << 23;

// Quantised weights on tiles cut to an expert's rows (28: e4m3, 49: mxfp4; gemm_ring.hip), which take a tile's weights once for up to
// 256 rows where the small tiles take them, and widen them, once for 64: from so many rows per expert on, and so much
// work in all that it pays for the schedule (7 us) and for a last round of tall tiles.  FFN in us, 64x128 / 28 and 64x256 / 49,
// even and skewed (0.8):
//   128 experts 2048 -> 8192, 48 rows per expert e4m3 889 / 848, 1041 / 987; 64 rows 914 / 869, 1186 / 1032 and 679 / 788, 963 / 971;
//   128 rows 1469 / 1150, 1777 / 1329 and 1242 / 1056, 1493 / 1241; 512 rows 5326 / 3265, 5798 / 3580 and 4552 / 3140, 4831 / 3400
//   64 experts 1024 -> 4096, 64 rows 142 / 135, 165 / 180 and 110 / 122, 135 / 181; 128 rows 204 / 175, 226 / 227 and 171 / 156, 223 / 222;
//   256 rows 364 / 258, 397 / 316 and 329 / 230, 370 / 290
//   16 experts 1024 -> 4096, 128 rows 72 / 80, 82 / 91 and 79 / 81, 89 / 92; 256 rows 102 / 99, 112 / 110 and 100 / 92, 123 / 106
//   8 experts 512 -> 2048, old / new at 1024 rows 0.99, 0.93 and 1.05, 1.07, at 1536 rows 1.08, 1.16 and 1.16, 1.10
// The least work is rows * D * F of base + per_weight * D * F up to most, a quarter more with a dimension of 768 or less (few columns
// and long K loops in one GEMM).  Over 35 layers of 2 to 512 experts, 256 -> 1024 to 4096 -> 14336, 32 to 4096 rows, even, skewed
// (0.5, 0.8) and half idle, the 1762 batches on the new side of the line take 0.80 of the old time in the mean, 1.16 at worst.
static bool quant_ring_pays(int64_t n_rows, int E, int N, int K, int64_t least_rows, double base, double per_weight, double most)
{
    const double weights = (double)N * K;
    double work = base + per_weight * weights;
    if (work > most) work = most;
    if ((N < K ? N : K) <= 768) work *= 1.25;
    return n_rows >= least_rows * E && (double)n_rows * weights >= work;
}

// 8-bit weights with fewer rows: the small tiles, three LDS stages deep (36 KB with 32 rows:
// four blocks per CU; a fourth stage leaves room for three: 16 experts 2048 -> 8192, 100 tokens 129 -> 137 us, 128 experts,
// 512 tokens 786 -> 797).  (Measured on 128 experts of 2048 x 8192 with 1 to 64 rows each: 2 to 6
// stages, 32x64 and 32x256 tiles and up to 6 blocks per CU all land within +-8 % of these two.)
int gemm_bf16_variant_w8(int64_t n_rows, int E, int N, int K)
{
    const int64_t avg = E > 0 ? n_rows / E : n_rows;
    if (gemm_ring_quant_ok(n_rows, N, K) && quant_ring_pays(n_rows, E, N, K, (int64_t)E * N * K >= 2 * kHeavyWeights ? 48 : 80, 12e9, 1000., 30e9)) return 28;
    // 64-row tiles, us against 32-row ones (128 experts 2048 -> 8192 / 64 experts 1024 -> 4096): 24 rows 942 / 993 and
    // 165 / 151, 36 rows 998 / 1250 and 171 / 203.  With fewer experts their smaller number counts for more, above all
    // where the rows are spread unevenly: 32 experts 2048 -> 8192, skewed, 30 rows 285 / 267, 36 rows 287 / 312; 8 experts
    // 512 -> 2048, 36 rows 44 / 41; 8 experts 2048 -> 8192, 32 rows even 112 / 108, skewed 117 / 106; 16 experts, 44 rows 188 / 176.
    return avg >= (E >= 64 ? 28 : E >= 32 ? 34 : 48) ? 22 : avg >= kNtRows ? 24 : avg >= kNtSoleRows ? 25 : 23;
}

// 4-bit weights with fewer rows: 43 = 32x256, 48 = 64x256, three LDS stages each plus the two scale buffers (32x256: 44 KB,
// three blocks per CU; a fourth stage would leave room for two, 0.141 -> 0.154 ms on the decoder's first
// GEMM; two stages 0.150).  (Measured on 128 experts of 2048 x 8192
// with 1 to 64 rows each: 256 columns per tile beat 128 by 25-30 % -- the A tile, re-read once per column
// tile, weighs as much as a 128-column B tile at 4 bits -- and 512 lost again.  Where the tiles are fewer than the CUs the
// time is the K loop of one tile, whatever its width or the pipeline's depth; those calls are gemm_stream.hip's.)
// 64-row tiles, us against 32-row ones: 128 experts 2048 -> 8192: 36 rows per expert 774 / 726, 64 rows 939 / 1113; 16
// experts 1024 -> 4096, whose 64 weight panels leave the chip to few tiles: 64 rows 95 / 80, 100 rows 97 / 99.  At 44 rows they
// gain on evenly spread rows only (even, skewed, more skewed: 32 experts 2048 -> 8192 210 / 236, 251 / 232, 259 / 238; 64
// experts 1024 -> 4096 137 / 141, 151 / 142, 157 / 145), at 56 on all (255 / 267, 265 / 281, 266 / 268; 155 / 159, 160 / 165, 168 / 164).
// From 2^30 weights per GEMM on, reading them once instead of twice pays at 44 (64 experts 2048 -> 8192 346 / 453, 422 / 444,
// 468 / 442; 128 experts 701 / 812, 773 / 794, 874 / 847).
int gemm_bf16_variant_w4(int64_t n_rows, int E, int N, int K, int num_cus)
{
    const int64_t avg = E > 0 ? n_rows / E : n_rows;
    const int64_t panels = (int64_t)E * (N < K ? N : K) / 256;
    if (gemm_ring_quant_ok(n_rows, N, K) && quant_ring_pays(n_rows, E, N, K, (int64_t)E * N * K >= 2 * kHeavyWeights || panels >= 512 ? 80 : 112, 6e9, 1500., 15e9)) return 49;
    return avg >= (4 * panels <= num_cus ? 96 : (int64_t)E * N * K >= 2 * kHeavyWeights ? 44 : 56) ? 48 : avg >= kNtRows ? 44 : 43;
}

// K ranges for the fp32-output plain GEMM (the gate): 1 unless the 32-row tiles would leave most of the
// chip idle; then the largest power of two <= 16 that divides the K tile count, keeps two K tiles per
// range and does not make more tiles than CUs.
int gemm_bf16_gate_split(int M, int N, int K, int num_cus)
{
    const int bn = N <= 32 ? 32 : (N <= 64 ? 64 : 128);
    const int64_t tiles = (int64_t)ceil_div(M, 32) * ceil_div(N, bn);
    if ((int64_t)ceil_div(M, 128) * ceil_div(N, 128) >= 2 * (int64_t)num_cus) return 1;  // the 128-row shape runs
    const int kt = ceil_div(K, BK);
    int s = 1;
    while (s * 2 <= 16 && kt % (s * 2) == 0 && kt / (s * 2) >= 2 && tiles * s * 2 <= num_cus) s *= 2;
    return s;
}

int gemm_bf16_variant_block_m(int v)
{
    switch (v) {
    case 8: case 28: case 49: return kRingMap;
    case 10: return 128;
    case 2: case 22: case 48: return 64;
    case 3: case 4: case 5: case 23: case 24: case 25: case 43: case 44: return 32;
    default: return 256;
    }
}

// Tile shapes of the grouped GEMM.  variant -> (BM, BN, waves, pipeline)
//   8: 32 .. 256 x 256, 8 waves, gemm_ring.hip    10: 128x128, 4 waves, register-staged
//   9: 256x256, register-staged, for what gemm_ring.hip cannot address
//   2: 64x128, 4 waves, direct-to-LDS    3, 4, 5: 32x128, the same, weights read non-temporally, plainly, by tile (kNtRows)
// By the average number of rows per expert, by how many 256-column weight panels there are (E * min(D, F) / 256, the
// same for both GEMMs of a layer), and by how many weights a GEMM streams.
//  * Tiles cut to an expert's rows (8) pay from 116 rows on, where most experts need two 128-row tiles: over six layers (24,
//    32, 48 experts 1000 -> 4000; 32, 64 experts 1024 -> 4096; 16 experts 2048 -> 8192) and even, skewed (exponent 0.5) and
//    more skewed (0.8) loads the mean of 10 / 8 is 0.92 at 108 rows, 1.01 at 116, 1.03 at 124, 1.05 at 128, 1.09 at 150, either
//    way by the layer and the load: FFN in us, 10 / 8, at 116 rows, 24 experts 1000 -> 4000 134 / 166, 134 / 166, 189 / 166; 48
//    experts 249 / 232, 312 / 248, 285 / 253; 64 experts 1024 -> 4096 298 / 277, 299 / 325, 307 / 313; at 150 rows 339 / 289,
//    356 / 324, 352 / 325.
//  * With a dimension of 768 or less, one GEMM has few K tiles a tile, which do not make up for its start, and the other few
//    columns: there it takes 192 rows, 144 tiles and 1024 as the other dimension.  Over 211 random layers with such a
//    dimension, 192 rows and more, and the three kinds of load the better of the two shapes is missed by 1.1 % in the mean, by
//    4.8 % without the last two conditions and by 4.0 % with 128x128 throughout.  10 / 8, even, skewed (0.5), more skewed
//    (0.8): 128 experts 512 -> 2048, 150 rows 205 / 214, 189 / 192, 191 / 198, 192 rows 204 / 198, 211 / 210, 212 / 213; 64
//    experts 512 -> 2048, 400 rows, even, more skewed 177 / 147, 176 / 172; 191 experts 256 -> 256, 228 rows 42 / 48; 25
//    experts 384 -> 1536, 477 rows 65 / 80, 66 / 78.
//  * They need tiles enough for the chip, 96 in the GEMM with fewer columns, and with fewer than 112 at least 120 rows.  Over
//    45 random layers (12 to 60 experts, 784 to 2032 -> 872 to 7928) and the same kinds of load the mean of 10 / 8 is 0.78 at
//    80 to 95 tiles; at 96 to 111 tiles 0.85 with 116 to 119 rows, 0.98 with 120 to 127, 1.06 with 128 to 132; at 112 to 140
//    tiles 1.02, 1.05 and 1.08.  With more rows, 10 / 8, even, skewed (0.5), more skewed (0.8), 64 to 95 tiles: 5 experts 2048
//    -> 4096, 298 rows 92 / 118, 93 / 119, 93 / 119; 13 experts 1536 -> 1536, 241 rows 73 / 81, 70 / 82, 76 / 83; 16 experts
//    1024 -> 4096, 224 rows 105 / 118, 130 / 127, 133 / 127; 5 experts 4096 -> 14336, 197 rows 436 / 446, 485 / 441, 471 / 449;
//    96 to 128 tiles: 6 experts 2048 -> 8192, 398 rows 250 / 238, 243 / 237, 250 / 243; 12 experts 2048 -> 4096, 176 rows 141 /
//    142, 158 / 142, 161 / 147; 14 experts 2048 -> 8192, 170 rows 293 / 271, 313 / 280, 306 / 292; 8 experts 4096 -> 14336, 128
//    rows, even 530 / 476.  The GEMM with fewer columns counts, also where the other one has many: 8 experts 256 -> 3328, 1500
//    rows (48 and 624) 80 / 103, 82 / 107.  An even batch with a mean just below 256 rows needs two tiles for a part of its
//    experts and counts so: 250 rows, 16 experts 1024 -> 4096 134 / 132, 132 / 132, 131 / 130; 8 experts 2048 -> 8192 244 /
//    230, 241 / 234, 262 / 236.
//  * GEMMs of 2^29 weights and more (1 GB, four times the last-level cache) take the time of one pass over an expert's weights.
//    There they pay from 8 rows on, given two 256-column panels per CU.  What ran before / 8, even, skewed (0.8):
//      128 experts 2048 -> 8192, 4 rows per expert 1319 / 1482, 1125 / 1293; 8 rows 1525 / 1427, 1549 / 1416; 25 rows 1453 / 1479, 1605 / 1642;
//      39 rows 1479 / 1508, 1648 / 1640; 78 rows 1588 / 1627, 1759 / 1786; 100 rows 1630 / 1693, 1973 / 1831 (2 to 4 % behind on
//      even batches of 25 to 100 rows: a 128x256 ring of fixed height ran there)
//      512 experts 1024 -> 4096, 8 rows 1513 / 1460, 1485 / 1427; 34 rows 1599 / 1569, 1691 / 1657; 64 rows 1685 / 1658, 1869 / 1794
//      64 experts 2048 -> 8192, 16 rows 787 / 762, 831 / 755; 64 rows 771 / 793, 921 / 926; half of the experts idle 394 / 387, 431 / 443
//    Not with a dimension of 768 or less, which the shapes for fewer weights serve (32x128, 64x128 or 128x128 / 8: 512 experts
//    512 -> 2048, 8 rows 384 / 401, 393 / 400; 40 rows 443 / 452, 472 / 499; 64 rows 491 / 489, 509 / 528; 1024 experts 512 -> 1024, 8
//    rows 401 / 430, 383 / 410; 400 experts 768 -> 2048, 24 rows 490 / 513, 514 / 525).
//    With one panel per CU and less they lose where rows are even or experts idle, 10 or 4 / 8, even, half of the experts idle,
//    skewed: 16 experts 4096 -> 14336, 32 rows 714 / 770, 397 / 476, 770 / 766; 100 rows 766 / 806, 564 / 527, 991 / 1007; 32
//    experts 2048 -> 8192, 8 rows 388 / 376, 219 / 245, 424 / 375; 4 experts 8192 -> 28672, 100 rows 760 / 887, 605 / 661.  With
//    fewer weights 8 does not pay at few rows (8 / small tiles at 24 rows: 128 experts 512 -> 2048 137 / 137, 159 / 135, 157 /
//    133).
//  * With fewer weights 64x128 is the steadiest shape from 34 to 63 rows, 32x128 / 64x128 / 128x128: 128 experts 512 -> 2048,
//    36 rows 171 / 161 / 162, 173 / 169 / 183, 170 / 164 / 176; 64 experts 1024 -> 4096, 48 rows 314 / 287 / 266, 327 / 280 /
//    309, 329 / 281 / 302; 16 experts 2048 -> 8192, 48 rows 292 / 291 / 279, 319 / 298 / 285, 310 / 297 / 323; at 64 rows
//    128x128 has caught up (342 / 320 / 284, 332 / 311 / 309, 342 / 308 / 338).
//    With 64 panels or fewer the 64-row tiles have the chip to themselves, as narrow ones with more stages (launch_gemm_bf16), and
//    take over from the streaming kernel and from 128x128, small / 2 / 10, even, skewed (0.8).  33 to 64 panels, from 8 to 95 rows (they
//    lose where half of the experts are idle and the others even, which the host does not see: 16 experts 1024 -> 4096, 8 rows 37 / 42, 16 rows
//    42 / 43; 4 experts 4096 -> 14336, 8 rows 108 / 119): 8
//    experts 2048 -> 8192, 6 rows 98 / 102, 108 / 102; 8 rows 102 / 102, 113 / 102; 18 rows 107 / 100, 144 / 100; 84 rows - / 147 / 148, - / 153 /
//    173; 100 rows - / 147 / 142, - / 160 / 157; 16 experts 1024 -> 4096, 8 rows 58 / 58, 77 / 58; 32 experts 512 -> 2048, 20 rows 39 / 38, 46 / 44;
//    80 rows - / 50 / 49, - / 54 / 55.  17 to 32 panels, where the streaming kernel has short rounds while an expert has one of its tiles, from 33 to
//    128 rows: 8 experts 1024 -> 4096, 28 rows 39 / 44, 56 / 48; 33 rows 56 / 44, 57 / 49; 90 rows 69 / 53 / 68, 76 / 53 / 76; 150 rows - / 62 /
//    58, - / 67 / 61; 2 experts 4096 -> 14336, 40 rows 168 / 122, 165 / 123.  16 and fewer, from 65 to 191: 8 experts 512 -> 2048, 50 rows 20 / 23, 21 /
//    24; 65 rows 29 / 24, 29 / 25; 250 rows - / 28 / 32, - / 35 / 35; 4 experts 1024 -> 4096, 80 rows 52 / 41, 51 / 41; 300 rows - / 59 / 56, - / 60 / 56.
//    33 to 64 panels of few weights: from 17 rows (small / 2, mean over even, skewed and half idle batches: 100 experts 128 -> 512, 8 rows 12.5 /
//    13.4, 24 rows 14.3 / 13.9; 64 experts 192 -> 768, 8 rows 15.5 / 16.8; 40 experts 320 -> 1280, 12 rows, half idle 15.5 / 17.7, 24 rows 25 / 22), with
//    a dimension of 64 from 48 (250 experts 64 -> 512, 24 rows 17.8 / 18.2, skewed 18.7 / 20.1; 48 rows - / 21 / 25).
//  * No dimension of 64 and less: 10 is ahead there of 256-row tiles too (9 / 10: 64 experts 64 -> 256, 800 rows 30 / 24; 64 ->
//    1024 62 / 55; 16 experts 4096 -> 64, 1000 rows 95 / 85; 128 experts 40 -> 512, 1000 rows 82 / 69).  9 is for operands that
//    8 cannot address (9 / 10: 8 experts 2048 -> 8192, 33750 rows 15550 / 20945; 8 experts 1000 -> 8200, 33000 rows 9183 /
//    16220).
//  * K that is no multiple of the K tile: with 64 panels and fewer the same lines (small / 2 / 10: 8 experts 1000 -> 4000, 40 rows 53 / 47 / 56,
//    68 / 60 / 64; 80 rows 71 / 55 / 60, 86 / 59 / 78; 32 experts 496 -> 4984, 30 rows 104 / 82 / 89, 135 / 129 / 138; 5 experts 520 -> 1560, 300 rows
//    - / 28 / 35) but for two, 2 / 10, mean and worst of even, random, skewed and half idle batches against 128x128 in registers: 33 to 47 panels from
//    60 rows 10 (17 experts 680 -> 5896, 64 rows 1.00, 1.18 / 0.83, 0.85; 6 experts 2040 -> 6000, 72 rows 0.93, 1.00 / 0.88, 0.89), 17 to 32 panels from 120
//    (8 experts 1000 -> 4000, 0.97, 1.15 / 0.91, 0.92; 16 experts 400 -> 4400, 128 rows 0.94, 1.08 / 0.87, 0.89).  With up to 96 panels, 128 of few
//    weights, 64x128 from 30 to 49 rows (24 experts 1000 -> 4000, 36 rows 0.93, 1.02, 48 rows 0.97, 1.05, 50 rows 1.01, 1.25; 36 experts 520 -> 2000,
//    48 rows 0.92, 0.95; 130 experts 200 -> 600, 30 rows 0.88, 0.93); with more the 128-row tiles throughout (36 rows: 28 experts 1000 -> 3000 1.05, 1.25; 47
//    experts 1496 -> 4504 1.01, 1.10; 52 experts 840 -> 7120 1.03, 1.29; 60 experts 1000 -> 2000 1.01, 1.24; 40 experts 1960 -> 3000 1.04, 1.17).
int gemm_bf16_variant(int64_t n_rows, int E, int N, int K, int num_cus)
{
    const int64_t avg = E > 0 ? n_rows / E : n_rows;
    const int width = N < K ? N : K;
    const int64_t panels = (int64_t)E * width / 256;
    const bool whole = N % BK == 0 && K % BK == 0;
    const bool heavy = whole && width > 768 && (int64_t)E * N * K >= kHeavyWeights;
    const int64_t tiles = (int64_t)E * ((avg + 8 + 255) / 256) * ceil_div(width, 256);
    const bool fills = width <= 768 ? avg >= 192 && tiles >= 144 && (N > K ? N : K) >= 1024
                                    : tiles >= 96 && avg >= (tiles < 112 ? 120 : 116);
    const bool streams = heavy && avg >= kNtRows && panels >= 2 * (int64_t)num_cus;
    const bool light = (int64_t)E * N * K < kLightWeights;
    if (gemm_ring_ok(n_rows, N, K) && (fills || streams)) return 8;
    if (avg >= 192) return gemm_ring_addresses(n_rows, N, K) ? 10 : 9;
    const int small = avg >= kNtRows ? 4 : avg >= kNtSoleRows ? 5 : 3;
    if (4 * panels <= num_cus) {
        const int from = width <= 64 ? 48 : light ? 17 : 8;
        if (8 * panels > num_cus) return avg >= (whole || 16 * panels >= 3 * num_cus ? 96 : 60) ? 10 : avg >= from ? 2 : small;
        return 16 * panels > num_cus ? (avg > (whole || light ? 128 : 119) ? 10 : avg > 32 ? 2 : small) : (avg > 64 ? 2 : small);
    }
    if (whole && !heavy && avg < 64) return avg >= 34 ? 2 : small;
    if (!whole && avg < 50 && (light ? 2 * panels <= num_cus : 8 * panels <= 3 * num_cus)) return avg >= 30 ? 2 : small;
    return avg >= 30 ? 10 : small;
}

// Whether a GEMM has at most so many tiles per CU, as estimated from the mean number of rows per expert times `spread`.
static bool few_tiles(const GemmParams &p, int block_m, int block_n, double spread, double per_cu, int num_cus)
{
    const int64_t rows = (int64_t)(spread * p.M / p.num_experts + 0.999);
    return (double)(p.num_experts * ((rows + block_m - 1) / block_m)) * ceil_div(p.N, block_n) <= per_cu * num_cus;
}

int launch_gemm_stream(const GemmParams &p, int wbits, bool relu, int num_cus, hipStream_t s, bool *taken);

template <int BM, int BN, int WM, int WN, int MINB, int STAGES = 2>
static int launch_grouped(const GemmParams &p, bool relu, int num_cus, hipStream_t s, int *main_grid = nullptr)
{
    return relu ? launch_one<BM, BN, WM, WN, false, true, true, MINB, STAGES>(p, num_cus, s, main_grid)
                : launch_one<BM, BN, WM, WN, false, false, true, MINB, STAGES>(p, num_cus, s, main_grid);
}

// Dispatch over the instantiated shapes.
int launch_gemm_bf16(const GemmParams &p, bool grouped, int variant, bool out_f32, bool relu, int num_cus,
                     hipStream_t s)
{
    if (!grouped) {
        // gate: fp32 logits, N = E is small
        if (relu) {
            set_error("plain bf16 GEMM is not instantiated with ReLU");
            return MOE_ERR_UNSUPPORTED;
        }
        // bf16 output: the dense mask multiplications of the static-capacity baseline
        if (!out_f32) return launch_one<256, 256, 2, 4, false, false, false, 1, REG_STAGED>(p, num_cus, s);
        // 128-row tiles when they still fill the chip twice over, else 32-row tiles: the K loop of such a
        // skinny GEMM is latency bound, so the number of tiles in flight is what streams x
        const bool tall = (int64_t)ceil_div(p.M, 128) * ceil_div(p.N, 128) >= 2 * (int64_t)num_cus;
        // 32-row tiles run four LDS stages deep (three K tiles in flight per block)
        if (p.N <= 32)
            return tall ? launch_one<128, 32, 4, 1, true, false, false, 2>(p, num_cus, s)
                        : launch_one<32, 32, 1, 1, true, false, false, 2, 4>(p, num_cus, s);
        if (p.N <= 64)
            return tall ? launch_one<128, 64, 2, 2, true, false, false, 2>(p, num_cus, s)
                        : launch_one<32, 64, 1, 2, true, false, false, 2, 4>(p, num_cus, s);
        return tall ? launch_one<128, 128, 2, 2, true, false, false, 2>(p, num_cus, s)
                    : launch_one<32, 128, 1, 4, true, false, false, 2, 4>(p, num_cus, s);
    }
    if (out_f32) {
        set_error("grouped bf16 GEMM is only instantiated for bf16 output");
        return MOE_ERR_UNSUPPORTED;
    }
    if (gemm_bf16_variant_block_m(variant) == 32) {
        bool taken = false;
        const int rc = launch_gemm_stream(p, variant >= 43 ? 4 : variant >= 23 ? 8 : 0, relu, num_cus, s, &taken);
        if (taken || rc != MOE_OK) return rc;
    }
    switch (variant) {
    case 8: return launch_gemm_ring(p, 0, relu, s);
    case 28: return launch_gemm_ring(p, 8, relu, s);
    case 49: return launch_gemm_ring(p, 4, relu, s);
    case 9: {
        // whole rounds as 256x256 tiles, the partly filled last round as 128x128 sub-tiles
        GemmParams q = p;
        int main_grid = 0;
        q.tail_mode = 1;
        const int rc = launch_grouped<256, 256, 2, 4, 1, REG_STAGED>(q, relu, num_cus, s, &main_grid);
        if (rc != MOE_OK || main_grid == 0) return rc;
        q.tail_mode = 2;
        return launch_grouped<128, 128, 2, 2, 2, REG_STAGED>(q, relu, num_cus, s, &main_grid);
    }
    case 10:
        // At most a tile per CU, also where some experts have half as many rows again: 128x64 tiles, four stages.  FFN in us, 128x128 /
        // these, even, skewed (0.8): 8 experts 1024 -> 4096, 150 rows 69 / 58, 73 / 61; 4 experts 2048 -> 8192, 150 rows 118 / 101, 126 / 105; 4
        // experts 1024 -> 4096, 300 rows 67 / 56, 67 / 56; 8 experts 512 -> 2048, 250 rows 37 / 32, 39 / 35.  Without the half: 8 experts 1024 ->
        // 4096, 240 rows 72 / 61, 82 / 98; 8 experts 2048 -> 8192, 100 rows 141 / 124, 156 / 184.
        if (few_tiles(p, 128, 64, 1.5, 1, num_cus)) return launch_grouped_dtl<128, 64, 2, 2, 2, 4, NT_NONE, 0>(p, relu, num_cus, s);
        return launch_grouped<128, 128, 2, 2, 2, REG_STAGED>(p, relu, num_cus, s);
    case 2:
        // With a tile or two per CU its time is that of the K loop, whose loads are as far ahead as the LDS has stages and which
        // narrower tiles share among more blocks.  FFN in us, 64x128 in two stages / in three / 64x64 in four, even, skewed (0.8): 8 experts
        // 2048 -> 8192, 64 rows 160 / 126 / 108, 168 / 132 / 141; 16 experts 1024 -> 4096, 48 rows 91 / 72 / 62, 95 / 76 / 79; 12
        // experts, 56 rows - / 64 / 55, - / 64 / 58; 4 experts 4096 -> 14336, 40 rows 281 / 209 / 177, 294 / 221 / 237; 16 experts 2048 ->
        // 8192, 48 rows 225 / 200 / 196, 237 / 242 / 246; with more tiles two stages, of which a CU holds three blocks: 64 experts
        // 1024 -> 4096, 40 rows 203 / 212, 226 / 231.  Up to 16 rows per expert 64x64 also with more tiles: most of a tile's rows are padding
        // then, and it is the weights' way that counts (64x128 in three stages / 64x64, half of the experts idle, 16 experts 1024 -> 4096, 8 rows 46 /
        // 42; 4 experts 4096 -> 14336 136 / 119; even 6 experts 2040 -> 6000, 12 rows 92 / 88).
        if (few_tiles(p, 64, 64, 1, 1, num_cus) || p.M <= 16ll * p.num_experts) return launch_grouped_dtl<64, 64, 2, 2, 2, 4, NT_NONE, 0>(p, relu, num_cus, s);
        return few_tiles(p, 64, 128, 1, 1.5, num_cus) ? launch_grouped_dtl<64, 128, 1, 4, 2, 3, NT_NONE, 0>(p, relu, num_cus, s)
                                         : launch_grouped_dtl<64, 128, 1, 4, 2, 2, NT_NONE, 0>(p, relu, num_cus, s);
    case 22: return launch_grouped_dtl<64, 128, 1, 4, 2, 3, NT_NONE, 8>(p, relu, num_cus, s);
    case 23: return launch_grouped_dtl<32, 128, 1, 4, 2, 3, NT_ALL, 8>(p, relu, num_cus, s);
    case 24: return launch_grouped_dtl<32, 128, 1, 4, 2, 3, NT_NONE, 8>(p, relu, num_cus, s);
    case 25: return launch_grouped_dtl<32, 128, 1, 4, 2, 3, NT_SOLE, 8>(p, relu, num_cus, s);
    case 43: return launch_grouped_dtl<32, 256, 1, 4, 2, 3, NT_ALL, 4>(p, relu, num_cus, s);
    case 44:
        // At most a tile per CU (64-row tiles: one for every other CU): half the columns, and a stage more.  FFN in us, 256 columns / 128, even,
        // skewed (0.8): 32 rows: 16 experts 2048 -> 8192, 36 rows 137 / 123, 140 / 126; 64 experts 1024 -> 4096, 20 rows 83 / 77, 94 / 85; 32
        // experts 2048 -> 8192, 30 rows 157 / 147, 182 / 167; 128 experts 512 -> 2048, 20 rows 50 / 47, 61 / 56; 64 rows: 8 experts 2048 ->
        // 8192, 100 rows 136 / 121, 136 / 121; 16 experts 1024 -> 4096, 100 rows 78 / 70, 78 / 70; 16 experts 2048 -> 8192, 60 rows 143 / 132,
        // 159 / 163; a tile per CU: 32 experts 2048 -> 8192, 60 rows 199 / 205, 250 / 260.  64-row tiles counted with 1.15 times the rows: near a
        // whole tile some experts have two (layer, random gate: 16 experts 2048 -> 8192, 60 rows 178 / 182, 32 experts 512 -> 2048, 128 rows 71 / 74).
        if (few_tiles(p, 32, 256, 1, 1, num_cus)) return launch_grouped_dtl<32, 128, 1, 4, 2, 4, NT_NONE, 4>(p, relu, num_cus, s);
        return launch_grouped_dtl<32, 256, 1, 4, 2, 3, NT_NONE, 4>(p, relu, num_cus, s);
    case 48:
        if (few_tiles(p, 64, 256, 1.15, 0.5, num_cus)) return launch_grouped_dtl<64, 128, 2, 2, 2, 4, NT_NONE, 4>(p, relu, num_cus, s);
        return launch_grouped_dtl<64, 256, 1, 4, 2, 3, NT_NONE, 4>(p, relu, num_cus, s);
    case 3: case 4: case 5: {
        // as the 64-row tiles, two stages / four: 8 experts 2048 -> 8192, 40 rows 158 / 113, 171 / 131; 16 experts 2048 -> 8192, 20 rows 209 / 189, 229 /
        // 236; 16 experts 1024 -> 4096, 36 rows 88 / 66, 95 / 73.  Not with a K tile or three (64 experts 192 -> 768, 12 rows 17.0 / 17.5).
        const bool deep = few_tiles(p, 32, 128, 1, 1.5, num_cus) && p.K >= 4 * BK;
        // K that ends inside a K tile: weight rows then begin inside a line, and the loads in flight in registers are as good (47 experts
        // 1496 -> 4504, 8 and 20 rows 293 / 296, 310 / 314 us register-staged / direct-to-LDS, non-temporal 380, 395), but for
        // few tiles (24 experts 1000 -> 4000, 16 rows 95 / 89, skewed 103 / 98)
        if (p.K % BK != 0 && !deep)
            return relu ? launch_k<32, 128, 1, 4, false, true, true, false, 2, REG_STAGED>(p, num_cus, s, nullptr)
                        : launch_k<32, 128, 1, 4, false, false, true, false, 2, REG_STAGED>(p, num_cus, s, nullptr);
        return variant == 3 && p.K % BK == 0 ? launch_grouped_dtl<32, 128, 1, 4, 2, 2, NT_ALL, 0>(p, relu, num_cus, s)
               : variant == 5 && p.K % BK == 0 ? launch_grouped_dtl<32, 128, 1, 4, 2, 2, NT_SOLE, 0>(p, relu, num_cus, s)
               : deep                          ? launch_grouped_dtl<32, 128, 1, 4, 2, 4, NT_NONE, 0>(p, relu, num_cus, s)
                                               : launch_grouped_dtl<32, 128, 1, 4, 2, 2, NT_NONE, 0>(p, relu, num_cus, s);
    }
    default:
        set_error("unsupported grouped GEMM variant %d", variant);
        return MOE_ERR_UNSUPPORTED;
    }
}

}  // namespace moe355
