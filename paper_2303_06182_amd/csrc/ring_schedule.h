// Arithmetic of the ring kernel's schedule (layout: moe_internal.h), as plain functions: the block that writes a schedule
// (ring_schedule, route.hip), the kernel that walks it (gemm_ring.hip) and the host's check of both take it from here.
#pragma once
#include <stdint.h>

namespace moe355 {

static constexpr int kRingCutShift = 20;  // a cut word: expert << kRingCutShift | 32-row unit

__host__ __device__ __forceinline__ int ring_units(int rows) { return (rows + 31) >> 5; }
// 256-row tiles that hold them
__host__ __device__ __forceinline__ int ring_tiles(int units) { return (units + 7) >> 3; }
// What it costs: see ring_schedule
__host__ __device__ __forceinline__ int ring_cost(int units) { return units == 0 ? 0 : (units > 4 ? units : 4) + 6 * ring_tiles(units); }

// An expert's pieces when the experts' rows, in order, are cut in eight parts of equal cost, between two tiles of an
// expert at most.  pre: cost of the experts in front of it, total: of all.  piece(part, first unit, units) for every part
// that receives some, cut(part, first unit) for every part the expert reaches into from an earlier one -- also for one
// that receives nothing, because the part in front of it ends there.
template <typename Piece, typename Cut>
__host__ __device__ __forceinline__ void ring_pieces(int units, int64_t pre, int total, const Piece &piece, const Cut &cut)
{
    if (units == 0) return;
    const int tiles = ring_tiles(units), height = (units + tiles - 1) / tiles, cost = ring_cost(units);
    int done = 0;
    for (int x = (int)(pre * 8 / total); x < 8 && done < units; ++x) {
        if (done > 0) cut(x, done);
        const int64_t in = (int64_t)total * (x + 1) - 8 * pre;  // 8 x cost of the expert in front of the part's end
        const int64_t at = (2 * in * tiles + 8 * cost) / (16 * (int64_t)cost);
        int end = x == 7 || at >= tiles ? units : (int)at * height;
        if (end > units) end = units;
        if (end > done) {
            piece(x, done, end - done);
            done = end;
        }
    }
}

// What the rounds of 2^log_blocks blocks cost that take n output tiles of each row tile, at the best of the heights tried, and
// that height: tried from 8 down, with the row tiles that the units make at each.  Below four units only to give every block of a
// single round a tile.
struct RingRounds {
    float cost = 0.f;
    int height = 8;
    bool open = true;
};
__host__ __device__ __forceinline__ void ring_try_height(RingRounds &r, int h, int tiles, float units, int n, int log_blocks)
{
    const int64_t out = (int64_t)tiles * n;
    r.open = r.open && tiles > 0 && (h >= 4 || out <= 1 << log_blocks);
    const float c = (float)((out + (1 << log_blocks) - 1) >> log_blocks) * (6.f + units / (float)tiles);
    if (r.open && (h == 8 || c < 0.97f * r.cost)) r.cost = c, r.height = h;
}

// Whether all XCDs share one list of experts, given the estimated cost of their eighths of it and of the slowest parts: see
// ring_schedule.
static constexpr int kRingSharedTiles = 32, kRingWindow = 64;
static constexpr float kRingSharedGain = 0.88f, kRingSharedFewGain = 0.95f;
static_assert(kRingSharedTiles <= kRingWindow, "the ring kernel expects a shared list in one window");
__host__ __device__ __forceinline__ bool ring_shares_pay(int E, int row_tiles, float eighths, float parts)
{
    return (E < row_tiles ? E : row_tiles) <= kRingWindow && eighths < (row_tiles <= kRingSharedTiles ? kRingSharedFewGain : kRingSharedGain) * parts;
}

// Where XCD x's tiles of a list of so many begin that all XCDs share.
__host__ __device__ __forceinline__ int ring_share(int tiles, int x)
{
    const int at = ((tiles + 7) >> 3) * x;
    return at < tiles ? at : tiles;
}

// Of the rows row0 ... row_end of an expert in a part's list, those that the part has; cut_first and cut_last are the cut
// words of the part and of the one behind it.
__host__ __device__ __forceinline__ void ring_clip(int expert, int cut_first, int cut_last, int &row0, int &row_end)
{
    const int first = row0;
    if (expert == cut_first >> kRingCutShift) row0 = first + 32 * (cut_first & ((1 << kRingCutShift) - 1));
    if (expert == cut_last >> kRingCutShift) {
        const int end = first + 32 * (cut_last & ((1 << kRingCutShift) - 1));
        if (end < row_end) row_end = end;
    }
}

}  // namespace moe355
