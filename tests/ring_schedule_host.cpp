// The ring kernel's schedule on the host: written and walked with the arithmetic of csrc/ring_schedule.h.
#include "ring_schedule.h"

using namespace moe355;

// covered[u]: how many parts multiply 32-row unit u, the experts' units one behind the other.  Returns the units that the
// parts multiply in all; part_cost[x]: what part x has to do.
extern "C" int ring_cover(const int *rows, int E, int *covered, int *part_cost)
{
    int64_t total = 0, pre = 0;
    for (int e = 0; e < E; ++e) total += ring_cost(ring_units(rows[e]));
    int cut_words[9], all = 0;
    for (int x = 0; x < 9; ++x) cut_words[x] = 1024 << kRingCutShift;
    for (int x = 0; x < 8; ++x) part_cost[x] = 0;
    static bool listed[8][1024];
    for (int e = 0; e < E; ++e) {
        for (int x = 0; x < 8; ++x) listed[x][e] = false;
        ring_pieces(ring_units(rows[e]), pre, (int)total, [&](int x, int, int) { listed[x][e] = true; },
                    [&](int x, int first) { cut_words[x] = e << kRingCutShift | first; });
        pre += ring_cost(ring_units(rows[e]));
    }
    for (int x = 0; x < 8; ++x) {
        int u0 = 0, r0 = 0;  // first unit and row of the expert
        for (int e = 0; e < E; ++e) {
            if (listed[x][e]) {
                int row0 = r0, row_end = r0 + rows[e];
                ring_clip(e, cut_words[x], cut_words[x + 1], row0, row_end);
                const int first = u0 + (row0 - r0) / 32, units = ring_units(row_end - row0);
                for (int u = first; u < first + units; ++u) ++covered[u];
                all += units;
                part_cost[x] += ring_cost(units);
            }
            u0 += ring_units(rows[e]);
            r0 += rows[e];
        }
    }
    return all;
}

// Whether the batch's experts become one list that all XCDs share, for GEMMs of n1 and n2 column tiles.
extern "C" int ring_is_shared(const int *rows, int E, int n1, int n2)
{
    int64_t total = 0, pre = 0;
    for (int e = 0; e < E; ++e) total += ring_cost(ring_units(rows[e]));
    int units[9] = {}, tiles[9][9] = {};  // [8]: of all parts
    for (int e = 0; e < E; ++e) {
        ring_pieces(
            ring_units(rows[e]), pre, (int)total,
            [&](int x, int, int u) {
                const int of[2] = {x, 8};
                for (int part : of) {
                    units[part] += u;
                    for (int h = 1; h <= 8; ++h) tiles[part][h] += (u + h - 1) / h;
                }
            },
            [](int, int) {});
        pre += ring_cost(ring_units(rows[e]));
    }
    float parts = 0.f, eighths = 0.f;
    for (int g = 0; g < 2; ++g) {
        const int n = g == 0 ? n1 : n2, k = g == 0 ? n2 : n1;
        float slowest = 0.f;
        for (int x = 0; x < 9; ++x) {
            RingRounds r;
            for (int h = 8; h >= 1; --h) ring_try_height(r, h, tiles[x][h], (float)units[x], n, x == 8 ? 8 : 5);
            if (x == 8) eighths += r.cost * (float)k;
            else if (r.cost > slowest) slowest = r.cost;
        }
        parts += slowest * (float)k;
    }
    return ring_shares_pay(E, tiles[8][8], eighths, parts);
}

// first[x] .. first[x + 1]: what XCD x takes of a list of so many tiles that all share
extern "C" void ring_shares(int tiles, int *first)
{
    for (int x = 0; x < 9; ++x) first[x] = ring_share(tiles, x);
}
