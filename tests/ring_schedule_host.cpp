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

// first[x] .. first[x + 1]: what XCD x takes of a list of so many tiles that all share
extern "C" void ring_shares(int tiles, int *first)
{
    for (int x = 0; x < 9; ++x) first[x] = ring_share(tiles, x);
}
