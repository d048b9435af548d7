// Launch shapes for grids that no tuned entry covers: a cost rule over a few
// measured shapes.
//
// A shape cuts the grid into strips and the march into chunks of z levels;
// every (strip, chunk) is one wavefront.  The chip holds `slots` wavefronts of
// the shape at once (1024 SIMDs times the one or two that its registers
// allow), and a wavefront's time is its levels plus the start of its pipeline
// (the planes before the first level: `start` levels, 1.5 for three fields and
// 2.5 for the adjoint's six arrays).  So with q = wavefronts / slots the march
// takes
//
//     cost * rounds(q) * (z + start),
//
// where whole rounds count one each and a partly filled round counts its
// share, but at least 0.8: below that the wavefronts in flight no longer
// saturate the memory and the round is as long as its latency.  Marches cut
// into as many chunks as one round holds are tried beside the fixed counts
// (3 % over 72 grids whose pick it changed).  `cost` is a shape's time per level
// of a full round, in arbitrary units within a list, and shapes of different
// widths compete through their wavefront counts: a strip that a narrow grid half
// fills costs as much as a full one, and at the grid's x end `ragged` times as
// much.  Tall shapes read less and take longer to start, so that small grids
// leave them to the others without a line in the number of points.
//
// The constants are fitted to sweeps over shapes and march lengths, whose grids
// and error stand with each list (2 to 7 % slower than the best shape of the
// sweep in the geometric mean; 16 x 16 x 16 to 1024 x 1024 x 256, most of them
// ragged).  The fixed shape with "about 2048 wavefronts, chunks of at least 8
// levels" that the rule replaced was 1.5 to 1.65 times slower than its picks: 9.5
// -> 3.5 us at 32x32x64 (chunks of one level: a march of eight is latency, and
// the grid has too few strips to hide it), 130 -> 42 us at 42x587x244 (one
// column per lane where four leave 5 lanes in 6 idle), 70 -> 43 us at 300x300x75.
#include <algorithm>

#include "pw_internal.h"

namespace pw {

TileCfg cheapest_shape(const ShapeCost *s, int n, int64_t lead, int64_t rows, int64_t march, bool may_pack) {
    // Runs on every untuned call: the fixed counts' marches are formed once for
    // all shapes (201x143x117 FP32: 1.25 us of host time with two divisions for
    // each, so 1.07).
    static const int kChunks[] = {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 16, 24, 32, 48, 64, 128};
    constexpr int kFixed = sizeof(kChunks) / sizeof(kChunks[0]);
    const int levels = static_cast<int>(std::min<int64_t>(march, INT32_MAX - 128));
    int z[kFixed + 1], chunks[kFixed + 1], tries = 1;   // the first is each shape's own
    for (int c : kChunks) {
        if (c > levels) break;
        z[tries] = (levels + c - 1) / c;
        chunks[tries] = (levels + z[tries] - 1) / z[tries];
        if (tries == 1 || z[tries] != z[tries - 1]) ++tries;
    }
    TileCfg best;
    double best_cost = -1.0;
    for (int i = 0; i < n; ++i) {
        const Strips st = strips_of(lead, rows, s[i].cols, s[i].ry, may_pack);
        const double strips = static_cast<double>(st.count);
        const double level = lead % s[i].cols == 0 || st.packed   // the strips at the x end weigh more
                                 ? s[i].cost
                                 : s[i].cost * (1.0 + (s[i].ragged - 1.0) / static_cast<double>((lead + s[i].cols - 1) / s[i].cols));
        const int fill = static_cast<int>(std::min(128.0, s[i].slots / strips));   // as many chunks as one round holds
        const bool own = fill >= 1 && fill <= levels;
        if (own) {
            z[0] = (levels + fill - 1) / fill;
            chunks[0] = (levels + z[0] - 1) / z[0];
        }
        for (int t = own ? 0 : 1; t < tries; ++t) {
            const double q = strips * chunks[t] / s[i].slots;
            const double whole = static_cast<double>(static_cast<int64_t>(q)), part = q - whole;
            const double rounds = whole + (part > 0.0 ? (part > 0.8 ? part : 0.8) : 0.0);
            const double cost = level * rounds * (z[t] + s[i].start);
            if (best_cost < 0.0 || cost < best_cost) {
                best_cost = cost;
                best = TileCfg{s[i].px, s[i].ry, z[t], s[i].wpb, s[i].depth, s[i].share};
            }
        }
    }
    return best;
}

}  // namespace pw
