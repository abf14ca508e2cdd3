// How a product of the token-wise library is laid out, by its sizes.  Host code only, without HIP, so that a
// plain C++ compiler takes it too: the tests ask it which tiles and splits a size runs.
#pragma once
#include <stdint.h>

#include <cmath>

namespace fpdt_tw {

constexpr int SK = 32;  // k per LDS stage, of one MFMA k-step

// The work of a product: the first `whole` of its tiles over all of k, the others divided into `splits`
// ranges of `split_stages` stages (the last one may be shorter).
struct Units {
    int tiles, tiles_n, whole, splits, split_stages;
};

// Output tile (64 wmt x 64 wnt), and which tiles are divided along k: the cheapest in units of the core
// clock, from
//   stage   the MFMAs of a wave (16 clocks each) or the bytes that a stage copies into LDS: 21 per clock and
//           compute unit, measured for all tile shapes
//   unit    a fixed part (first operands, epilogue)
//   rounds  of 256 units (512 where two fit a CU).  Tiles that do not fill the last round are divided, so
//           that it is full and short; with fewer tiles than slots all of them are
//   sums    of the divided tiles: one more launch and (splits + 1) passes over them at about 4.5 bytes per ns
// Measured, all tiles whole -> the rest divided (most of it without a free round at the end, some from the
// epilogues out of step): SwiGLU block at 16K tokens 21.1 -> 18.9 ms, GELU block on 3001 tokens 1562 -> 1458
// us, 4096 x 14336 += 4096 rows 586 -> 475 us.
struct Plan { int wmt, wnt; Units u; };
static inline Plan plan_product(int64_t M, int64_t N, int stages)
{
    static const int shapes[][2] = {{4, 4}, {3, 4}, {2, 4}, {1, 4}, {2, 2}};
    Plan best = {4, 4, {}};
    double best_cost = 0.0;
    for (const auto& sh : shapes) {
        const int wm = sh[0], wn = sh[1];
        const double mfma = 64.0 * wm * wn + 100.0, copies = 192.0 * (wm + wn);
        const double stage = mfma > copies ? mfma : copies, fixed = 1200.0 + 160.0 * wm * wn;
        const int slots = wm * wn <= 4 && wn == 2 ? 512 : 256;
        const double share = slots / 256.0;
        const int64_t tiles_n = (N + 64 * wn - 1) / (64 * wn), tiles = (M + 64 * wm - 1) / (64 * wm) * tiles_n;
        if (tiles > (int64_t)1 << 30) continue;
        const int64_t rest = tiles % slots, whole = tiles - rest;
        for (int sp = 1; sp <= 16; ++sp) {
            const int per = (stages + sp - 1) / sp;
            if (sp > 1 && (rest == 0 || per < 8 || (int64_t)(sp - 1) * per >= stages)) continue;
            double cost = (double)(whole / slots) * (stages * stage + fixed);
            cost += std::ceil((double)(rest * sp) / slots) * (per * stage + fixed);
            cost *= share;
            if (sp > 1) cost += 9000.0 + (sp + 1) * 4.0 * (double)rest * (64 * wm) * (64 * wn) / 2250.0;
            if (best_cost == 0.0 || cost < 0.98 * best_cost) {
                best = {wm, wn, {(int)tiles, (int)tiles_n, (int)(sp == 1 ? tiles : whole), sp, per}};
                best_cost = cost;
            }
        }
    }
    return best;
}

}  // namespace fpdt_tw
