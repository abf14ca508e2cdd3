// How a product of the token-wise library is laid out, by its sizes.  Host code only, without HIP, so that a
// plain C++ compiler takes it too: the tests ask it which tiles and splits a size runs.
#pragma once
#include <stdint.h>

#include <cmath>

namespace fpdt_tw {

constexpr int SK = 32;       // k of an MFMA k-step
constexpr int STAGE_K = 64;  // k of an LDS stage: two k-steps

// The work of a product: the first `whole` of its tiles over all of k, the others divided into `splits`
// ranges of `split_stages` stages (the last one may be shorter).
struct Units {
    int tiles, tiles_n, whole, splits, split_stages;
};

static inline Units make_units(int64_t tiles, int64_t tiles_n, int64_t whole, int splits, int steps)
{
    const int stages = steps * SK / STAGE_K;
    const int per = splits > 1 && stages > 0 ? (stages + splits - 1) / splits : stages;
    const int used = per > 0 ? (stages + per - 1) / per : 1;  // ranges are whole stages
    return {(int)tiles, (int)tiles_n, (int)(used > 1 ? whole : tiles), used, per};
}

// Output tile (64 wmt x 64 wnt), and which tiles are divided along k: the cheapest in units of the core
// clock, from
//   step    the MFMAs of a wave for 32 k (16 clocks each) or the bytes that they copy into LDS: 21 per clock and
//           compute unit
//   unit    a fixed part (first operands, epilogue)
//   rounds  of 256 units (512 where two fit a CU).  Tiles that do not fill the last round are divided, so
//           that it is full and short; with fewer tiles than slots all of them are
//   sums    of the divided tiles: one more launch and (splits + 1) passes over them at about 4.5 bytes per ns
// Measured, all tiles whole -> the rest divided (most of it without a free round at the end, some from the
// epilogues out of step): SwiGLU block at 16K tokens 21.1 -> 18.9 ms, GELU block on 3001 tokens 1562 -> 1458
// us, 4096 x 14336 += 4096 rows 586 -> 475 us.
// (The constants are those of a kernel with stages of 32 k; plan_launch corrects the answer where the present one was measured.)
struct Plan { int wmt, wnt; Units u; };
static inline Plan plan_product(int64_t M, int64_t N, int steps)
{
    static const int shapes[][2] = {{4, 4}, {3, 4}, {2, 4}, {1, 4}, {2, 2}};
    Plan best = {4, 4, {}};
    double best_cost = 0.0;
    for (const auto& sh : shapes) {
        const int wm = sh[0], wn = sh[1];
        const double mfma = 64.0 * wm * wn + 100.0, copies = 192.0 * (wm + wn);
        const double step = mfma > copies ? mfma : copies, fixed = 1200.0 + 160.0 * wm * wn;
        const int slots = wm * wn <= 4 && wn == 2 ? 512 : 256;
        const double share = slots / 256.0;
        const int64_t tiles_n = (N + 64 * wn - 1) / (64 * wn), tiles = (M + 64 * wm - 1) / (64 * wm) * tiles_n;
        if (tiles > (int64_t)1 << 30) continue;
        const int64_t rest = tiles % slots, whole = tiles - rest;
        for (int sp = 1; sp <= 16; ++sp) {
            const int per = (steps + sp - 1) / sp;
            if (sp > 1 && (rest == 0 || per < 8 || (int64_t)(sp - 1) * per >= steps)) continue;
            double cost = (double)(whole / slots) * (steps * step + fixed);
            cost += std::ceil((double)(rest * sp) / slots) * (per * step + fixed);
            cost *= share;
            if (sp > 1) cost += 9000.0 + (sp + 1) * 4.0 * (double)rest * (64 * wm) * (64 * wn) / 2250.0;
            if (best_cost == 0.0 || cost < 0.98 * best_cost) {
                best = {wm, wn, make_units(tiles, tiles_n, sp == 1 ? tiles : whole, sp, steps)};
                best_cost = cost;
            }
        }
    }
    return best;
}

// Clocks of a launch: `whole` tiles over all of k and `rest` tiles in `sp` splits each (plan_launch says from what)
static inline double launch_cost(int wm, int wn, double whole, double rest, int sp, int steps)
{
    const bool two = wm * wn <= 4;
    const double slots = two ? 512.0 : 256.0, per = sp == 1 ? steps : (double)(((steps + sp - 1) / sp + 1) / 2 * 2);
    const double mfma = two ? 161.0 * wm * wn + 158.0 : 64.0 * wm * wn + 116.0, copies = (two ? 175.0 : 85.0) * (wm + wn);
    const double step = mfma > copies ? mfma : copies, fixed = two ? 8100.0 + 1385.0 * wm * wn : 6900.0 + 1630.0 * wm * wn;
    const double units = rest * sp, full = std::floor(units / slots), last = units - full * slots;
    double c = whole / slots * (steps * step + fixed) + full * (per * step + fixed) + 7600.0;
    if (last > 0.0) c += (per * step + fixed) * (two && last <= 256.0 ? 0.56 : 1.0);
    if (sp > 1) c += 3800.0 + (sp + 1) * 4.0 * rest * (64 * wm) * (64 * wn) / 8300.0;
    return c;
}

// What a launch runs: plan_product's answer, or another tile and division that the measured times of 68 products
// (M and N of 300 .. 16384, k of 65 .. 15776, every tile and division; 2.8% above the best of them on average,
// plan_product alone 8.2%) put at least 5% below it.  The terms are plan_product's, but with two workgroups on
// a compute unit (128 x 128 and 64 x 256 tiles) the MFMAs of one run under the copies and the epilogue of the other,
// which decides where k is short: us, plan_product's answer -> this, 7416 x 1816 x 250 39.9 -> 26.9, 1680 x 4848 x
// 269 29.2 -> 20.7, 1920 x 2512 x 667 23.0 -> 19.3, 6144 x 4096 x 4096 (384 tiles of 256 x 256, the rest in two splits,
// -> 512 tiles of 192 x 256) 177 -> 161.
// It stands for products with a side of less than 512 (4000 of them: 5.4% above the best plan on average, launch_cost's choice
// 5.5%), and for whole tiles with a rest that is divided by three or more (at most a third of a round, within 4% of the best).
static inline Plan plan_launch(int64_t M, int64_t N, int steps)
{
    static const int shapes[][2] = {{4, 4}, {3, 4}, {2, 4}, {1, 4}, {2, 2}};
    const Plan first = plan_product(M, N, steps);
    if (first.u.tiles == 0 || M < 512 || N < 512 || (first.u.splits > 2 && first.u.whole > 0)) return first;
    auto cost = [&](int wm, int wn, double whole, double rest, int sp) { return launch_cost(wm, wn, whole, rest, sp, steps); };
    Plan best = first;
    double best_cost = 0.0;
    for (const auto& sh : shapes) {
        const int wm = sh[0], wn = sh[1], slots = wm * wn <= 4 ? 512 : 256;
        const int64_t tiles_n = (N + 64 * wn - 1) / (64 * wn), tiles = (M + 64 * wm - 1) / (64 * wm) * tiles_n;
        if (tiles > (int64_t)1 << 30) continue;
        const int64_t rest = tiles % slots, whole = tiles - rest;
        for (int sp = 1; sp <= 16; ++sp) {
            const int per = ((steps + sp - 1) / sp + 1) / 2 * 2;
            if (sp > 1 && (rest == 0 || per < 8 || (int64_t)(sp - 1) * per >= steps / 2 * 2)) continue;
            const double c = cost(wm, wn, (double)whole, (double)rest, sp);
            if (best_cost == 0.0 || c < best_cost) {
                best = {wm, wn, make_units(tiles, tiles_n, sp == 1 ? tiles : whole, sp, steps)};
                best_cost = c;
            }
        }
    }
    const int slots = first.wmt * first.wnt <= 4 ? 512 : 256;
    const int64_t rest = first.u.tiles % slots;
    return best_cost < 0.95 * cost(first.wmt, first.wnt, (double)(first.u.tiles - rest), (double)rest, first.u.splits) ? best : first;
}

// Clocks of the products of `n` rows of logits, `step` rows at a time
static inline double loss_cost(int64_t n, int64_t step, int64_t vocab, int64_t hidden)
{
    const int steps = (int)((hidden < SK ? SK : hidden) / SK);
    auto one = [&](int64_t rows) {
        const Plan p = plan_launch(rows, vocab, steps);
        const int rest = p.u.tiles % (p.wmt * p.wnt <= 4 ? 512 : 256);
        return launch_cost(p.wmt, p.wnt, p.u.tiles - rest, rest, p.u.splits, steps);
    };
    return (n >= step ? (double)(n / step) * one(step) : 0.0) + (n % step ? one(n % step) : 0.0);
}

// Rows of logits that the loss computes at a time, of `n` rows of which `full` have room: whole tile rows (256), or as many as
// there is room for, where that is one product or costs at least a sixteenth less.  Measured (us, as whole tile rows | as many
// as have room): forward, 300 rows, hidden 2048, vocabulary 8000: 52.5 | 38.6; hidden 1024, 32000: 61.5 | 43.0; 3396 rows, room
// for 1273, 4096, 16384: 428 | 470; with gradients, 2075 rows, room for 390, 2048, 50304: 1426 | 1495; 1602 rows, room for 400,
// 1024, 8000: 261 | 245.
static inline int64_t loss_step(int64_t n, int64_t full, int64_t vocab, int64_t hidden)
{
    const int64_t tiles = full / 256 * 256;
    if (tiles == 0 || n <= full) return full;
    return 15 * loss_cost(n, tiles, vocab, hidden) <= 16 * loss_cost(n, full, vocab, hidden) ? tiles : full;
}

// Rows whose logit gradients the loss gathers before it multiplies them: a chunk's `c`, or where at least two chunks make 2
// `hidden` rows, as many groups as it takes at 2 `hidden` rows each, of about the same size, in whole tiles of 256 rows
// unless that would be more than 2 `hidden`, which bounds the scratch.
static inline int64_t loss_group(int64_t rows, int64_t c, int64_t hidden)
{
    if (hidden < c) return c;
    const int64_t groups = (rows + 2 * hidden - 1) / (2 * hidden), even = (rows + groups - 1) / groups, tiles = (even + 255) / 256 * 256;
    return tiles <= 2 * hidden ? tiles : even;
}

}  // namespace fpdt_tw
