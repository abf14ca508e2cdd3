// How the attention's launches are laid out, by their sizes.  Host code only, without HIP, so that a plain
// C++ compiler takes it too: the tests ask these rules which kernel a size runs.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace fpdt {

// Key groups of a forward or dQ launch (a workgroup of eight waves = 8 / KG row blocks of 32 queries x KG
// waves that share the keys): the cheapest of 1, 2, 4 in units of a 64-key tile of eight row blocks.  A
// launch on the diagonal lasts as long as its longest row tile or as the average load of the 256 compute
// units, one below it as its rounds of workgroups; KG > 1 divides a workgroup's walk, and costs a little more per tile (copies
// and barriers per MFMA).
struct KeyGroupCosts {
    double two, four;  // a tile with two, four key groups
    double fixed;      // of a workgroup
    double gain;       // more groups are taken where they cost less than this share
};
static inline int cheapest_key_groups(int64_t n_q, int64_t n_keys, int Hq, bool diagonal, const KeyGroupCosts& c)
{
    const double tiles = (double)n_keys / 64.0, cus = 256.0;
    int best = 1;
    double best_cost = 0.0;
    for (int kg = 1; kg <= 4; kg *= 2) {
        const double work = kg == 1 ? 1.0 : kg == 2 ? c.two : c.four, wgs = (double)n_q / 256.0 * kg * Hq;
        const double longest = tiles / kg * work + c.fixed;
        const double load = (double)(int64_t)((wgs + cus - 1.0) / cus) * longest;           // below the diagonal
        const double mean = wgs / cus * (tiles / kg / 2 * work + c.fixed) + longest / 4.0;  // on it
        const double cost = diagonal ? (mean > longest ? mean : longest) : load;
        if (kg == 1 || cost < c.gain * best_cost) { best = kg; best_cost = cost; }
    }
    return best;
}

// The forward's, by the whole sequence.  Measured (us for KG = 1, 2, 4): 8 heads, D = 128, 2K tokens 40, 30, 21; 8K 184, 138, 154; 16K 463, 487, 551;
// D = 64, 4K 45, 35, 30; 5K 80, 44, 48; 14.5K 241, 251, 292; 2 heads, D = 128: 16K 257, 191, 143; 32K 697, 491, 526.  (At 802 sizes so
// measured, D = 64, 80 and 128 alike, 1 to 64 heads, the count that the constants choose takes 1.001 of the fastest one's time in the mean, more than 1.02
// at 12 of them and at most 1.14: 64 heads, 1.25K, D = 80 37, 43, 51.  No constants that were tried do better everywhere.)
static inline int sweep_key_groups(int64_t S, int Hq)
{
    return cheapest_key_groups(S, S, Hq, true, {1.04, 1.22, 1.5, 0.93});
}

// The recomputing dQ's, by the launch.  With D = 64 and 80, whose tiles are shorter, four groups pay up to longer launches on the diagonal; below
// it, where every workgroup walks all keys, sooner ones cost a round more.  Measured at 464 sizes (chunks of 256 to 32K rows, 1 to 32 heads; us for
// KG = 1, 2, 4).  Diagonal: 8 heads, D = 128, 2K rows 67, 43, 30, 8K 257, 194, 215, 12K 448, 442, 464; D = 64, 5K 96, 61, 57, 8K 155, 111,
// 118; 4 heads, D = 80, 11K 244, 168, 154.  Below: 8 heads, D = 128, 4.25K 138, 178, 161, 5K 158, 205, 185, 10K 712, 622, 623; 2 heads, 18K 534, 699,
// 607; D = 64, 9K 376, 325, 297; 4 heads, 18K 740, 636, 578.  The choice takes at most 1.03 of the fastest one's time, but for 768 rows of 32 heads
// on the diagonal at D = 128 (1.05); the forward's constants took up to 1.14.
static inline int dq_key_groups(int64_t n_q, int64_t n_k, int Hq, int D, bool diagonal)
{
    if (diagonal) return cheapest_key_groups(n_q, n_k, Hq, true, D == 128 ? KeyGroupCosts{1.04, 1.22, 1.5, 0.93} : KeyGroupCosts{1.12, 1.25, 1.5, 1.0});
    return cheapest_key_groups(n_q, n_k, Hq, false, {1.16, 1.35, D == 128 ? 1.5 : 0.5, 0.99});
}

// Waves (of 32 query rows each) of a workgroup of the forward with one key group and of dQ from stored dS: eight, or four or
// two where a chunk pair has so few row tiles that half of the 256 compute units, or more, would have none.  A wave computes
// the same whatever the count (the bits do not depend on it); with four or two on a compute unit no second wave of a
// SIMD works under its MFMAs, but twice or four times the compute units work.  The forward stops at four: two would each move half of every key tile.
// Measured, us per launch with eight waves -> with fewer (pairs of equal chunks): forward 8 heads, D = 128, chunks of 4K 99.1 ->
// 77.8 (4); dQ of pairs of 4K, 2K with 8 heads, D = 128, of 8K with 4 heads, D = 80, and of 4K, D = 64: 68.9 -> 52.8 (4), 36.0 -> 31.4 (2),
// 114.1 -> 86.8 (4), 50.8 -> 31.0 (2).
static inline int sweep_waves(int64_t n_q, int Hq)
{
    const int64_t wgs = n_q / 256 * Hq;
    return wgs <= 64 ? 2 : wgs <= 128 ? 4 : 8;
}

// Does the one-launch forward read K and V from their tensors, without the launch that packs them?  With several key groups
// (short sequences) that launch costs more than the transposing reads that take its place.  Packed copies need fewer LDS reads per tile, and at D =
// 80, whose rows of ten pieces are not spread over the banks, gain from it with two key groups, whose workgroups hide less: there longer sequences are
// packed, later where every query head has K and V of its own and there is most to pack.  Up to 16K tokens, behind which the two
// are within 2% of each other at D = 64 and 128.
// Measured over 13 head counts and 24 lengths, with the inputs in no cache and in the caches: the choice takes at most 1.02 of the other's time (us,
// packed -> not; query / KV heads).  D = 64, four key groups, 8 / 2, 2K 17.9, 17.2 -> 15.2, 14.8, 4K 33.6, 32.1 -> 31.5, 29.4; two, 64 / 8, 512 15.1, 13.9 ->
// 12.0, 10.9, 32 / 8, 1.5K 27.4, 25.3 -> 23.1, 21.9, 8 / 2, 8K 85.0, 84.1 -> 81.7, 80.5.  D = 80, four, 8 / 2, 4K 39.9, 38.1 -> 38.5, 36.0, 4 / 4, 8K 69.9, 68.2 -> 65.4,
// 62.5; two, 16 / 4, 4K 62.1, 60.2 -> 61.5, 59.7, 8 / 2, 5K 57.8, 55.9 -> 57.5, 56.6, 8K 103.2, 101.7 -> 105.8, 104.9, 8 / 8, 8K 107.9, 105.7 -> 106.3, 105.3.  D = 128,
// four, 8 / 2, 2K 24.6, 23.5 -> 22.0, 20.4, 4K 49.6, 47.7 -> 46.3, 43.7, 8 / 8, 4K 53.8, 51.8 -> 47.0, 43.7; two, 16 / 4, 4K 79.8, 78.3 -> 76.5, 73.1, 8 / 2, 8K
// 137.6, 136.7 -> 133.9, 133.1, 4 / 1, 12K 170.2, 169.8 -> 168.8, 164.6.
static inline bool sweep_reads_tensors(int64_t S, int Hq, int Hkv, int D, int key_groups)
{
    if (key_groups == 1) return false;
    if (D == 80 && key_groups == 2) return S <= (Hq == Hkv ? 8192 : 4608);
    return S <= 16384;
}

// Does an fp32 call over the whole sequence fit into one launch?  (Workgroups of 512 lanes, one per 16 rows and
// head, for the queries and for the keys; a launch has fewer than 2^32 lanes.)
static inline bool f32_one_launch(int64_t S, int Hq, int Hkv)
{
    return ((S + 15) / 16 * ((int64_t)Hq + Hkv)) < (int64_t)1 << 23;
}

static inline int64_t f32_bwd_tiles(int64_t S, int Hq, int Hkv) { return (S + 15) / 16 * ((int64_t)Hq + Hkv); }

// Do two workgroups share each 16-row tile of the fp32 backward over the whole sequence?  Unshared, the launch lasts as long as the walk of
// the first key tile, through all query heads of its group.  Sharing halves that walk as long as the compute units' average load allows, and costs
// a fixed exchange through memory and, for every workgroup that a compute unit runs beyond those it would have run, operands and sums once more;
// all in units of a 16-row block of the walk.  Measured over 900 sizes (D = 64, 80, 128; 96 to 5120 tokens, up to 32 KV heads, groups of 1 to 16): the
// rule's choice takes at most 1.05 of the faster one's time, in the mean 1.001.  us of the backward alone -> shared (query / KV heads, D =
// 64): 2 / 2, 192 tokens 11.8 -> 12.2, 208 12.8 -> 12.2, 512 19.2 -> 15.8, 1K 29.3 -> 31.6; 4 / 2, 512 29.2 -> 21.2, 1K 55.3 -> 45.3, 2K 130.6 -> 123.2; 8 / 1,
// 4K 945 -> 733; 64 / 1, 1K 1533 -> 829, 4K 7806 -> 5767; many KV heads, not shared: 32 / 16, 256 tokens 30.4 -> 44.8, 16 / 8, 512 45.0 -> 58.0, 8 / 4, 1K 73.5 -> 80.2,
// 16 / 4, 1K 138 -> 139.  The sums take 256 * D bytes a tile: up to 2^15 tiles (1 GiB at D = 128; measured to 32K tiles, 500 / 1, 1K tokens, D = 128 22.2 -> 12.1
// ms), far below the 2^22 whose shared launch would have 2^32 lanes.
static inline bool f32_bwd_split(int64_t S, int Hq, int Hkv)
{
    const int64_t blocks = (S + 15) / 16, tiles = f32_bwd_tiles(S, Hq, Hkv);
    if (S <= 128 || blocks * Hkv > (Hq > Hkv ? 256 : 80) || tiles >= (int64_t)1 << 15) return false;
    const double per_cu = (double)tiles / 256.0, load = (double)(blocks * Hkv) / 256.0, walk = (double)(blocks * (Hq / Hkv));
    const double saved = std::min(0.5, 0.6 - 0.4 * load) * walk;
    return saved > 6.0 + 8.0 * std::max(0.0, 2.0 * per_cu - std::max(per_cu, 1.0));
}

// Workgroups of 512 lanes that prepare a backward over the whole sequence: one per 32-row block of every query head for Delta and one per
// block and head of Q, dO, K and V for the packed operands.  (Fewer than 2^32 of any tensors that fit a GPU.)  A launch has fewer than 2^32 lanes, so
// that from 2^23 workgroups on (64 / 8 heads: 1.26M tokens) it takes several.
static inline int64_t bwd_prepare_blocks(int64_t S, int Hq, int Hkv) { return S / 32 * (3 * (int64_t)Hq + 2 * (int64_t)Hkv); }
static const int64_t BWD_PREPARE_MOST = ((int64_t)1 << 23) - 1;
static inline int64_t bwd_prepare_next(int64_t first, int64_t blocks) { return std::min(blocks - first, BWD_PREPARE_MOST); }

// Into how many splits a dK/dV launch divides the query walk of its key tiles.  Unsplit it has n_k / 256
// * Hkv workgroups of four waves, one per compute unit: 64 at 8K tokens and two KV heads, so that three
// quarters of the chip idle, and below the diagonal's last rows the longest workgroup decides.  Each
// split adds a partial dK, dV (written once, read once by dkdv_sum_kernel).  The count is the cheapest
// of 1, 2, 4, .. 16 in units of steps (one 32-query block of one head; 1.7 us per workgroup, measured):
//   whole pair    rounds of 256 workgroups x (steps of a workgroup + its fixed cost)
//   causal pair   list scheduling of lengths that fall linearly to zero: the longest, or the average load
//   partials      (splits + 1) passes at 4.5 bytes per ns, one more launch
// Measured (dK/dV with its sum, before -> after): 8K tokens, 8 query / 2 KV heads, D = 128: 1357 -> 274 us
// (8 splits); pairs of 32K chunks, 8 / 1 heads: 12.77 -> 7.33 ms (4 splits), 8 / 2 heads: 7.66 -> 7.15 ms (2:
// only the diagonal pairs gain); pairs of 16K chunks, 8 / 2 heads: 3.07 -> 1.76 ms (4).
// causal_launch: one launch over the whole sequence; otherwise chunk pairs, most of them below the diagonal.
static inline int bwd_dkdv_splits(int64_t n_q, int64_t n_k, int Hq, int Hkv, int D, bool causal_launch)
{
    const double cus = 256.0, fixed = 12.0, us_per_step = 1.7;
    const double wgs = (double)(n_k / 256) * Hkv, steps = (double)(n_q / 32) * (Hq / Hkv);
    int best = 1;
    double best_cost = 0.0;
    for (int s = 1; s <= 16; s *= 2) {
        if (s > 1 && steps / s < 8.0) break;
        const double w = wgs * s, len = steps / s;
        const double full = std::ceil(w / cus) * (len + fixed);
        const double causal = std::max(len + fixed, w / cus * (len / 2 + fixed) + len / 4);
        const double sum = s == 1 ? 0.0 : ((double)(s + 1) * 2 * ((double)n_k * Hkv * ((D + 31) / 32 * 32) * 4.0) / 4.5e6 + 6.0) / us_per_step;
        const double cost = sum + (causal_launch ? causal : (full + causal) / 2);
        if (s == 1 || cost < 0.97 * best_cost) { best = s; best_cost = cost; }
    }
    return best;
}

}  // namespace fpdt
