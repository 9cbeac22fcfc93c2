// Which launch a call takes, from its sizes: plain functions of the host, without HIP, so that the
// rules can be read and tested where there is no GPU.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <cmath>

// ---- attention: blocks of 256 (token, query head) columns, n_row_tiles per kv head, up to t_max key
// tiles each.  WHOLE: a workgroup per block.  CUT: `pieces` workgroups per block, equal runs of its key tiles.
// EVEN: `ranges` workgroups over the key tiles of all blocks, no range shorter than per_min units. ----
#define CC_ATTN_EVEN_START 5        // units that a block costs in an even grid besides its key tiles
#define CC_ATTN_EVEN_MAX_TILES 1024 // row tiles whose first units fit an even grid's LDS table
enum { CC_ATTN_WHOLE = 0, CC_ATTN_CUT = 1, CC_ATTN_EVEN = 2 };
struct cc_attn_plan {
    int kind, pieces, ranges, per_min;
};

// Shortest range of an even grid, in units: the pieces of a block are merged one batch after the other,
// so a longer block takes longer ranges (12000 slots, 2 blocks: ranges of 2, 5, 7 and 12 units 30.6 / 22.0 / 22.2 /
// 25.6 us; 592 slots, 8 blocks: 2, 3 and 5 units 18.2 / 18.6 / 20.9).
inline int cc_attn_even_min(int64_t t_max) { return std::max(2, (int)(0.45 * std::sqrt((double)t_max) + 0.5)); }

// Most workgroups that a call of up to `tiles` blocks over up to t_max key tiles leaves pieces with; two
// slots of the workspace each.
inline int cc_plan_attn_workgroups(int n_cu, int64_t tiles, int64_t t_max) {
    return (int)std::min<int64_t>(n_cu, std::max(tiles * (t_max + CC_ATTN_EVEN_START) / 2 + 1, 8 * tiles));
}

// Estimated microseconds of the three, the least is taken; a merge has to save 15 %.
//   a key tile of 256 columns costs 1.75 (d_h = 128) or 1.5 (64) of a workgroup's time, the call itself 8;
//   pieces cost a merge, 0.6 and 0.2 per MB of fp32 sums (written and read at 5 TB/s);
//   an even grid costs 6 more (its table of units, ranges that walk their keys out of step);
//   a block is half of the longest on average, more where there are few (rows spread over the
//   context), and the largest share of a workgroup 20 % above the mean.
// Measured over 750 calls (8 head layouts, 70 to 40000 slots, 16 to 2600 rows, up to 520 blocks), event
// microseconds, whole / cut (its best) / even (its best):
//   64 query heads of 8, d_h = 128:  N = 330, 256 rows 20.5 / 21.1 / 26.8;  N = 592, 512 rows 26.4 / 29.1 / 33.6;
//   N = 1104, 16 rows 29.6 / 14.5 / 15.6, 256 rows 35.5 / 27.5 / 28.8;  N = 2112, 1024 rows 56.5 / 63.6 / 64.9;  N = 4224,
//   512 rows 92.3 / 63.6 / 56.7;
//   28 of 4, d_h = 128, N = 20000, 1536 rows 390 / 254 / 213;  32 of 32, N = 20000, 16 rows 363 / 62 / 67.
// The choice is within 1.1 % of the best of all tried, on average.
// `wide`: token strides that need 64-bit lane offsets, for which there is no even grid.
inline cc_attn_plan cc_plan_attention(int n_cu, int n_row_tiles, int H_kv, int d_h, int t_max, int slots, bool wide,
                                      int override_pieces) {
    const int64_t n_wg = (int64_t)n_row_tiles * H_kv;
    const int64_t most_units = n_wg * (t_max + CC_ATTN_EVEN_START);
    const bool even_ok = !wide && n_row_tiles <= CC_ATTN_EVEN_MAX_TILES && most_units < (1 << 30) && slots >= 2;
    cc_attn_plan p = {CC_ATTN_WHOLE, 1, 0, 0};
    auto even = [&](int per_min, int64_t most_ranges) {
        p.kind = CC_ATTN_EVEN;
        p.per_min = per_min;
        p.ranges = (int)std::min<int64_t>({most_units / per_min + 1, (int64_t)slots / 2, most_ranges});
    };
    if (override_pieces == 1) return p;
    if (override_pieces > 1) {
        const int cut = (int)std::min<int64_t>({override_pieces, t_max, slots / n_wg});
        if (even_ok) even((t_max + override_pieces - 1) / override_pieces, slots);
        else if (wide && cut > 1) p.kind = CC_ATTN_CUT, p.pieces = cut;
        return p;
    }
    const double tile_us = d_h == 128 ? 1.75 : 1.5, slot_us = 0.2 * 256 * (d_h + 4) * 4 / 1e6;
    const double mean = 1.2 * (n_row_tiles + 1) / (2.0 * n_row_tiles);       // of t_max, in a block
    const double share = mean * n_wg / n_cu;                                 // of t_max, of a CU
    double best = 0.85 * (8.0 + tile_us * t_max * std::max(1.0, share));
    for (int s = 2; s <= 8 && s <= t_max && t_max > 3; ++s) {       // three tiles are loaded together anyway
        if (n_wg * s > n_cu || n_wg * s > slots) break;
        const double t = 8.6 + tile_us * ((t_max + s - 1) / s) + slot_us * n_wg * s;
        if (t < best) best = t, p.kind = CC_ATTN_CUT, p.pieces = s;
    }
    const double units = std::max<double>(cc_attn_even_min(t_max), share * (t_max + CC_ATTN_EVEN_START));
    const double pieces = std::min<double>(n_cu, mean * most_units / units);
    if (even_ok && 14.6 + tile_us * units + slot_us * pieces < best) even(cc_attn_even_min(t_max), n_cu);
    return p;
}
