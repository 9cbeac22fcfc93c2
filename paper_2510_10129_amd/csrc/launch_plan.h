// Which launch a call takes, from its sizes: plain functions of the host, without HIP, so that the
// rules can be read and tested where there is no GPU.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "cacheclip.h"

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

// ---- GEMM: C[M, N] = A[M, K] B[N, K]^T in row x column tiles.  tile: 'b' 256x256 (ping-pong loop, 8 waves, least
// LDS and L2 traffic per flop, one workgroup per CU), 'h' 256x128 (duo loop, 8 waves of 64x64, one per CU), 's' 128x128 (duo loop, 8 waves of 64x64 in two groups along K, one per
// CU; ring loop, 4 waves of 64x64, two per CU), 't' 64x128 (thin loop).
// Where K is not a multiple of 128 the 256x256 and 128x128 shapes run the staged loop.  shares: of K ('b', 'h': of
// the last round's tiles only; 't': of all), in whole groups ('t': slices of 64 columns), the first ones longer by one where
// they do not divide. ----
#define CC_GEMM_SLICE 32            // K columns of a ring slice
#define CC_GEMM_GROUP 128           // the ring and ping-pong loops take K in groups of this many columns
#define CC_THIN_M 64
#define CC_THIN_N 128
struct cc_gemm_plan {
    char tile;
    bool ring;
    int shares;
    bool duo;       // 's': the duo loop (else the ring or staged loop); 'h' always
    bool stream;    // 't': the weights go past the caches
    bool staged_parts;   // 'b' in shares: the sums leave through LDS instead of from the accumulators
};
// Sums of shares go through LDS where an eighth or more of the row tiles' rows lie past M (see gemm_pingpong_parts_kernel).
// From the accumulators / through LDS: d = 8192, down, 65 rows 123 / 93.2, 128 125 / 104; d = 3584, down, 300 rows 79.0 / 68.3, 384 86.6 / 71.6,
// 448 81.7 / 76.2, 560 95.0 / 90.6; 640 and 850 rows within 1 %;  d = 4096, down, 480 rows 67.6 / 71.2, 512 70.5 / 73.4; QKV 768 56.2 / 58.7.
inline bool cc_gemm_stages_parts(int M) {
    const int rows = (M + 255) / 256 * 256;
    return 8 * (int64_t)(rows - M) >= rows;
}
// Weights that one row tile reads, each line once, go past the caches, but for widths up to 640: a layer of those takes 13 MB at
// most, and the 256 MB cache holds two dozen until their next call.  us of a whole layer, distinct layers in a row, all weights
// past the caches / none (4224 slots; 64 rows, 8 rows):  6 layers of d = 4096 127.1 / 136.3, 107.6 / 116.9;  16 of 2048 78.7 / 81.0, 62.2 / 65.4;
// 24 of 1024 61.1 / 62.5, 50.4 / 52.3;  24 of 768 58.9 / 60.7, 48.8 / 50.9;  24 of 576 54.9 / 53.8, 45.4 / 44.2;  24 of 512 50.8 / 48.5, 42.0 / 39.9.
// QKV and O of d = 4096 by themselves are faster through the caches at 64 rows (18.7 against 19.7 us, 15.7 against 17.8); the layer
// is not (129.1 against 127.9).
inline bool cc_gemm_streams(int M, int N, int K) {
    return M <= CC_THIN_M && (N < K ? N : K) > 640;
}
inline cc_gemm_plan cc_plan_gemm(int n_cu, int M, int N, int K, int64_t lda, int64_t ldb, bool ws, int64_t ws_floats,
                                 const cc_launch_override& ovr) {
    const char force = (char)ovr.gemm_tile;                   // 0: the launcher's choice
    auto tiles_of = [&](int bm, int bn) { return (long)((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    auto rounds_of = [&](int bm, int bn) { return (tiles_of(bm, bn) + n_cu - 1) / n_cu; };   // one tile per CU
    // ring loop: whole groups of slices, 32-bit lane offsets within a tile's rows
    const bool ring = K % CC_GEMM_GROUP == 0 && lda * 256 * 2 < (1ll << 31) && ldb * 256 * 2 < (1ll << 31) && ovr.gemm_staged != 1;
    // Microseconds of a round of workgroups (a grid runs as a whole number of them): the ends of its
    // tiles, and 32 columns of K; and what both cost more where every CU has a tile (power, and the
    // traffic behind the caches) in proportion to the CUs that have one.
    // Fitted to event times of the four projections of nine models (d = 256 to 8192, f = 1024 to 28672), 1 to
    // 8320 rows, weights cold, every shape and most shares forced; 256x128 and thin tiles fitted again with their present loops, to
    // 1572 calls of those and two models without the ring loops: the choice 0.6 % above the fastest on average (1.3 % before).
    // The rates without the ring loops are of 364 calls of such models: there the large tile is no
    // faster than it was (M = 3000, N = 10880, K = 1984: three rounds of 256x256 179 us, four of 128x128 147).
    // The ends count where K is short (K = 256, 2048 columns, M = 5120: 256x256 tiles 21.4 us, 128x128 in the ring 18.4, with
    // two of its tiles on a CU).
    struct Round { double ends, slice, more_ends, more_slice; };
    const Round rb = ring ? Round{7.1, 0.41, 7.3, 0.151} : Round{21.6, 0.736, 0, 0},
                rh = {6.1, 0.323, 2.87, 0.063}, rsd = {7.6, 0.21, 0, 0.047};
    // 128x128 tiles in the ring or staged loop: two on a CU, or one where there are no more
    const Round rs = ring ? Round{2.3, 0.6, 0, 0} : Round{11.9, 0.451, 0, 0},
                rs_short = ring ? Round{3.9, 0.34, 2.1, 0.104} : Round{4.6, 0.497, 0, 0};
    const double slices = (double)K / CC_GEMM_SLICE;
    auto us = [&](const Round& r, double fill, int share) {   // a round with tiles on `fill` of the CUs, 1 / share of K
        const int groups = K / CC_GEMM_GROUP;                 // the longest share
        const double sl = share == 1 ? slices : (double)((groups + share - 1) / share * (CC_GEMM_GROUP / CC_GEMM_SLICE));
        return r.ends + r.more_ends * fill + (r.slice + r.more_slice * fill) * sl;
    };
    auto grid_us = [&](const Round& r, int bm, int bn) {
        const double fill = (double)tiles_of(bm, bn) / n_cu;  // of all its rounds
        return rounds_of(bm, bn) * us(r, 0, 1) + fill * (us(r, 1, 1) - us(r, 0, 1));
    };
    const long st = tiles_of(128, 128), s_last = st % (2 * n_cu);
    const double tb = grid_us(rb, 256, 256);
    const double ts = st / (2 * n_cu) * us(rs, 1, 1) +
                      (s_last == 0 ? 0.0 : s_last <= n_cu ? us(rs_short, (double)s_last / n_cu, 1) : us(rs, 1, 1));
    char pick = tb <= ts ? 'b' : 's';
    double t_best = std::min(tb, ts);
    bool duo_s = false;
    const bool half_tiles = ring && !ovr.gemm_mfma32;           // 256x128 has no other loop than the duo loop
    if (ring) {
        const double tsd = grid_us(rsd, 128, 128), th = grid_us(rh, 256, 128);
        duo_s = ovr.gemm_staged ? ovr.gemm_staged == 2 : tsd < ts;
        if (tsd < t_best) pick = 's', t_best = tsd;
        if (half_tiles && th < t_best) pick = 'h', t_best = th;
    }
    if (force == 'b' || force == 's' || (force == 'h' && half_tiles)) pick = force;
    // Split-K for the part of a grid that leaves most CUs idle: the tiles of a last round that
    // fills at most half the chip (all tiles, if there is no full round) are computed by S
    // workgroup rows, each over a share of K's groups, with S x tiles <= CUs, and a finishing pass; the full
    // rounds before them run as a launch of their own.  256-row tiles only.  The extra launches and
    // the shares' traffic cost 4.45 us and 6.75 TB/s.
    // Shares need not be equal: 84 tiles of 256x256 over 148 groups take 2 shares, 168 workgroups, if they have to be,
    // 3 and 252 if not (M = 1523, N = 3584, K = 18944: 203 -> 173 us with the finishing pass).
    int S = 1;
    if (ring && ws) {
        const int groups = K / CC_GEMM_GROUP;
        struct Shape { char tile; int bm, bn; const Round& r; };
        const Shape shapes[2] = {{'b', 256, 256, rb}, {'h', 256, 128, rh}};
        auto rem_of = [&](const Shape& h) {
            const long tiles = tiles_of(h.bm, h.bn);
            return (int)(tiles % n_cu == 0 && tiles > 0 ? n_cu : tiles % n_cu);
        };
        auto split_ok = [&](const Shape& h, int sp, int k_min) {
            const int rem = rem_of(h);
            return groups / sp * CC_GEMM_GROUP >= k_min && (long)rem * sp <= n_cu &&
                   (double)sp * rem * (256.0 * h.bn) <= (double)ws_floats;          // slots of 256 rows
        };
        if (ovr.gemm_splitk > 0) {
            const int sp = ovr.gemm_splitk;
            const Shape& h = shapes[force == 'h' && half_tiles];
            if (sp > 1 && sp <= 16 && split_ok(h, sp, CC_GEMM_GROUP)) S = sp, pick = h.tile;
        } else if (!force && !ovr.gemm_staged) {
            for (const Shape& h : shapes) {
                if (h.tile == 'h' && !half_tiles) continue;
                const long full_rounds = rounds_of(h.bm, h.bn) - 1;
                const int rem = rem_of(h);
                for (int sp = 2; sp <= 16; ++sp) {
                    if (!split_ok(h, sp, 512)) continue;
                    const double t = full_rounds * us(h.r, 1, 1) + us(h.r, (double)rem * sp / n_cu, sp) + 4.45 +
                                     (double)sp * rem * (256.0 * h.bn) * 4 / 6.75e6;
                    if (t < t_best) t_best = t, S = sp, pick = h.tile;
                }
            }
        }
    }
    // Few rows: 64x128 tiles (gemm_thin_kernel), K cut into shares where the grid leaves CUs idle.
    // From the same measurements: 3.1 us for the ends of a round's tiles, 0.41 per 64 columns, the weights no faster
    // than 7.7 TB/s, a finishing pass 2.3 and its rows' traffic at 3.4; the estimate has to be 2 % below the other.
    // Event microseconds (2.5 of them the events' own), d = 4096, f = 14336, 870 MB of other weights between two
    // reads of one, the best of the thin tiles and of the larger ones:  M = 64: QKV 19.7 / 25.7, O 17.8 / 22.5, gate/up
    // 41.2 / 46.3, down 28.3 / 39.0;  M = 128: 24.8 / 27.0, 18.6 / 23.1, 67.3 / 52.9, 39.9 / 41.9;  M = 192: 33.0 / 30.4, 24.1 /
    // 25.5, 92.4 / 65.0, 56.6 / 45.3.
    const long thin_tiles = tiles_of(CC_THIN_M, CC_THIN_N);
    const bool thin_ok = lda * CC_THIN_M * 2 < (1ll << 31) && ldb * CC_THIN_N * 2 < (1ll << 31);
    auto thin_split_ok = [&](int sp) {
        return K / 64 >= sp && ws && (double)sp * thin_tiles * (CC_THIN_M * CC_THIN_N) <= (double)ws_floats;
    };
    if (thin_ok && force == 't') {
        const int sp = ovr.gemm_splitk;
        return {'t', ring, sp > 1 && thin_split_ok(sp) ? sp : 1, false, cc_gemm_streams(M, N, K), false};
    }
    if (thin_ok && !force && !ovr.gemm_staged && !ovr.gemm_mfma32 && ovr.gemm_splitk == 0) {
        for (int sp = 1; sp <= 16; ++sp) {
            if (sp > 1 && (!thin_split_ok(sp) || K / sp < 256 || thin_tiles * sp > n_cu)) continue;
            const long rounds = (thin_tiles * sp + n_cu - 1) / n_cu;
            double t = rounds * ((K / 64 + sp - 1) / sp * 0.41 + 3.1);
            t = std::max(t, 2.0 * N * K / 7.7e6);
            if (sp > 1) t += 2.3 + (double)sp * M * N * 8 / 3.4e6;
            if (t < 0.98 * t_best) t_best = t / 0.98, pick = 't', S = sp;
        }
    }
    return {pick, ring, S, pick == 'h' || (pick == 's' && duo_s), pick == 't' && cc_gemm_streams(M, N, K),
            pick == 'b' && S > 1 && cc_gemm_stages_parts(M)};
}

// ---- selection: one workgroup up to CC_SEL_ONE_MAX tokens (6.5 us and 0.36 us more per 1024 tokens), beyond that four launches
// over tiles (21 us and next to nothing more), which take the ranges of the keys and their workspace.  One workgroup / four
// launches, microseconds: scores of a softmax 16384: 12.1 / 21.0, 20480: 13.8 / 21.2; crowded by a zero 20480: 23.9 / 30.  The line
// lies where the one workgroup's arrays end (five rows of 4096 keys in LDS, 95 KB with the rest), not where the two meet: by these
// rates that would be further up, but no larger one is built or measured. ----
#define CC_SEL_ONE_MAX 20480
inline bool cc_select_uses_ranges(int T) { return T > CC_SEL_ONE_MAX; }

// ---- row norms: waves that share a row of d elements of elem_bytes (2: bf16 hidden rows, 4: the fp32 residual; a
// workgroup is four waves, 8 of them are resident on a CU).  Event microseconds with one, two and four waves:
//   short rows leave waves without a chunk:  d = 576 fp32, M = 16384 13.2 / 12.6 / 15.5;  d = 1024 bf16 16.1 / 16.3 / 20.2;
//   few rows want every wave:  d = 4096 bf16, M = 64 6.7 / 6.1 / 6.2, 884 9.8 / 8.0 / 7.3;  d = 8192 fp32, 64 11.2 / 6.9 / 6.4,
//   2047 24.0 / 18.7 / 18.4, 16384 180 / 168 / 160;
//   bf16 rows a little past one round of workgroups pay for the second:  d = 4096, M = 4096 15.3 / 14.7 / 17.1, 8192
//   24.7 / 27.6 / 27.5, 12000 39.0 / 37.3 / 36.9;  d = 8192, M = 3000 20.8 / 19.3 / 22.0, 6000 42.8 / 39.5 / 38.9;  d = 1088, M = 16384
//   18.7 / 19.0 / 21.1. ----
inline int cc_norm_waves(int n_cu, int M, int d, int elem_bytes) {
    if (d <= 1024) return 1;
    if (elem_bytes == 4 || M <= 8 * n_cu) return 4;
    if (d <= 1536 || (d <= 4096 && M <= 40 * n_cu)) return 1;
    return d <= 8192 && M <= 16 * n_cu ? 2 : 4;
}

// ---- cache assembly: destination rows of `width` elements (all heads) that a wave moves, of n_rows.  Event
// microseconds with 4, 8 and 16:  width 1024 (8 heads of 128): 1072 rows 7.2 / 7.7 / 9.7, 4144: 11.6 / 10.6 / 12.7, 65584: 98 /
// 94 / 99;  width 4096: 1072: 15.6 / 18.4 / 26.3, 28720: 183 / 186 / 200, 65584: 402 / 420 / 459;  width 512 (8 of 64): 4144: 9.4 /
// 9.1 / 9.8, 16432: 20.5 / 18.6 / 16.9, 65584: 64 / 56 / 53;  width 64: 4144: 6.4 / 6.5 / 6.3, 65584: 28.6 / 19.0 / 13.8. ----
inline int cc_asm_rows(int64_t n_rows, int width) {
    if (n_rows < 2048) return 4;
    return width >= 1024 || n_rows < 6000 ? 8 : 16;
}
