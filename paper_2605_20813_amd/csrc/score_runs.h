// How the scoring passes cut the streamed rows of a head: into segments, whose sums are formed and added up in the
// same way whatever the grid, and segments into runs, one workgroup each.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pulsecol {

constexpr int kScoreTile_bf16 = 64;       // streamed rows per tile (fp32: two blocks of 32 rows)
constexpr int kScoreBlock_bf16 = 256;     // stationary rows per workgroup
constexpr int kScoreBlock_f32 = 128;
constexpr int kMaxScoreSegments = 24;

// The segments of a head of n rows: of three tiles or more, as even as they come.  Their number follows from n alone, so
// that a row's or a column's sum has the same bits in every launch that holds its head.  Twelve can be shared out evenly
// among two, three, four or six runs, twenty-four also among eight; eight in the place of twelve would save 32 heads of 4096
// rows, which are not cut, 0.5% and cost elements of 3000 rows in three runs 2.5%.
// fp32: a tile of 128 stationary rows takes three times as long, so that segments of two tiles are long enough and small grids
// can be cut further: both passes, D = 128, 8 heads of 700 rows in eleven tiles, two segments / four, 41.5 -> 29.1 us.
struct ScoreSegments {
    int count, tiles;
    uint32_t reciprocal;                      // 2^32 / count, rounded up
    __host__ __device__ explicit ScoreSegments(int n, bool f32 = false) {
        tiles = (n + kScoreTile_bf16 - 1) / kScoreTile_bf16;
        if (f32) {
            if (tiles >= 48) { count = 24; reciprocal = 178956971u; }
            else if (tiles >= 30) { count = 12; reciprocal = 357913942u; }
            else if (tiles >= 20) { count = 10; reciprocal = 429496730u; }
            else if (tiles >= 16) { count = 8; reciprocal = 536870912u; }
            else if (tiles >= 12) { count = 6; reciprocal = 715827883u; }
            else if (tiles >= 8) { count = 4; reciprocal = 1073741824u; }
            else if (tiles >= 6) { count = 3; reciprocal = 1431655766u; }
            else if (tiles >= 4) { count = 2; reciprocal = 2147483648u; }
            else { count = 1; reciprocal = 0u; }
        }
        else if (tiles >= 192) { count = 24; reciprocal = 178956971u; }
        else if (tiles >= 36) { count = 12; reciprocal = 357913942u; }
        else if (tiles >= 24) { count = 8; reciprocal = 536870912u; }
        else if (tiles >= 20) { count = 5; reciprocal = 858993460u; }
        else if (tiles >= 16) { count = 4; reciprocal = 1073741824u; }
        else if (tiles >= 12) { count = 3; reciprocal = 1431655766u; }
        else if (tiles >= 8) { count = 2; reciprocal = 2147483648u; }
        else { count = 1; reciprocal = 0u; }
    }
    // first tile of segment i: i * tiles / count (the product is below 2^22, the reciprocal exact enough for 2^28); i = count:
    // the number of tiles
    __host__ __device__ int first_tile(int i) const {
        return i == count ? tiles : (int)(((uint64_t)(uint32_t)(i * tiles) * reciprocal) >> 32);
    }
    // first segment of run r, from the reciprocal of the number of runs (run_reciprocal): r * count / runs
    __host__ __device__ int first_of_run(int r, uint32_t reciprocal_of_runs) const { return (int)((uint32_t)(r * count) * reciprocal_of_runs >> 16); }
};

// 2^16 / runs, rounded up: exact enough for products up to 24 * 24
inline uint32_t run_reciprocal(int runs) { return (65536u + (uint32_t)runs - 1u) / (uint32_t)runs; }

// Runs per head and block for a scoring pass with this many blocks of stationary rows over all heads that stream `longest`
// rows each (blocks of shorter elements count by their share).  A CU holds two workgroups of either pass at D = 128 and
// three at D = 64 (registers); fewer leave its matrix pipe idle while they form weights, a grid smaller than the chip leaves
// CUs idle altogether, and so does the last round of one a little larger.  The rule counts rounds of that many workgroups in
// units of a tile: a run costs the tiles of the longest one and 2 for its start (stationary rows and first tiles from memory), a last
// round that leaves one workgroup to a CU 0.6 (D = 128) or 0.5 of a full one, two of three 0.75, the launches that add the
// segments up 4.  Fitted to 20 grids of 64 to 1024 blocks and 16 to 240 tiles at either head dimension: the choice is within 1.5%
// (D = 128) and 2.2% (D = 64) of the best number of runs on all of them.
// Both passes together, uncut and cut, D = 128: 4 heads of 8192 rows 228 -> 130 us, 3 heads 230 -> 115, 32 heads of 1000
// 38.5 -> 28.5, 20 heads of 8192 666 -> 601, 28 heads 883 -> 832, 10 heads of 15360 1230 -> 1079; D = 64: 4 heads of 8192 190 -> 91,
// 3 heads 191 -> 76, 36 heads of 4100 (612 blocks, less than a round) 238 -> 211, 60 heads of 1500 66.5 -> 58.
struct RunCosts {                             // in tiles
    int per_cu;                               // workgroups that a CU holds
    double one, two;                          // a last round that leaves one to a CU, or two of three, as a part of a full one
    double start, collect;                    // start of a run; the launch that adds the segments up
};
struct Runs { int count; double cost, rounds; int most; };       // most: tiles of the longest run
inline Runs cheapest_runs(int64_t blocks, const ScoreSegments& segments, const RunCosts& costs, int compute_units) {
    Runs best{1, 0.0, 0.0, 0};
    for (int s = 1; s <= segments.count; ++s) {
        int most = 0;                            // tiles of the longest run
        const uint32_t reciprocal = run_reciprocal(s);
        for (int r = 0; r < s; ++r) {
            const int t = segments.first_tile(segments.first_of_run(r + 1, reciprocal)) - segments.first_tile(segments.first_of_run(r, reciprocal));
            most = t > most ? t : most;
        }
        const double rounds = (double)blocks * s / ((double)costs.per_cu * compute_units), whole = __builtin_floor(rounds);
        const double on_cu = (rounds - whole) * costs.per_cu;         // workgroups to a CU in the last round
        double last = 1.0;
        if (on_cu == 0.0) last = 0.0;
        else if (on_cu <= 1.0) last = costs.one;
        else if (on_cu <= 2.0 && costs.per_cu == 3) last = costs.two;
        const double cost = (whole + last) * (most + costs.start) + (s > 1 ? costs.collect : 0.0);
        if (s == 1 || cost < best.cost) best = {s, cost, whole + last, most};
    }
    return best;
}
inline RunCosts run_costs(int head_dim) { return head_dim == 128 ? RunCosts{2, 0.6, 1.0, 2.0, 4.0} : RunCosts{3, 0.5, 0.75, 2.0, 4.0}; }
inline int score_splits(int64_t blocks, int32_t longest, int head_dim, int compute_units) {
    return cheapest_runs(blocks, ScoreSegments(longest), run_costs(head_dim), compute_units).count;
}

// Small bf16 grids run in blocks of 128 rows instead, uncut, with one team of four waves or with two that share out a head's segments:
// nothing is left to be added up by another launch, but a fragment read from LDS feeds one matrix instruction instead of
// two, and a wave's fixed work per tile (barrier, first fragments, check of the blocks) stands against half the products: 12% where the chip
// is full (32 heads of 4096 rows 249 / 281 us).  The rule weighs the microseconds of both passes, fitted to 65 grids of 4 to 1200 blocks
// of 128 rows; q = blocks of 128 per CU, r = rounds of blocks of 256 as above, m = tiles of the longest run:
//   blocks of 256   6.0 + 3.38 r (m + 0.6) / 3.7 + 3.39 r (m + 1.3), 7.7 more where cut
//   one team    7.0 + tiles (1.95 [q / 2] + 1.2 or, above one block to a CU in the last round, 1.88) / 6.7 + tiles (1.31 [q / 2] + 0.96 or 1.42)
//   two teams   9.0 + 1.04 tiles / 9.1 + 0.66 tiles, for up to a block per CU
// Blocks of 256 / one team / two, us: D = 128, 32 heads of 256 15.7 / 11.6 / 13.9, 32 of 640 26.2 / 18.3 / 17.8, 32 of 1000 29.7 / 26.8 / 25.1, 8 of
// 1000 22.1 / 26.6 / 24.1, 48 of 1300 72 / 63 / 85, 32 of 2048 71 / 73 / 80; D = 64, 32 of 1000 24.6 / 22.4 / 19.7.
// Returns the number of teams, 0: blocks of 256 rows.
inline int score_teams(int64_t blocks256, int64_t blocks128, int32_t longest, int head_dim, int compute_units) {
    const ScoreSegments segments(longest);
    if (segments.tiles > 48) return 0;
    const bool wide = head_dim == 128;
    const Runs runs = cheapest_runs(blocks256, segments, run_costs(head_dim), compute_units);
    const double whole = (wide ? 6.0 : 3.7) + 3.38 * runs.rounds * (runs.most + (wide ? 0.6 : 1.3)) + (runs.count > 1 ? 7.7 : 0.0);
    const double q = (double)blocks128 / compute_units, full = __builtin_floor(q / 2.0), rest = q - 2.0 * full;
    const double last = rest == 0.0 ? 0.0 : rest <= 1.0 ? (wide ? 1.2 : 0.96) : (wide ? 1.88 : 1.42);
    const double one = (wide ? 7.0 : 6.7) + segments.tiles * ((wide ? 1.95 : 1.31) * full + last);
    const double two = (wide ? 9.0 : 9.1) + (wide ? 1.04 : 0.66) * segments.tiles;
    const int teams = q <= 1.0 && segments.count > 1 && two < one ? 2 : 1;
    return (teams == 2 ? two : one) < 0.95 * whole ? teams : 0;
}

// fp32: whether the passes run in workgroups of 32 stationary rows, whose eight waves share the streamed rows out (fp32 matrix
// instruction, no barrier on the way): where they all find a CU and a wave has two blocks of 32 rows or three at most.  Beyond, blocks of
// 128 rows in split products and runs.  Both passes, 32 / 128 rows, us: D = 128, 2 heads of 256 22.5 / 27.0, 8 of 384 28.0 / 35.6,
// 32 of 384 43.0 / 35.7, 8 of 700 43.5 / 41.5; D = 64, 2 heads of 256 14.5 / 17.2, 8 of 512 20.3 / 23.3, 8 of 700 25.7 / 28.2, 2 of 3000 74 / 42.
inline bool score_blocks_small_f32(int n, int64_t heads, int head_dim, int compute_units) {
    return n <= (head_dim == 64 ? 768 : 512) && (int64_t)((n + 31) / 32) * heads <= compute_units;
}
// Runs in blocks of 128 rows: the rule above with what a tile of 96 (48) matrix instructions per wave costs, two workgroups counted to a CU at
// either head dimension (at D = 64 it holds three, but with two its matrix pipe is busy: counted as three, with the costs above, the choice
// is no nearer).  On 17 grids of 2 to 64 heads and 900 to 4100 rows the choice is within 8.4% of the best number of runs at D = 64, 1.1% on
// average, and within 5.2% at D = 128, 0.6% on average, but for 2 heads of 3000 rows: in four runs 106 us, in twelve 78.  Both passes,
// uncut / in 2 / 5 / 10 runs, us: D = 128, 8 heads of 1500 rows 112 / 72 / 64 / 71, 16 heads 116 / 117 / 111 / 123; D = 64 68 / 47 / 41 / 43,
// 72 / 70 / 65 / 70.
inline int score_splits_f32(int64_t blocks, int32_t longest, int compute_units) {
    return cheapest_runs(blocks, ScoreSegments(longest, true), RunCosts{2, 0.6, 1.0, 1.0, 1.5}, compute_units).count;
}

}  // namespace pulsecol
