// How the scoring passes (bf16) cut the streamed rows of a head: into segments, whose sums are formed and added up in the
// same way whatever the grid, and segments into runs, one workgroup each.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pulsecol {

constexpr int kScoreTile_bf16 = 64;       // streamed rows per tile
constexpr int kScoreBlock_bf16 = 256;     // stationary rows per workgroup
constexpr int kMaxScoreSegments = 24;

// The segments of a head of n rows: of three tiles or more, as even as they come.  Their number follows from n alone, so
// that a row's or a column's sum has the same bits in every launch that holds its head.  Twelve can be shared out evenly
// among two, three, four or six runs, twenty-four also among eight; eight in the place of twelve would save 32 heads of 4096
// rows, which are not cut, 0.5% and cost elements of 3000 rows in three runs 2.5%.
struct ScoreSegments {
    int count, tiles;
    uint32_t reciprocal;                      // 2^32 / count, rounded up
    __host__ __device__ explicit ScoreSegments(int n) {
        tiles = (n + kScoreTile_bf16 - 1) / kScoreTile_bf16;
        if (tiles >= 192) { count = 24; reciprocal = 178956971u; }
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
inline int score_splits(int64_t blocks, int32_t longest, int head_dim, int compute_units) {
    const ScoreSegments segments(longest);
    const int per_cu = head_dim == 128 ? 2 : 3;
    int best = 1;
    double best_cost = 0.0;
    for (int s = 1; s <= segments.count; ++s) {
        int most = 0;                            // tiles of the longest run
        const uint32_t reciprocal = run_reciprocal(s);
        for (int r = 0; r < s; ++r) {
            const int t = segments.first_tile(segments.first_of_run(r + 1, reciprocal)) - segments.first_tile(segments.first_of_run(r, reciprocal));
            most = t > most ? t : most;
        }
        const double rounds = (double)blocks * s / ((double)per_cu * compute_units), whole = __builtin_floor(rounds);
        const double on_cu = (rounds - whole) * per_cu;               // workgroups to a CU in the last round
        double last = 1.0;
        if (on_cu == 0.0) last = 0.0;
        else if (on_cu <= 1.0) last = per_cu == 2 ? 0.6 : 0.5;
        else if (on_cu <= 2.0 && per_cu == 3) last = 0.75;
        const double cost = (whole + last) * (most + 2.0) + (s > 1 ? 4.0 : 0.0);
        if (s == 1 || cost < best_cost) { best = s; best_cost = cost; }
    }
    return best;
}

}  // namespace pulsecol
