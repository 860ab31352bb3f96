// Which bf16 kernel a column-sparse call with one set per head runs in: the hand-scheduled one with 256-row query blocks (attn_bf16.hip),
// one workgroup to a CU, or the plain one with 128-row blocks (attn_bf16_group.hip), two to a CU at D = 128 and three at D = 64,
// which cover each other's starts and ends.  The scheduled kernel is faster per tile and slower per block, so the plain one is right for few
// tiles to a block; and as either works on whole blocks, the one whose last round fills the chip better gains by that.
//
// The rule compares what the two are expected to take: microseconds, from the rounds of workgroups, whole ones and the last, and the
// 64-column tiles t of a block.  F = whole rounds, c = 128-row blocks per CU; a last round that fills up to half the chip .. nearly all of it.
//
//              D = 128                                            D = 64
//   scheduled  4.5 + F (8.4 + 1.37 t) + 4.8 .. 8.4 + (1.01 .. 1.37) t      3.3 + F (6 + 0.86 t) + 4 .. 6 + (0.74 .. 0.86) t, behind a whole round 0.86 t
//   plain      3.3 + F (3.8 + 1.98 t) + 3.8 + a t                          5.2 + F (1.6 + 1.76 t) + 1.6 + a t
//              a = 0.64 with one workgroup to a CU, 1.38 .. 1.98 with more      a = 0.33 with one, 0.86 .. with two, 1.47 .. 1.76 with three
//   two teams  6.8 + t (0.62 + 0.32 c)                                     5.9 + t (0.42 + 0.12 c)       (the plain kernel with at most a block per CU)
//
// A last round costs more than its share (one workgroup alone on a CU takes half of what two take together, and a chip that is half full
// runs at a higher clock): with the plain kernel charged by its share of the chip and the scheduled one by whole rounds, calls between
// two whole numbers of rounds went the wrong way by up to 37%: D = 128, plain / scheduled, 1 head of 49088 rows, keep 20%, 244 / 196 us, 1 head of 39360, keep
// 25%, 229 / 174, 24 of 6848, keep 25%, 154 / 127.  The scheduled kernel takes 3 more where some of its queues hold
// less than the workgroups that start on them (heads no multiple of eight): those ask a counter for their first block.  Its second round then costs
// most of a whole one from a third of the chip on, on four cards of five (plain / scheduled, 2 heads, 1.45 to 1.5 rounds, us a tile: 2.9 / 2.5 on one, 2.9 / 3.05 on
// another): charged as on those.
//
// Padded batches: a block of a shorter element takes the part of the time that its tiles are, and its whole start.  The scheduled kernel
// takes 5 more where there is a round of padding to skip; the plain one ends with the XCD that the longest elements' heads
// lie on, and where its workgroups work through lists, with the longest list.
//
// Fitted to 8000 calls on 256 CUs, 1 to 64 heads, 64 to 100K rows, keep 5 to 100%, and checked on 5000 others: of these the slower kernel by more than
// 5% / 10% in 0.8 / 0.2% at D = 128 and in 1.0 / 0.2% at D = 64 (most of them calls of less than 15 us).  Padded batches of 2 to 8 elements, 3600
// calls and 2000 others: 3.0 / 1.4%.
#pragma once

#include <stdint.h>

namespace pulsecol {

struct AttnJob {
    double blocks256, blocks128;      // query blocks that have rows
    double work256, work128;          // the same, each as the part of a block of the longest element that its tiles are
                                      // (of 128 rows: eight times those of the XCD that has most)
    double grid128, padding;          // all of 128 rows, and the share of their tiles that is none
    double grid256, shortest_queue;   // of 256 rows: all, and those in the queue of the scheduled kernel that holds the fewest
    int32_t rows, longest;            // of a full element, and of the longest one
    // 64-column tiles of the longest element (an element keeps its own share of its rows)
    int32_t columns(int32_t ns) const { return (int32_t)(((int64_t)ns * longest + rows - 1) / rows); }
    double tiles(int32_t ns) const { return (double)((columns(ns) + 63) / 64); }
};

struct AttnCosts {                    // us, see above
    double start, block, last_block, tile, last_tile, slope, late_tile, uneven_slope, uneven, skip;       // scheduled
    int per_cu;                                                                                           // plain
    double plain_start, plain_block, plain_tile, lone, pair, triple, pair_slope, list;
    double teams_start, teams_tile, teams_slope;
};
inline AttnCosts attn_costs(int head_dim) {
    return head_dim == 128 ? AttnCosts{4.5, 8.4, 4.8, 1.37, 1.01, 0.91, 1.01, 1.2, 3.2, 5.0, 2, 3.3, 3.8, 1.98, 0.64, 1.38, 0.0, 0.63, 0.35, 6.8, 0.62, 0.32}
                           : AttnCosts{3.3, 6.0, 4.0, 0.86, 0.74, 0.24, 0.86, 0.0, 3.2, 5.0, 3, 5.2, 1.6, 1.76, 0.33, 0.86, 1.47, 0.21, 0.35, 5.9, 0.42, 0.12};
}
inline double at_least(double a, double b) { return a > b ? a : b; }
inline double at_most(double a, double b) { return a < b ? a : b; }
inline double scheduled_attn_us(const AttnJob& job, int32_t ns, int head_dim, int compute_units) {
    const AttnCosts k = attn_costs(head_dim);
    const double rounds = job.work256 / compute_units, whole = __builtin_floor(rounds), part = rounds - whole;
    const double begun = job.blocks256 / compute_units, begun_whole = __builtin_floor(begun), begun_part = begun - begun_whole;
    const double last_block = begun_part == 0.0 ? 0.0 : k.last_block + (k.block - k.last_block) * at_least(2.0 * begun_part - 1.0, 0.0);
    const double skipped = (job.grid256 - job.blocks256) / compute_units;
    const double ids = __builtin_ceil(at_most(job.grid256, (double)compute_units) / 8.0);       // workgroups that start on a queue
    const bool uneven = job.shortest_queue < ids;
    const double skip = skipped > 0.0 ? k.skip * at_most(skipped, 1.0) : uneven ? k.uneven : 0.0;
    double last = 0.0;
    if (part > 0.0) {
        last = (whole > 0.0 ? k.late_tile : k.last_tile) + k.slope * at_least(part - 0.5, 0.0);
        if (whole > 0.0 && uneven) last = at_least(last, k.late_tile + k.uneven_slope * at_least(part - 0.25, 0.0));
        last = at_most(last, k.tile);
    }
    return k.start + skip + k.block * begun_whole + last_block + job.tiles(ns) * (k.tile * whole + last);
}
inline double plain_attn_us(const AttnJob& job, int32_t ns, int head_dim, int compute_units) {
    const AttnCosts k = attn_costs(head_dim);
    const double tiles = job.tiles(ns), slots = (double)k.per_cu * compute_units;
    if (job.grid128 <= compute_units && ns >= 128)
        return k.teams_start + tiles * (k.teams_tile + k.teams_slope * job.blocks128 / compute_units);
    const double whole = __builtin_floor(job.work128 / slots), on_cu = job.work128 / compute_units - k.per_cu * whole;
    double last = on_cu <= 0.0 ? 0.0 : k.lone;
    if (on_cu > 1.0) last = at_most(k.pair + k.pair_slope * (on_cu - 1.0), k.plain_tile);
    if (on_cu > 2.0) last = at_most(k.triple + k.pair_slope * (on_cu - 2.0), k.plain_tile);
    const double us = k.plain_start + k.plain_block * __builtin_ceil(job.blocks128 / slots) + tiles * (k.plain_tile * whole + last);
    return job.grid128 > slots ? us * (1.0 + k.list * job.padding) : us;
}
inline bool plain_attn_is_faster(const AttnJob& job, int32_t ns, int head_dim, int compute_units) {
    return plain_attn_us(job, ns, head_dim, compute_units) < scheduled_attn_us(job, ns, head_dim, compute_units);
}

// The job of `batch` elements (lens: their rows, nullptr: n in each)
inline AttnJob attn_job(int64_t batch, int64_t heads, int32_t n, const int32_t* lens) {
    AttnJob job{};
    const int64_t all = batch * heads, whole_heads = all & ~(int64_t)7;
    int32_t longest = lens ? 1 : n;
    for (int64_t b = 0; lens && b < batch; ++b) longest = lens[b] > longest ? lens[b] : longest;
    double on_xcd[8] = {}, work_on_xcd[8] = {}, rest = 0.0, work_rest = 0.0, work = 0.0;
    for (int64_t b = 0; b < (lens ? batch : 1); ++b) {
        const int32_t rows = lens ? lens[b] : n;
        const double part = (double)rows / longest, blocks = (double)((rows + 127) / 128);
        const int64_t first = b * heads, end = lens ? first + heads : all;
        job.blocks256 += (double)((rows + 255) / 256) * (end - first);
        job.work256 += part * ((rows + 255) / 256) * (end - first);
        work += part * blocks * (end - first);
        // heads y, y + 8, ... of the whole eights lie on XCD y, the blocks of the others on all
        const int64_t stop = end < whole_heads ? end : whole_heads;
        for (int y = 0; y < 8; ++y) {
            const int64_t count = stop > first ? (stop - y + 7) / 8 - (first - y + 7) / 8 : 0;
            on_xcd[y] += blocks * count;
            work_on_xcd[y] += part * blocks * count;
        }
        const int64_t left = end - (first > whole_heads ? first : whole_heads);
        if (left > 0) { rest += blocks * left; work_rest += part * blocks * left; }
    }
    for (int y = 0; y < 8; ++y) {
        if (work_on_xcd[y] >= job.work128) { job.work128 = work_on_xcd[y]; job.blocks128 = on_xcd[y]; }
    }
    job.work128 = 8.0 * job.work128 + work_rest;
    job.blocks128 = 8.0 * job.blocks128 + rest;
    const double per_head = (double)((n + 255) / 256);
    job.grid256 = per_head * all;
    job.shortest_queue = per_head * (all / 8);
    job.grid128 = (double)((n + 127) / 128) * all;
    job.padding = 1.0 - work / job.grid128;
    job.rows = n;
    job.longest = longest;
    return job;
}

}  // namespace pulsecol
