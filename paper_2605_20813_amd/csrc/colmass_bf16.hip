// The two scoring passes of the identification step, bf16 inputs (Sec. 3.3, score equation):
//   row pass     lse_i = log sum_j exp(z_ij),  z_ij = q_i . k_j * scale
//   column pass  s_{u,j} = (1/|G_u|) sum_{i in G_u} exp(z_ij - lse_i)
// for the query groups G_u of a head (consecutive runs of group_size rows; one group = the whole
// head on the hot path).  The row pass hands its result over in log2 units, so that
// p_ij = exp2(z_ij * scale * log2(e) - lse2_i).
//
// One structure for both.  A workgroup owns 256 stationary rows (4 waves x 64; query rows in the row
// pass, key rows in the column pass), each wave's in registers as the MFMA B operand, and streams
// 64-row tiles of the other tensor through LDS as the A operand: direct-to-LDS loads into one of three
// tile slots, issued two tiles ahead of their use.  In S[streamed][stationary] a lane owns one
// stationary row and its 16 registers are 16 streamed rows, so the sum over the streamed rows is an
// in-lane sum (a short accumulator, in the column pass four interleaved ones, that is added to a long one now and
// then) and the two half-waves meet at the end of a segment (column pass with several query groups: of a group).
//   column pass: exp2(z*c - lse_i) takes lse_i per register row, read from LDS four at a time.
//   row pass: exp2(z*c - ref) against one reference per lane, a whole number, at first 3 log2 units above
//     the maximum of the first 32 keys (ordinary rows rise 5 to 10 units above it, and a raise costs the
//     wave a block's weights anew).  z*c - ref is rounded at its own size, so a reference far below the
//     weights that dominate a row costs their precision: where the weights of a block of 32 keys outgrow
//     2^8 in some lane, the reference goes up with the block's maximum, the sums so far are scaled by that
//     exact power of two and the block's weights formed anew from its scores, which are still there.
// P never leaves fp32 and there are no floating-point atomics: the result is bit-identical
// from run to run.
//
// The streamed range of a head is made of segments (score_runs.h), each with a sum and (row pass) a reference of its
// own, which are added up in order.  Where one workgroup per head and block would leave the chip idle the segments are
// shared out among several (`splits` runs, score_splits): each leaves the results of its segments, and a small
// kernel adds them up, in the same order: a head's scores do not depend on the grid, the other heads or the other
// elements of a batch.  (Column pass with more than one query group: the sums are those of the groups, runs end at
// group boundaries, and nothing is left to add.)
//
// Short contexts and small grids run in blocks of 128 rows (a wave holds 32), uncut, where a second team of four waves may take the second half of
// the segments of the same rows: no launch adds anything up (score_teams says where; 32 heads of 1000 rows, both
// passes, 30.5 -> 25.1 us, of 256 15.7 -> 11.6).
//
// What bounds it: two weights and a matrix instruction per 32 cycles of the matrix pipe, about as much as one wave
// can issue, and over long runs the power limit (both passes, 32 heads of 8192 rows: 1.12 PFLOP/s on random operands, 1.55 on
// all-zero ones).  The row pass used to be a mode of the 256-row attention kernel, 62 KB of straight-line code that every
// launch fetches anew; this one is 23 KB, 6 of them the raises, out of the way.  D = 128, 32 heads of 4096 rows: row
// pass 172 us in that form, 126 with a reference that stays and runs of free length, 133 now (the check of every block
// 2.5, the ends of segments the rest); column pass 132.  Both passes, 16384 rows: 3.72 ms (1% of it), 65536 rows 58.4 ms (nothing).
#include <utility>

#include "pulsecol_device.h"
#include "pulsecol_kernels.h"
#include "score_sums.h"

namespace pulsecol {
namespace {

typedef unsigned char byte;

constexpr int NTHREADS = 256;
constexpr int QT = kScoreTile_bf16;         // rows per streamed tile
constexpr int FLUSH = 16;           // most tiles between flushes of the short accumulator into the long one

// s_waitcnt vmcnt(v) with the other counters left alone (gfx9 encoding: vmcnt in [3:0] and [15:14])
template <int v>
__device__ __forceinline__ void wait_vmcnt_at_most() {
    static_assert(v >= 0 && v < 64, "six bits");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (v & 0xF) | ((v & 0x30) << 10));
}
// nothing that touches memory moves across this point, neither in the compiler nor in its scheduler
__device__ __forceinline__ void memory_order_point() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// One streamed tile and (column pass) its 64 log-sum-exp values, this wave's share: CH loads of 64 x 16
// bytes into the 1 KB chunks wave*CH + i of the slot (lane L lands at chunk byte 16*L = tile row
// chunk*RPC + L/PIECES, LDS piece L%PIECES, and fetches the global piece (L%PIECES) ^ swizzle(row) of
// its row: xoff[i] is that piece's byte offset from the row's start), and one load of 64 x 4 bytes for
// the tile's log-sum-exp values.  Rows past the end of the head read the last row instead; the caller
// gives them weight zero.
// (The slot pointer is a restrict parameter so that the loads carry an alias scope: the compiler
// then does not make LDS reads of the other slots wait for these loads.  A slot is ONE object,
// the tile followed by its log-sum-exp values: the compiler tells only a handful of such load
// targets apart, and beyond that number every LDS read waits for every load.)
template <int CH, bool ROWS>
__device__ __forceinline__ void issue_tile(byte* __restrict__ slot, byte* __restrict__ lse_slot,
                                           const byte* __restrict__ X, const float* __restrict__ lse,
                                           int t, int n, uint32_t row_bytes, const int (&trow)[CH],
                                           const uint32_t (&xoff)[CH], int wave, int lane) {
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int row = t * QT + trow[i];
        // both factors are below 2^24 and the product below 2^32 (checked on the host)
        const uint32_t off = __umul24((uint32_t)(row < n ? row : n - 1), row_bytes) + xoff[i];
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(X + off),
                                         (PULSECOL_LDS void*)(slot + (wave * CH + i) * 1024), 16, 0, 0);
    }
    if constexpr (!ROWS) {
        // every wave brings all 64 values (the same bytes four times over): no branch in here, which
        // keeps the compiler's own bookkeeping of these loads exact
        const int row = t * QT + lane;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(lse + (uint32_t)(row < n ? row : n - 1)),
                                         (PULSECOL_LDS void*)lse_slot, 4, 0, 0);
    }
}

// LDS fragment reads as inline assembly with hand-placed waits.  (The compiler's own wait-count
// insertion drains lgkmcnt to zero in front of every LDS read while a direct-to-LDS load is in
// flight; LDS returns data in order, so "all but the N newest reads" is exact.)  For these loads the
// compiler knows neither the latency nor that the destination is written later: nothing may read
// the variable before the wait that covers it.  tests/test_asm_hazards.py checks the generated code.
template <int OFF>
__device__ __forceinline__ bf16x8 lds_read_b128_at(uint32_t addr) {
    bf16x8 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(v) : "v"(addr), "n"(OFF));
    return v;
}
template <int OFF>
__device__ __forceinline__ f32x4 lds_read_f32x4_at(uint32_t addr) {
    f32x4 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(v) : "v"(addr), "n"(OFF));
    return v;
}
__device__ __forceinline__ void fence() { __builtin_amdgcn_sched_barrier(0); }
__device__ __forceinline__ uint32_t lds_address(const void* generic_lds_ptr) {
    return (uint32_t)(uintptr_t)(PULSECOL_LDS const void*)generic_lds_ptr;
}

// A tile is two blocks of 32 streamed rows; a block's scores take 2 * KK matrix instructions (KK
// fragments of the block's rows, each against the wave's two blocks of 32 stationary rows) and 32 softmax
// weights per lane (fma, exp2, add each).  The two kinds of work are interleaved instruction by
// instruction: while the matrix instructions of a block issue, the weights of the block before it are
// formed, a few per matrix instruction, so that every wave's instruction stream feeds the matrix pipe
// and the vector pipe evenly.  (Written as two phases per block -- all matrix instructions, then all
// weights -- the two waves that share a SIMD fall into step: both in the matrix phase, then both in
// the vector phase, each pipe idle half of the time.)
template <int D, bool ROWS, int KB>
struct ScoreWave {
    static constexpr int PIECES = D / 8;
    static constexpr int KK = D / 16;
    static constexpr int ROW_BYTES = D * 2;
    static constexpr int TILE_BYTES = QT * ROW_BYTES;
    static constexpr int NPAIR = 2 * KK;                      // fragment reads (= pairs of matrix instructions) per tile
    static constexpr int AHEAD = KK / 2;                      // fragment reads in flight ahead of their use
    static constexpr int PER_SLOT = 16 / KK;                  // weights formed behind each matrix instruction
    // row pass: behind all but the last one, which covers the closing of the block's sums: the first weight of slot s
    static constexpr int row_weight(int s) { return s >= KB * KK - 1 ? 16 * KB : 16 * KB * s / (KB * KK - 1); }
    static constexpr int LSE_RING = 4;                        // tiles whose log-sum-exp values LDS holds at a time
    static constexpr int LSE_BYTES = QT * 4;
    static constexpr int LSE_BASE = 3 * TILE_BYTES;           // the ring follows the three tile slots
    // Pairs between a log-sum-exp read and its first use.  LDS returns data in order, so the read has landed
    // once a fragment requested after it has: the fragment of the pair that uses it is requested AHEAD pairs
    // before that pair, hence AHEAD + 1.
    static constexpr int LEAD = AHEAD + 1;
    static_assert(KK == 4 || KK == 8, "head dimension 64 or 128");
    // The weights of a block are formed in register order, two key blocks per register: pair x of the KK pairs
    // of a block handles registers x * PER_SLOT .. +PER_SLOT-1, so the log-sum-exp group g (registers 4g .. 4g+3,
    // four consecutive query rows) is first needed in pair first_use(g), and is read LEAD pairs before that --
    // which for the first groups falls into the block before, while that block's own scores are still being
    // computed.
    static constexpr int first_use(int g) { return g * KK / 4; }
    // group read in the second slot of in-block pair x: for the block being consumed (>= 0), or -1
    static constexpr int lse_group_consumed(int x) {
        for (int g = 0; g < 4; ++g) if (first_use(g) - LEAD == x) return g;
        return -1;
    }
    // ... for the block being computed, which is consumed next (>= 0), or -1
    static constexpr int lse_group_computed(int x) {
        for (int g = 0; g < 4; ++g) if (first_use(g) - LEAD + KK == x) return g;
        return -1;
    }
    // log-sum-exp reads in pair q of a tile (FIRST: the head's first tile, whose first block has no block before
    // it to consume)
    template <bool FIRST>
    static constexpr int lse_reads(int q) {
        if (ROWS) return 0;
        const int x = q % KK;
        return ((lse_group_consumed(x) >= 0 && !(FIRST && q < KK)) ? 1 : 0) + (lse_group_computed(x) >= 0 ? 1 : 0);
    }
    // LDS reads issued behind fragment p before pair p waits for it: the fragments requested ahead, and the
    // log-sum-exp reads of the pairs since fragment p was requested
    template <bool FIRST>
    static constexpr int newer(int p) {
        int c = (p + AHEAD - 1 < NPAIR - 1 ? p + AHEAD - 1 : NPAIR - 1) - p;
        for (int q = (p - AHEAD > 0 ? p - AHEAD : 0); q < p; ++q) c += lse_reads<FIRST>(q);
        return c;
    }
    static_assert(lse_group_consumed(0) < 0 || lse_group_computed(0) < 0, "one log-sum-exp read per pair at most");

    bf16x8 yf[KB][KK];        // stationary fragments: B operand, [row lq of block kb][d = kk*16 + 8*lh .. +7]
    f32x16 sb[2][KB];         // scores [streamed block qb][stationary block kb]
    f32x4 lr[4];              // column pass: log-sum-exp (log2 units) of four query rows each, of the block whose weights are being formed
    float ref[KB];            // row pass: the reference (log2 units, whole) of this lane's query rows
    float blk[KB][4], sum[KB];       // row pass: the sums of the block whose weights are being formed
    uint64_t grown;           // row pass: lanes whose sums have outgrown the reference
    static constexpr int NACC = ROWS ? 1 : 4;       // (row pass: whole blocks are added up)
    float acc_short[KB][NACC], acc_long[KB];
    uint32_t xv[KK];          // LDS address of this lane's fragment kk in slot 0, first block
    uint32_t lv;              // column pass: LDS address of this lane's first log-sum-exp group in ring entry 0
    float c2;

    // weight e (0 .. 16 * KB - 1) of streamed block cq: register e / KB, stationary block e % KB
    __device__ __forceinline__ void weight(int cq, int e) {
        const int r = e / KB, kb = e % KB;
        add_weight(kb, r, fast_exp2(__builtin_fmaf(sb[cq][kb][r], c2, ROWS ? -ref[kb] : -lr[r >> 2][r & 3])));
    }
    __device__ __forceinline__ void add_weight(int kb, int r, float e) {
        if constexpr (ROWS) {
            blk[kb][r & 3] = r < 4 ? e : blk[kb][r & 3] + e;
        } else {
            acc_short[kb][r & 3] += e;
        }
    }
    // row pass: a block's sums, and the lanes where they outgrow the reference (or are NaN)
    __device__ __forceinline__ void sum_block() {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) sum[kb] = (blk[kb][0] + blk[kb][1]) + (blk[kb][2] + blk[kb][3]);
        grown = __ballot(!(sum[0] <= kGrowthLimit) | !(sum[KB - 1] <= kGrowthLimit));
    }
    // row pass: a reference from 32 keys, the next whole number above their maximum and kHeadroom more (both half-waves get
    // the same one)
    __device__ __forceinline__ float reference_of(const f32x16& s) const {
        float mx = s[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
        // (the bound: a block of keys without a finite logit leaves the reference finite and adds nothing)
        return fmaxf(ceilf(half_max(mx) * c2) + kHeadroom, kNoReference);
    }
    __device__ __forceinline__ void set_reference(const f32x16 (&s)[KB]) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) ref[kb] = reference_of(s[kb]);
    }
    // row pass: accept the sums of a block (sum_block), or raise the reference first.  The scores `s` are the block's.
    __device__ __forceinline__ void close_block(const f32x16 (&s)[KB]) {
        if (__builtin_expect(grown != 0ull, 0)) {
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                const float top = reference_of(s[kb]);
                // (by the row's own sums, of either half-wave: not by those of the rows that share the wave, which are others in blocks of 128)
                if (half_max(sum[kb]) > kGrowthLimit && top > ref[kb]) {
                    // (a row without a finite logit so far has nothing to scale)
                    const float down = ref[kb] == kNoReference ? 0.f : fast_exp2(ref[kb] - top);
                    acc_short[kb][0] *= down;
                    acc_long[kb] *= down;
                    ref[kb] = top;
#pragma unroll
                    for (int r = 0; r < 16; ++r) add_weight(kb, r, fast_exp2(__builtin_fmaf(s[kb][r], c2, -top)));
                    sum[kb] = (blk[kb][0] + blk[kb][1]) + (blk[kb][2] + blk[kb][3]);
                }
            }
        }
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) acc_short[kb][0] += sum[kb];
    }
    template <int OFF>
    __device__ __forceinline__ void read_lse(int g, uint32_t ring_addr) {
        // (one statement per group so that the destination is a whole variable)
        if (g == 0) lr[0] = lds_read_f32x4_at<LSE_BASE + OFF>(ring_addr);
        if (g == 1) lr[1] = lds_read_f32x4_at<LSE_BASE + OFF + 32>(ring_addr);
        if (g == 2) lr[2] = lds_read_f32x4_at<LSE_BASE + OFF + 64>(ring_addr);
        if (g == 3) lr[3] = lds_read_f32x4_at<LSE_BASE + OFF + 96>(ring_addr);
    }

    // the weights behind matrix instruction SLOT of a block
    template <int SLOT>
    __device__ __forceinline__ void slot_weights(int cq) {
        if constexpr (ROWS) {
#pragma unroll
            for (int e = row_weight(SLOT); e < row_weight(SLOT + 1); ++e) weight(cq, e);
            if constexpr (SLOT == KB * KK - 1) sum_block();
        } else {
#pragma unroll
            for (int i = 0; i < PER_SLOT; ++i) weight(cq, SLOT * PER_SLOT + i);
        }
    }

    // Pair P of the tile in slot S: KB matrix instructions on fragment P, the request for fragment P + AHEAD,
    // at most one log-sum-exp read, and (CONSUME) KB * PER_SLOT weights of the block before.  ring_cur / ring_prev:
    // LDS addresses (lane's first group) of the log-sum-exp values of this tile and of the tile before.
    template <int S, int P, bool FIRST>
    __device__ __forceinline__ void pair(bf16x8 (&fr)[NPAIR], uint32_t ring_cur, uint32_t ring_prev) {
        constexpr int qb = P / KK, x = P % KK, cq = 1 - qb;
        constexpr bool CONSUME = !(FIRST && qb == 0);
        constexpr int SLOT = S * TILE_BYTES;
        auto product = [&](int kb) {
            if constexpr (x == 0) {
                f32x16 zero;
#pragma unroll
                for (int r = 0; r < 16; ++r) zero[r] = 0.f;
                sb[qb][kb] = mfma_bf16(fr[P], yf[kb][x], zero);
            } else {
                sb[qb][kb] = mfma_bf16(fr[P], yf[kb][x], sb[qb][kb]);
            }
            fence();
        };
        asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(fr[P]) : "n"(newer<FIRST>(P)));
        product(0);
        if constexpr (P + AHEAD < NPAIR) {
            constexpr int Q = P + AHEAD;
            fr[Q] = lds_read_b128_at<SLOT + (Q / KK) * 32 * ROW_BYTES>(xv[Q % KK]);
        }
        if constexpr (CONSUME) slot_weights<KB * x>(cq);
        fence();
        if constexpr (KB == 2) product(1);
        // the block being consumed: second block of the tile before (qb == 0) or first block of this tile
        if constexpr (!ROWS && CONSUME && lse_group_consumed(x) >= 0) {
            if constexpr (qb == 0) read_lse<32 * 4>(lse_group_consumed(x), ring_prev);
            else read_lse<0>(lse_group_consumed(x), ring_cur);
        }
        // the block being computed, whose weights the next block's pairs will form
        if constexpr (!ROWS && lse_group_computed(x) >= 0) read_lse<qb * 32 * 4>(lse_group_computed(x), ring_cur);
        if constexpr (KB == 2 && CONSUME) slot_weights<2 * x + 1>(cq);
        fence();
    }
    template <int S, int P0, bool FIRST, int... Ps>
    __device__ __forceinline__ void pairs(bf16x8 (&fr)[NPAIR], uint32_t ring_cur, uint32_t ring_prev, std::integer_sequence<int, Ps...>) {
        (pair<S, P0 + Ps, FIRST>(fr, ring_cur, ring_prev), ...);
    }
    // the first AHEAD fragments of a tile (behind the barrier that says the tile has landed)
    template <int S>
    __device__ __forceinline__ void request_first(bf16x8 (&fr)[NPAIR]) {
        static_assert(AHEAD == 2 || AHEAD == 4, "written out for two and four");
        fr[0] = lds_read_b128_at<S * TILE_BYTES>(xv[0]);
        fr[1] = lds_read_b128_at<S * TILE_BYTES>(xv[1]);
        if constexpr (AHEAD == 4) {
            fr[2] = lds_read_b128_at<S * TILE_BYTES>(xv[2]);
            fr[3] = lds_read_b128_at<S * TILE_BYTES>(xv[3]);
        }
    }
    // The weights of a block outside the interleave (the last full block of a head): the groups that the
    // interleave would have read in the following block are read here.
    __device__ __forceinline__ void weights_alone(int cq, uint32_t ring_addr) {
        if constexpr (!ROWS) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                if (first_use(g) - LEAD >= 0) {
                    if (g == 1) lr[1] = lds_read_f32x4_at<LSE_BASE + 32 * 4 + 32>(ring_addr);
                    if (g == 2) lr[2] = lds_read_f32x4_at<LSE_BASE + 32 * 4 + 64>(ring_addr);
                    if (g == 3) lr[3] = lds_read_f32x4_at<LSE_BASE + 32 * 4 + 96>(ring_addr);
                }
            }
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(lr[0]), "+v"(lr[1]), "+v"(lr[2]), "+v"(lr[3]));
        }
#pragma unroll
        for (int e = 0; e < 16 * KB; ++e) weight(cq, e);
        if constexpr (ROWS) sum_block();
    }
};

// GROUPED: column pass with several query groups.  CUT: the head's segments (groups) are shared out among several runs.
// KB: blocks of 32 stationary rows per wave.  TEAMS: two teams of four waves share out the segments (groups) of the same stationary
// rows; the second leaves its segments' results in LDS and the first adds them up behind its own.
template <int D, bool ROWS, bool GROUPED, bool CUT, int KB, int TEAMS>
__device__ __forceinline__ void score_pass(const ScoreParams& p) {
    using W = ScoreWave<D, ROWS, KB>;
    constexpr int ROWS_PER_WG = 128 * KB;
    constexpr int TEAM_BYTES = 3 * W::TILE_BYTES + (ROWS ? 0 : W::LSE_RING * W::LSE_BYTES);
    constexpr bool KEEP = TEAMS > 1 && !GROUPED;      // results of the second team's segments: sums, then references
    static_assert(TEAMS == 1 || !CUT, "teams are runs inside the workgroup");
    constexpr int PIECES = W::PIECES;
    constexpr int KK = W::KK;
    constexpr int ROW_BYTES = W::ROW_BYTES;
    constexpr int TILE_BYTES = W::TILE_BYTES;
    constexpr int NPAIR = W::NPAIR;
    constexpr int RPC = 64 / PIECES;                  // tile rows per 1 KB chunk
    constexpr int CH = TILE_BYTES / 1024 / 4;         // chunks per wave and tile
    constexpr int VM_PER_TILE = CH + (ROWS ? 0 : 1);  // vector memory operations a wave issues per tile
    static_assert(CH >= 1 && CH * 4 * 1024 == TILE_BYTES, "the waves' chunks cover the tile exactly");

    // ONE array: three tile slots, then a ring of four tiles' log-sum-exp values (64 each).  Slot and block
    // are instruction offsets of the fragment reads.  The ring is one entry longer than the slots because the
    // weights of a tile's second block are formed during the first block of the next tile, after the barrier
    // that frees the tile's slot.
    // (With two teams, one after the other.)
    __shared__ __attribute__((aligned(1024))) byte lds_teams[TEAMS * TEAM_BYTES];
    __shared__ float kept[KEEP ? kMaxScoreSegments : 1][KEEP ? (ROWS ? 2 : 1) : 1][KEEP ? ROWS_PER_WG : 1];

    // every kernel argument with the first batch of scalar loads: left to itself the compiler loads them where they
    // are first used, one memory round trip after another
    asm volatile("" : : "s"(p.q), "s"(p.k), "s"(p.lse), "s"(p.scores), "s"(p.td.sb), "s"(p.td.sh), "s"(p.td.sn),
                         "s"(p.td_kv.sb), "s"(p.td_kv.sh), "s"(p.td_kv.sn), "s"(p.kv_heads), "s"(p.batch), "s"(p.heads),
                         "s"(p.n), "s"(p.groups), "s"(p.group_size), "s"(p.scale), "s"(p.varlen), "s"(p.part),
                         "s"(ROWS ? p.row_splits : p.col_splits));
    // (run `split` of the head's streamed range: the z planes; only few layers of heads are ever cut into runs)
    const int splits = ROWS ? p.row_splits : p.col_splits;
    const int split = CUT ? blockIdx.z : 0;
    int bh, blk, b, h;
    if (!head_and_block(CUT ? blockIdx.y : blockIdx.z * kLayersPerZ + blockIdx.y, p.batch * p.heads,
                        (p.n + ROWS_PER_WG - 1) / ROWS_PER_WG, &bh, &blk)) return;
    split_head(bh, p.batch, p.heads, &b, &h);
    // variable-length batches: queries and keys of this batch element end at its own length
    const int n = p.varlen != nullptr ? p.varlen[b] : p.n;
    if (blk * ROWS_PER_WG >= n) return;     // a block of padding rows: what belongs to it is left untouched
    const int64_t q_off = (int64_t)b * p.td.sb + (int64_t)h * p.td.sh;
    // grouped-query layout: query head h reads K/V head h / (heads / kv_heads)
    const int64_t k_off = (int64_t)b * p.td_kv.sb + (int64_t)kv_head_of(h, p.heads, p.kv_heads) * p.td_kv.sh;
    const byte* __restrict__ X = (const byte*)(ROWS ? (const __bf16*)p.k + k_off : (const __bf16*)p.q + q_off);      // streamed
    const __bf16* __restrict__ Y = ROWS ? (const __bf16*)p.q + q_off : (const __bf16*)p.k + k_off;                   // stationary
    const int64_t y_stride = ROWS ? p.td.sn : p.td_kv.sn;
    const uint32_t row_bytes = (uint32_t)(ROWS ? p.td_kv.sn : p.td.sn) * 2u;
    const float* __restrict__ lse = p.lse + (int64_t)bh * p.n;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave_wg = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int team = TEAMS > 1 ? wave_wg >> 2 : 0, wave = wave_wg & 3;
    byte* const lds_all = lds_teams + team * TEAM_BYTES;
    const int lq = lane & 31, lh = lane >> 5;
    const int y0 = blk * ROWS_PER_WG + wave * (32 * KB);

    // the streamed rows of this run: segments seg .. , tiles t0 .. t1-1, rows up to x_end
    const ScoreSegments segments(n);
    int seg = 0, t0 = 0, t1 = segments.tiles;
    int steps = 0;              // two teams: tiles of the one that has more
    if constexpr (CUT || TEAMS > 1) {
        if constexpr (GROUPED) {
            const TileRun run = group_run(segments.tiles, TEAMS > 1 ? team : split, TEAMS > 1 ? TEAMS : splits, p.group_size);
            t0 = run.first;
            t1 = run.last;
        } else if constexpr (TEAMS > 1) {
            const int half = segments.count >> 1;             // (segments of the first team)
            seg = team == 0 ? 0 : half;
            t0 = segments.first_tile(seg);
            t1 = segments.first_tile(team == 0 ? half : segments.count);
        } else {
            const uint32_t reciprocal = ROWS ? p.row_reciprocal : p.col_reciprocal;
            seg = segments.first_of_run(split, reciprocal);
            t0 = segments.first_tile(seg);
            t1 = segments.first_tile(segments.first_of_run(split + 1, reciprocal));
        }
    }
    if constexpr (TEAMS > 1) {
        const int others = segments.tiles - (t1 - t0);        // (both teams' tiles make up the head)
        steps = others > t1 - t0 ? others : t1 - t0;
    } else {
        if (t0 >= t1) return;   // more runs than an element of a padded batch has segments
    }
    const int x_end = t1 * QT < n ? t1 * QT : n;
    const int64_t all_rows = (int64_t)p.batch * p.heads * p.n;
    const int64_t sums_at = p.segment_room * all_rows;          // row pass: the sums follow the references
    const int kept_first = seg;
    int seg_first = t0, seg_end = GROUPED ? t1 : segments.first_tile(seg + 1);      // the running segment's tiles
    // the next tile in front of which something is to be done but forming weights: the end of the running segment, or a
    // flush of the short accumulators every FLUSH tiles of it (groups: of the head)
    int stop = t0 + FLUSH - (GROUPED ? t0 % FLUSH : 0);
    stop = stop < seg_end ? stop : seg_end;

    W w;
    // ---- stationary fragments
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        int row = y0 + kb * 32 + lq;
        row = row < n ? row : n - 1;
        const __bf16* src = Y + (int64_t)row * y_stride + 8 * lh;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) w.yf[kb][kk] = *(const bf16x8*)(src + kk * 16);
    }

    // ---- load geometry of this lane: chunk i of its wave covers tile row trow[i]
    int trow[CH];
    uint32_t xoff[CH];
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        trow[i] = (wave * CH + i) * RPC + lane / PIECES;
        xoff[i] = (uint32_t)((lane % PIECES) ^ swizzle_k<PIECES>(trow[i])) * 16u;
    }
    // ---- fragment addresses: fragment kk of streamed block qb = tile row qb*32 + lq, piece 2*kk + lh
    // (rows 32 apart share a swizzle: the block is an instruction offset); log-sum-exp group g of block qb =
    // rows qb*32 + 8*g + 4*lh .. +3
    const uint32_t lds0 = lds_address(lds_all);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) w.xv[kk] = lds0 + (uint32_t)(lq * ROW_BYTES + (((2 * kk + lh) ^ swizzle_k<PIECES>(lq)) << 4));
    w.lv = lds0 + (uint32_t)(16 * lh);
    static_assert(PIECES <= 32, "rows 32 apart share a swizzle");

    // whole tiles: the interleaved steps; a ragged last tile is computed apart (a team without tiles may stand behind it)
    const int nfull = t0 < t1 ? x_end / QT - t0 : 0;
    w.c2 = p.scale * kLog2e;
    w.ref[0] = w.ref[KB - 1] = 0.f;
    // per stationary block kb, this lane's row; (column pass) four interleaved partial sums keep the add chains independent
    auto start_sums = [&] {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            w.acc_long[kb] = 0.f;
#pragma unroll
            for (int c = 0; c < W::NACC; ++c) w.acc_short[kb][c] = 0.f;
        }
    };
    start_sums();
    auto flush = [&] {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            if constexpr (ROWS) w.acc_long[kb] += w.acc_short[kb][0];
            else w.acc_long[kb] += (w.acc_short[kb][0] + w.acc_short[kb][1]) + (w.acc_short[kb][2] + w.acc_short[kb][3]);
#pragma unroll
            for (int c = 0; c < W::NACC; ++c) w.acc_short[kb][c] = 0.f;
        }
    };
    // this lane's sum of stationary block kb over both half-waves (they hold the same stationary rows, other streamed
    // rows), behind a flush
    auto total = [&](int kb) { return half_sum(w.acc_long[kb]); };

    // column pass with several query groups: rows until the running one ends (a run starts at a group's first row)
    int rows_to_group_end = p.group_size;

    SegmentSum all[KB];                     // of the segments that have ended
    all[0].ref = all[KB - 1].ref = kNoReference;
    // The end of segment `seg`: its sum (row pass: and reference) into registers, or to memory, to be added up when all runs
    // have ended; accumulators start over.
    auto end_segment = [&] {
        flush();
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const float v = total(kb);
            const int row = y0 + kb * 32 + lq;
            if constexpr (CUT) {
                if (lh == 0 && row < n) {
                    float* const at = p.part + (seg * all_rows + (int64_t)bh * p.n + row);
                    if (ROWS) { at[0] = w.ref[kb]; at[sums_at] = v; }
                    else at[0] = v;
                }
            } else if (KEEP && team == 1) {
                if (lh == 0) {
                    kept[seg - kept_first][0][wave * (32 * KB) + kb * 32 + lq] = v;
                    if constexpr (ROWS) kept[seg - kept_first][KEEP ? 1 : 0][wave * (32 * KB) + kb * 32 + lq] = w.ref[kb];
                }
            } else if constexpr (ROWS) {
                all[kb].add(w.ref[kb], v);
            } else {
                all[kb].add(v);
            }
            w.acc_long[kb] = 0.f;
        }
        ++seg;
    };

    // What follows the weights of block qb of the run's tile t: the periodic flush of the short accumulators,
    // the end of a segment inside the run, and in the column pass with several query groups at
    // the last rows of one (groups are multiples of 32 rows), the group's score row: add the two half-waves,
    // divide by the group's size, store, start over.
    auto block_done = [&](int t, int qb) {
        if (qb == 1 && __builtin_expect(t0 + t + 1 == stop, 0)) {
            if (stop < seg_end) {
                flush();
            } else if (seg_end < t1) {
                end_segment();
                seg_first = seg_end;
                seg_end = segments.first_tile(seg + 1);
            }
            stop = stop + FLUSH < seg_end ? stop + FLUSH : seg_end;
        }
        if constexpr (GROUPED) {
            const int rows_done = (t0 + t) * QT + (qb + 1) * 32;
            rows_to_group_end -= 32;
            const bool group_end = (rows_done >= x_end) || (rows_to_group_end == 0 && rows_done < x_end);
            if (rows_to_group_end == 0) rows_to_group_end = p.group_size;
            if (group_end) {
                const int rows_seen = rows_done < x_end ? rows_done : x_end;
                const int u = (rows_seen - 1) / p.group_size;
                const int g_rows = rows_seen - u * p.group_size;
                const float inv = 1.0f / (float)g_rows;
                float* __restrict__ out = p.scores + ((int64_t)bh * p.groups + u) * p.n;
                flush();
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) {
                    const float v = total(kb);
                    const int key = y0 + kb * 32 + lq;
                    if (lh == 0 && key < n) out[key] = v * inv;
                    w.acc_long[kb] = 0.f;
                }
            }
        }
    };
    auto ring_of = [&](int t) { return w.lv + (uint32_t)((t & (W::LSE_RING - 1)) * W::LSE_BYTES); };
    // (t counts the run's tiles: slot and ring entry follow it)
    auto issue = [&](int t) {
        issue_tile<CH, ROWS>(lds_all + (t % 3) * TILE_BYTES, lds_all + W::LSE_BASE + (t & (W::LSE_RING - 1)) * W::LSE_BYTES,
                             X, lse, t0 + t, n, row_bytes, trow, xoff, wave, lane);
    };

    // ---- tiles 0 and 1 go out
    issue(0);
    issue(1);

    // Step t (tile t in slot S = t % 3): tile t has landed in every wave once this wave's loads of tile t+1 are
    // the only ones it still may have in flight (vector memory completes in issue order, and whatever this
    // step issues comes later still) and all waves have said so at the barrier.  The barrier also tells that
    // every wave is done with the slot of tile t-1 and with the log-sum-exp values of tile t-2, which the
    // loads of tile t+2 now replace.  Loads are issued for tiles past the end as well (the head's last row,
    // slots never read), so the count in flight is the same at every step.
    auto step = [&](auto slot_c, auto first_c, int t) {
        constexpr int S = decltype(slot_c)::value;
        constexpr bool FIRST = decltype(first_c)::value;     // no block before this tile's first: nothing to consume
        wait_vmcnt_at_most<VM_PER_TILE>();
        memory_order_point();
        __builtin_amdgcn_s_barrier();
        memory_order_point();
        bf16x8 fr[NPAIR];
        w.template request_first<S>(fr);
        memory_order_point();
        issue(t + 2);
        memory_order_point();
        const uint32_t ring_cur = ring_of(t), ring_prev = ring_of(t - 1);
        // first block of the tile, with the weights of the second block of the tile before
        w.template pairs<S, 0, FIRST>(fr, ring_cur, ring_prev, std::make_integer_sequence<int, KK>{});
        if constexpr (ROWS && !FIRST) w.close_block(w.sb[1]);
        if (!FIRST) block_done(t - 1, 1);
        // (a segment that starts with this tile: its reference)
        if (ROWS && (FIRST || __builtin_expect(seg_first == t0 + t, 0))) w.set_reference(w.sb[0]);
        // second block, with the weights of the first
        w.template pairs<S, KK, FIRST>(fr, ring_cur, ring_prev, std::make_integer_sequence<int, KK>{});
        if constexpr (ROWS) w.close_block(w.sb[0]);
        block_done(t, 0);
    };
    if (nfull > 0) {
        step(std::integral_constant<int, 0>{}, std::true_type{}, 0);
        for (int t = 1; t < nfull; t += 3) {
            step(std::integral_constant<int, 1>{}, std::false_type{}, t);
            if (t + 1 >= nfull) break;
            step(std::integral_constant<int, 2>{}, std::false_type{}, t + 1);
            if (t + 2 >= nfull) break;
            step(std::integral_constant<int, 0>{}, std::false_type{}, t + 2);
        }
        // the weights of the last whole tile's second block, on their own
        w.weights_alone(1, ring_of(nfull - 1));
        if constexpr (ROWS) w.close_block(w.sb[1]);
        block_done(nfull - 1, 1);
    }
    wait_vmcnt_at_most<0>();
    if (nfull < t1 - t0) {
        // ---- a ragged last tile, in plain code: rows past the end of the head add nothing to any sum
        memory_order_point();
        __builtin_amdgcn_s_barrier();
        memory_order_point();
        const int t = nfull;
        const byte* xslot = lds_all + (t % 3) * TILE_BYTES;
        const float* lslot = (const float*)(lds_all + W::LSE_BASE + (t & (W::LSE_RING - 1)) * W::LSE_BYTES);
        const int valid = n - (t0 + t) * QT;
#pragma nounroll
        for (int qb = 0; qb < 2; ++qb) {
            if (qb * 32 >= valid) break;
            f32x16 s[KB];
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r) s[kb][r] = 0.f;
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                const bf16x8 xfrag = *(const bf16x8*)(xslot + qb * 32 * ROW_BYTES + (w.xv[kk] - lds0));
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) s[kb] = mfma_bf16(xfrag, w.yf[kb][kk], s[kb]);
            }
            f32x4 l2[4];
            if constexpr (ROWS) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (qb * 32 + acc_row(r, lh) >= valid) { s[0][r] = -INFINITY; s[KB - 1][r] = -INFINITY; }
                if (nfull == 0 && qb == 0) w.set_reference(s);
            } else {
#pragma unroll
                for (int g = 0; g < 4; ++g) l2[g] = *(const f32x4*)(lslot + qb * 32 + 8 * g + 4 * lh);
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) {
                    const float e = fast_exp2(__builtin_fmaf(s[kb][r], w.c2, ROWS ? -w.ref[kb] : -l2[r >> 2][r & 3]));
                    w.add_weight(kb, r, (ROWS || qb * 32 + acc_row(r, lh) < valid) ? e : 0.f);
                }
            }
            if constexpr (ROWS) { w.sum_block(); w.close_block(s); }
            block_done(t, qb);
        }
    }

    if constexpr (!GROUPED) {
        if (TEAMS == 1 || t0 < t1) end_segment();             // the run's last one
        if constexpr (TEAMS > 1) {
            for (int t = t1 - t0; t < steps; ++t) __builtin_amdgcn_s_barrier();      // (the other team has more tiles)
            __syncthreads();
            if (team == 1) return;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                for (int s = 0; s < segments.count - (segments.count >> 1); ++s) {
                    const int at = wave * (32 * KB) + kb * 32 + lq;
                    if constexpr (ROWS) all[kb].add(kept[s][KEEP ? 1 : 0][at], kept[s][0][at]);
                    else all[kb].add(kept[s][0][at]);
                }
            }
        }
        if constexpr (!CUT) {
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                const int row = y0 + kb * 32 + lq;
                if (lh == 0 && row < n) {
                    if (ROWS) p.lse[(int64_t)bh * p.n + row] = log2_of(all[kb].ref, all[kb].total());
                    else p.scores[(int64_t)bh * p.n + row] = all[kb].total() * (1.0f / (float)n);
                }
            }
        }
    } else if constexpr (TEAMS > 1) {
        for (int t = t1 - t0; t < steps; ++t) __builtin_amdgcn_s_barrier();
    }
}

template <int D>
__global__ void __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(2)))
rowlse_bf16_kernel(ScoreParams p) { score_pass<D, true, false, false, 2, 1>(p); }

template <int D>
__global__ void __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(2)))
rowlse_runs_bf16_kernel(ScoreParams p) { score_pass<D, true, false, true, 2, 1>(p); }

template <int D>
__global__ void __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(2)))
colmass_bf16_kernel(ScoreParams p) { score_pass<D, false, false, false, 2, 1>(p); }

template <int D>
__global__ void __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(2)))
colmass_runs_bf16_kernel(ScoreParams p) { score_pass<D, false, false, true, 2, 1>(p); }

template <int D>
__global__ void __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(2)))
colmass_groups_bf16_kernel(ScoreParams p) { score_pass<D, false, true, false, 2, 1>(p); }

template <int D>
__global__ void __launch_bounds__(NTHREADS) __attribute__((amdgpu_waves_per_eu(2)))
colmass_groups_runs_bf16_kernel(ScoreParams p) { score_pass<D, false, true, true, 2, 1>(p); }

// Blocks of 128 rows, with one or two teams (score_teams)
template <int D, bool ROWS, bool GROUPED, int TEAMS>
__global__ void __launch_bounds__(NTHREADS * TEAMS) __attribute__((amdgpu_waves_per_eu(2)))
score_half_bf16_kernel(ScoreParams p) { score_pass<D, ROWS, GROUPED, false, 1, TEAMS>(p); }

// ---- the segments of heads that were cut into runs, added up in order.  One thread per row (row pass) or key (column
// pass), y = the head; latency-bound: all loads go out at once, and the sums are scaled to the last reference in one
// step (by exact powers of two: the same bits).
// MOST: segments that a head may have
template <bool ROWS, int MOST>
__global__ void __launch_bounds__(NTHREADS) score_combine_kernel(ScoreParams p) {
    const int bh = blockIdx.y, row = blockIdx.x * NTHREADS + threadIdx.x;
    int n = p.n;
    if (p.varlen != nullptr) n = p.varlen[bh / p.heads];
    if (row >= n) return;                    // (padding: left untouched)
    const int segments = ScoreSegments(n, p.f32).count;
    const int64_t count = (int64_t)p.batch * p.heads * p.n, at = (int64_t)bh * p.n + row;
    const float* __restrict__ first = p.part + at;
    const float* __restrict__ second = first + p.segment_room * count;
    float a[MOST], b[MOST];
#pragma unroll
    for (int s = 0; s < MOST; ++s) {
        const int64_t from = (s < segments ? s : 0) * count;
        a[s] = first[from];
        if (ROWS) b[s] = second[from];
    }
    SegmentSum all;
    all.ref = kNoReference;
    if (ROWS) {
#pragma unroll
        for (int s = 0; s < MOST; ++s) all.ref = fmaxf(all.ref, a[s]);
#pragma unroll
        for (int s = 0; s < MOST; ++s) a[s] = ldexpf(b[s], log2_units(a[s] - all.ref));
    }
#pragma unroll
    for (int s = 0; s < MOST; ++s) if (s < segments) all.add(a[s]);
    if (ROWS) p.lse[at] = log2_of(all.ref, all.total());
    else p.scores[at] = all.total() * (1.0f / (float)n);
}

dim3 grid_of(const ScoreParams& p, int splits, int rows) {
    dim3 g = head_grid((int64_t)p.batch * p.heads, (p.n + rows - 1) / rows);
    if (splits > 1) g.z = splits;
    return g;
}
template <bool ROWS, bool GROUPED>
void launch_half(const ScoreParams& p, int head_dim, int teams, hipStream_t s) {
    const dim3 grid = grid_of(p, 1, 128);
    auto* const kernel = head_dim == 128 ? (teams == 2 ? score_half_bf16_kernel<128, ROWS, GROUPED, 2> : score_half_bf16_kernel<128, ROWS, GROUPED, 1>)
                                         : (teams == 2 ? score_half_bf16_kernel<64, ROWS, GROUPED, 2> : score_half_bf16_kernel<64, ROWS, GROUPED, 1>);
    hipLaunchKernelGGL(kernel, grid, dim3(NTHREADS * teams), 0, s, p);
}

template <bool ROWS>
void launch_combine(const ScoreParams& p, hipStream_t s) {
    const dim3 grid((unsigned)((p.n + NTHREADS - 1) / NTHREADS), (unsigned)(p.batch * p.heads));
    if (p.segment_room <= 4) hipLaunchKernelGGL((score_combine_kernel<ROWS, 4>), grid, dim3(NTHREADS), 0, s, p);
    else if (p.segment_room <= 12) hipLaunchKernelGGL((score_combine_kernel<ROWS, 12>), grid, dim3(NTHREADS), 0, s, p);
    else hipLaunchKernelGGL((score_combine_kernel<ROWS, kMaxScoreSegments>), grid, dim3(NTHREADS), 0, s, p);
}

}  // namespace

void launch_score_combine(const ScoreParams& p, bool rows, hipStream_t s) {
    if (rows) launch_combine<true>(p, s);
    else launch_combine<false>(p, s);
}

hipError_t launch_rowlse_bf16(const ScoreParams& p, int head_dim, hipStream_t s) {
    if (!splits_fit(p, p.row_splits) || (head_dim != 128 && head_dim != 64)) return hipErrorInvalidValue;
    if (p.teams > 0) {
        launch_half<true, false>(p, head_dim, p.teams, s);
        return hipGetLastError();
    }
    const bool cut = p.row_splits > 1;
    const dim3 grid = grid_of(p, p.row_splits, kScoreBlock_bf16);
    auto* const kernel = head_dim == 128 ? (cut ? rowlse_runs_bf16_kernel<128> : rowlse_bf16_kernel<128>)
                                         : (cut ? rowlse_runs_bf16_kernel<64> : rowlse_bf16_kernel<64>);
    hipLaunchKernelGGL(kernel, grid, dim3(NTHREADS), 0, s, p);
    if (cut) launch_score_combine(p, true, s);
    return hipGetLastError();
}

template <int D>
static auto* colmass_kernel(bool groups, bool cut) {
    if (groups) return cut ? colmass_groups_runs_bf16_kernel<D> : colmass_groups_bf16_kernel<D>;
    return cut ? colmass_runs_bf16_kernel<D> : colmass_bf16_kernel<D>;
}

hipError_t launch_colmass_bf16(const ScoreParams& p, int head_dim, hipStream_t s) {
    if (!splits_fit(p, p.col_splits) || (head_dim != 128 && head_dim != 64)) return hipErrorInvalidValue;
    const bool cut = p.col_splits > 1, groups = p.groups > 1;
    if (p.teams > 0) {
        // (teams share out whole groups: two of them only where neither gets much less than half)
        if (groups) launch_half<false, true>(p, head_dim, p.groups >= 8 ? p.teams : 1, s);
        else launch_half<false, false>(p, head_dim, p.teams, s);
        return hipGetLastError();
    }
    const dim3 grid = grid_of(p, p.col_splits, kScoreBlock_bf16);
    hipLaunchKernelGGL((head_dim == 128 ? colmass_kernel<128>(groups, cut) : colmass_kernel<64>(groups, cut)), grid, dim3(NTHREADS), 0, s, p);
    if (cut && !groups) launch_score_combine(p, false, s);
    return hipGetLastError();
}

}  // namespace pulsecol
