// Column-sparse attention with query blocks of 32, 64 or 128 rows: query groups smaller than the 256-row
// query block of the main bf16 kernel (Sec. 3.3: group-wise sets with G = 32, 64 or 128 queries; Sec. 3.4
// and the appendix listing "Column-Sparse Attention Forward" for the computation itself), and short jobs
// with one set per head.
//
// A workgroup = one query block of 32 * NW rows, 32 per wave.  Tiles of 32 gathered rows go straight from
// global memory into one of three LDS slots per operand (two for V in one form; direct-to-LDS loads, issued two
// iterations ahead of their use), online softmax against a lazily raised reference.  Same MFMA orientation as the main
// kernel: S^T = K_tile Q^T, O^T = V^T P^T, P in registers.
//
// Software pipeline: iteration t issues the matrix instructions of S(t+1) = K(t+1) Q^T and of
// O += V(t-1) P(t-1), alternating, while the vector pipe turns S(t) into P(t), one weight behind every
// matrix instruction.  Fences keep that interleaving; the fragment reads are issued from assembly with
// exact wait counts.  (With the three steps of a tile one after the other -- scores, weights, output --
// the waves that share a SIMD fall into step and each pipe idles while the other works, whatever the
// gathers do: with every column set pointing at a single row the kernel took five sixths of its time.)
//
// What bounds it: the matrix pipe under the power limit (32 heads of 8192 rows, D = 128, groups of 128, whole calls: 887
// TFLOP/s on random operands, 1150 on all-zero ones) and the start and end of a block, some 3 us each at keep 10%
// (the four-wave form spills four registers there).  Against the three-step form, inputs from memory: that shape
// 139 -> 136 us, its groups of 64 159 -> 143, of 32 271 -> 232; one set per head, 32 heads of 4096: 42.1 -> 39.7,
// 4 heads of 8192 37.5 -> 21.4; 64K rows: groups of 128 6.69 -> 6.56 ms, 2 heads in groups of 64 1.98 -> 0.47, 32 heads in
// groups of 32 at 32K 3.55 -> 3.08.  Groups of 64 with D = 128 have two V slots: with three a CU holds three workgroups
// of two waves, which was slower than the three-step form at 8 heads of 8192 and over long contexts; with two it holds four.
// 8 heads of 8192 rows three-step form / three V slots / two 40.6 / 47.1 / 37.7 us, 32 heads of 16K 579 / 582 / 528,
// of 64K 8.60 / 8.69 / 7.63 ms.  A fourth slot per operand is slower where every group gathers its own rows (145 us:
// more requests in flight, fewer of them served by the L2), and no faster elsewhere.
//
// Start and end of a query block: a workgroup works through a list of blocks, and requests what the next block needs
// first -- its row numbers, its Q rows (whole rows straight into LDS, into the chunks of the K slots that this wave
// alone fills; read back as fragments), its first K tiles -- while it finishes the running one.  The output tile is
// turned around in the same chunks and leaves in whole rows.
//
// KS > 1: the workgroup has KS teams of NW waves; team s takes the tiles s, s + KS, ... of the same query
// block, and the teams' results are merged through LDS at the end.  For grids that leave CUs with one
// workgroup each.
#include <utility>

#include "attn_reference.h"
#include "pulsecol_device.h"
#include "pulsecol_kernels.h"

namespace pulsecol {
namespace {

typedef unsigned char byte;

constexpr int BN = 32;      // gathered rows per tile
constexpr int NBUF = 3;     // LDS tile slots per operand: one being read, two on their way
constexpr float kNoReference = -1e30f;      // of a query whose first tile holds no finite logit: the tile adds nothing

// s_waitcnt vmcnt(v) with the other counters left alone (gfx9 encoding: vmcnt in [3:0] and [15:14])
template <int v>
__device__ __forceinline__ void wait_vmcnt_at_most() {
    static_assert(v >= 0 && v < 64, "six bits");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (v & 0xF) | ((v & 0x30) << 10));
}
__device__ __forceinline__ void fence() { __builtin_amdgcn_sched_barrier(0); }
// nothing that touches memory moves across this point, neither in the compiler nor in its scheduler
__device__ __forceinline__ void memory_order_point() {
    asm volatile("" ::: "memory");
    fence();
}
__device__ __forceinline__ uint32_t lds_address(const void* generic_lds_ptr) {
    return (uint32_t)(uintptr_t)(PULSECOL_LDS const void*)generic_lds_ptr;
}
// LDS fragment reads as inline assembly with hand-placed waits: the compiler's own wait-count insertion
// drains lgkmcnt to zero in front of every LDS read while a direct-to-LDS load is in flight; LDS returns data
// in order, so "all but the N newest reads" is exact.  The compiler knows neither the latency of these loads
// nor that the destination is written later: each is one statement whose output is a whole variable, and
// nothing reads the variable before the wait that covers it.
template <int OFF>
__device__ __forceinline__ bf16x8 lds_read_b128_at(uint32_t addr) {
    bf16x8 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(v) : "v"(addr), "n"(OFF));
    return v;
}
template <int OFF>
__device__ __forceinline__ bf16x4 lds_read_tr_at(uint32_t addr) {
    bf16x4 v;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=&v"(v) : "v"(addr), "n"(OFF));
    return v;
}
// O += a * p, from assembly so that O stays where it is (left to the compiler the accumulator wanders through the
// register file, twice its size).  In vector registers: a kernel that uses accumulation registers at all gets half of
// its budget as those, and the scores would have to be moved from one half to the other.  The compiler does not know the latency: mfma_settle stands in
// front of every place where the vector pipe reads the accumulator.
__device__ __forceinline__ void mfma_pv(f32x16& o, bf16x8 a, bf16x8 p) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(o) : "v"(a), "v"(p));
}
// Waits out the write-back of every matrix instruction issued so far (the longest MFMA-result-to-VALU hazard on
// gfx950 is 18 wait states); the values are routed through the statement so that no use of them comes before it.
template <int N>
__device__ __forceinline__ void mfma_settle(f32x16 (&o)[N]) {
    static_assert(N == 2 || N == 4, "accumulator blocks");
    if constexpr (N == 4) asm volatile("s_nop 15\n\ts_nop 15" : "+v"(o[0]), "+v"(o[1]), "+v"(o[2]), "+v"(o[3]));
    else asm volatile("s_nop 15\n\ts_nop 15" : "+v"(o[0]), "+v"(o[1]));
}
// One tile of K or of V, this wave's share: CH direct-to-LDS loads, each moving 64 x 16 bytes into the 1 KB
// chunk (wave*CH + i) of the slot.  Lane L lands at chunk byte 16*L, i.e. tile row chunk*RPC + L/PIECES, LDS
// piece L%PIECES, and therefore fetches the global piece (L%PIECES) ^ swizzle(row) of its row: piece_off holds
// that piece's byte offset inside a row.
template <int CH>
__device__ __forceinline__ void issue_tile(byte* __restrict__ slot, const byte* __restrict__ base, const int (&rows)[CH],
                                           const uint32_t (&piece_off)[CH], uint32_t row_bytes, int wave) {
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        // both factors are below 2^24 and the product below 2^32 (checked on the host)
        const uint32_t off = __umul24((uint32_t)rows[i], row_bytes) + piece_off[i];
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(base + off),
                                         (PULSECOL_LDS void*)(slot + (wave * CH + i) * 1024), 16, 0, 0);
    }
}

template <int D, int NW>
struct GroupWave {
    static constexpr int PIECES = D / 8;                 // 16-byte pieces per row
    static constexpr int KK = D / 16;                    // contraction steps of Q K^T
    static constexpr int DB = D / 32;                    // 32-wide blocks of the head dimension
    static constexpr int NPV = 2 * DB;                   // V fragments of a tile: two halves of 16 rows x DB blocks
    static constexpr int ROW_BYTES = D * 2;
    static constexpr int TILE_BYTES = BN * ROW_BYTES;
    static constexpr int RPC = 64 / PIECES;              // tile rows per 1 KB chunk
    static constexpr int CH = TILE_BYTES / 1024 / NW;    // chunks per wave, tile and operand
    static_assert(CH >= 1 && CH * NW * 1024 == TILE_BYTES, "the waves' chunks cover the tile exactly");
    static_assert(KK == NPV, "scores and output take the same number of matrix instructions");
    static constexpr int AHEAD = 4;                      // fragments requested ahead of their use

    int lq, lh;
    float c2;
    bf16x8 qf[KK];               // Q fragments: B operand, [query lq][d = kk*16 + 8*lh .. +7]
    f32x16 o_acc[DB];
    float ref, l_run;            // reference (log2 units) of this lane's query; sum over this lane's keys
    uint32_t kaddr[KK];          // LDS address of K fragment kk in slot 0: tile row lq, piece 2*kk + lh
    uint32_t vaddr[DB];          // ... of the first four rows of the V fragment of d-block db

    // The matrix instructions of an iteration in issue order: scores and output alternate where both run.
    // Instruction f is a K fragment (is_k) with number num(f), and its fragment takes ops(f) LDS reads.
    template <bool QK, bool PV> static constexpr int count() { return (QK ? KK : 0) + (PV ? NPV : 0); }
    template <bool QK, bool PV> static constexpr bool is_k(int f) { return QK && (!PV || f % 2 == 0); }
    template <bool QK, bool PV> static constexpr int num(int f) { return QK && PV ? f / 2 : f; }
    template <bool QK, bool PV> static constexpr int ops(int f) { return is_k<QK, PV>(f) ? 1 : 2; }
    // LDS reads issued behind fragment f when instruction f waits for it
    template <bool QK, bool PV> static constexpr int newer(int f) {
        int c = 0;
        for (int g = f + 1; g < f + AHEAD && g < count<QK, PV>(); ++g) c += ops<QK, PV>(g);
        return c;
    }

    struct Fragment { bf16x8 k; bf16x4 lo, hi; };
    template <bool QK, bool PV, int F, int KOFF, int VOFF>
    __device__ __forceinline__ void request(Fragment& fr) const {
        constexpr int q = num<QK, PV>(F);
        if constexpr (is_k<QK, PV>(F)) {
            fr.k = lds_read_b128_at<KOFF>(kaddr[q]);
        } else {
            // contraction element e of this lane <-> tile row hf*16 + 8*(e/4) + 4*lh + e%4
            constexpr int hf = q / DB, db = q % DB;
            fr.lo = lds_read_tr_at<VOFF + hf * 16 * ROW_BYTES>(vaddr[db]);
            fr.hi = lds_read_tr_at<VOFF + hf * 16 * ROW_BYTES + 8 * ROW_BYTES>(vaddr[db]);
        }
    }

    // Weight of value r of a tile: P in bf16 as the operand of the output product, the row sum in fp32.  Value r is
    // formed while value r-1 is added and packed (an exponential's result may not be used by the next instruction).
    // Pairs are packed at once (the compiler would keep all sixteen weights until the tile is closed); the statement
    // names the sum so that it follows the addition.
    struct Sums { float rs, even, e; };
    __device__ __forceinline__ void add_weight(int r, u32x4 (&P)[2], Sums& sm) const {
        sm.rs = r == 0 ? sm.e : sm.rs + sm.e;
        if (r & 1) {
            uint32_t pair;
            asm volatile("v_cvt_pk_bf16_f32 %0, %2, %3" : "=v"(pair), "+v"(sm.rs) : "v"(sm.even), "v"(sm.e));
            P[r >> 3][(r & 7) >> 1] = pair;
        } else {
            sm.even = sm.e;
        }
    }
    __device__ __forceinline__ void weight(int r, const f32x16& s, u32x4 (&P)[2], Sums& sm) const {
        const float t = __builtin_fmaf(s[r], c2, -ref);
        if (r > 0) add_weight(r - 1, P, sm);
        sm.e = fast_exp2(t);
        if (r == 15) add_weight(15, P, sm);
    }

    template <bool QK, bool PV, bool SM, int F, int KOFF, int VOFF>
    __device__ __forceinline__ void slot(Fragment (&fr)[KK + NPV], const f32x16& s, f32x16& s_next,
                                         const u32x4 (&P_prev)[2], u32x4 (&P)[2], Sums& sm) {
        constexpr int N = count<QK, PV>(), q = num<QK, PV>(F);
        if constexpr (is_k<QK, PV>(F)) {
            asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(fr[F].k) : "n"(newer<QK, PV>(F)));
            if constexpr (q == 0) {
                f32x16 zero;
#pragma unroll
                for (int r = 0; r < 16; ++r) zero[r] = 0.f;
                s_next = mfma_bf16(fr[F].k, qf[q], zero);
            } else {
                s_next = mfma_bf16(fr[F].k, qf[q], s_next);
            }
        } else {
            asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(fr[F].lo), "+v"(fr[F].hi) : "n"(newer<QK, PV>(F)));
            const bf16x8 a = __builtin_shufflevector(fr[F].lo, fr[F].hi, 0, 1, 2, 3, 4, 5, 6, 7);
            mfma_pv(o_acc[q % DB], a, __builtin_bit_cast(bf16x8, P_prev[q / DB]));
        }
        fence();
        if constexpr (F + AHEAD < N) request<QK, PV, F + AHEAD, KOFF, VOFF>(fr[F + AHEAD]);
        if constexpr (SM) {
#pragma unroll
            for (int r = 16 * F / N; r < 16 * (F + 1) / N; ++r) weight(r, s, P, sm);
        }
        fence();
    }
    template <bool QK, bool PV, bool SM, int KOFF, int VOFF, int... Fs>
    __device__ __forceinline__ void slots(Fragment (&fr)[KK + NPV], const f32x16& s, f32x16& s_next,
                                          const u32x4 (&P_prev)[2], u32x4 (&P)[2], Sums& sm, std::integer_sequence<int, Fs...>) {
        (slot<QK, PV, SM, Fs, KOFF, VOFF>(fr, s, s_next, P_prev, P, sm), ...);
    }
    template <bool QK, bool PV, int KOFF, int VOFF>
    __device__ __forceinline__ void request_first(Fragment (&fr)[KK + NPV]) const {
        static_assert(AHEAD == 4, "written out for four");
        request<QK, PV, 0, KOFF, VOFF>(fr[0]);
        request<QK, PV, 1, KOFF, VOFF>(fr[1]);
        request<QK, PV, 2, KOFF, VOFF>(fr[2]);
        request<QK, PV, 3, KOFF, VOFF>(fr[3]);
    }

    // Accept the row sum of a tile, or -- if some lane's weights outgrew the reference (or are NaN) -- fix the
    // reference first: true maximum of the tile per query, reference up by a whole number of log2 units, l and the
    // accumulator scaled by that exact power of two, P recomputed.  Every product that adds an earlier tile's P to
    // the accumulator has been issued.
    __device__ __forceinline__ void close_tile(const f32x16& s, u32x4 (&P)[2], Sums sm) {
        if (__builtin_expect(__ballot(!(sm.rs <= kAttnGrowthLimit)) != 0ull, 0)) {
            float mx = s[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[r]);
            const float m2 = half_max(mx) * c2;              // same value in both half-waves
            if (m2 > ref + 1.0f) {
                const float steps = ceilf(m2 - ref) + kAttnHeadroom;
                const float alpha = fast_exp2(-steps);
                ref = ref == kNoReference ? m2 + kAttnHeadroom : ref + steps;         // (no finite logit so far: alpha is zero)
                l_run *= alpha;
                mfma_settle(o_acc);
#pragma unroll
                for (int db = 0; db < DB; ++db) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) o_acc[db][r] *= alpha;
                    asm volatile("" : "+v"(o_acc[db]));
                }
#pragma unroll
                for (int r = 0; r < 16; ++r) weight(r, s, P, sm);
            }
        }
        l_run += sm.rs;
    }
};

template <int D, int NW, int KS>
__global__ void __launch_bounds__(64 * NW * KS) __attribute__((amdgpu_waves_per_eu(NW == 1 ? 1 : 2)))
attn_bf16_group_kernel(AttnParams p) {
    using W = GroupWave<D, NW>;
    constexpr int BM = 32 * NW;
    constexpr int PIECES = W::PIECES;
    constexpr int KK = W::KK;
    constexpr int DB = W::DB;
    constexpr int ROW_BYTES = W::ROW_BYTES;
    constexpr int TILE_BYTES = W::TILE_BYTES;
    constexpr int RPC = W::RPC;
    constexpr int CH = W::CH;
    // V slots: one fewer for the two-wave block at D = 128, whose V tiles are then requested one iteration ahead of their
    // use: 40 KB of slots leave a CU four workgroups, 48 KB three.
    constexpr int NBUF_V = NW == 2 && D == 128 ? 2 : NBUF;
    constexpr bool LATE_V = NBUF_V == 2;
    constexpr int TEAM_BYTES = (NBUF + NBUF_V) * TILE_BYTES;    // K slots, then V slots
    // Several blocks per workgroup, the next one's start under the end of the running one: for the 128-row block, two
    // workgroups to a CU.  (Smaller ones come three to a CU and cover each other, and have no registers for it.)
    constexpr bool LIST = KS == 1 && NW == 4;

    // (two teams: the reference of every query of the block behind the tile slots)
    __shared__ __attribute__((aligned(1024))) byte lds_all[KS * TEAM_BYTES + (KS > 1 ? BM * 4 : 0)];

    // every kernel argument with the first batch of scalar loads: left to itself the compiler loads them where they
    // are first used, one memory round trip after another
    asm volatile("" : : "s"(p.q), "s"(p.k), "s"(p.v), "s"(p.o), "s"(p.idx), "s"(p.td.sb), "s"(p.td.sh), "s"(p.td.sn),
                         "s"(p.td_kv.sb), "s"(p.td_kv.sh), "s"(p.td_kv.sn), "s"(p.kv_heads), "s"(p.batch), "s"(p.heads),
                         "s"(p.n), "s"(p.ns), "s"(p.groups), "s"(p.group_size), "s"(p.scale), "s"(p.varlen));
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave_wg = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int team = KS > 1 ? wave_wg / NW : 0;
    const int wave = wave_wg - team * NW;
    const int lq = lane & 31;       // query column (and K/V row) this lane owns inside a 32-block
    const int lh = lane >> 5;       // which half of the wave
    // The blocks of XCD x: block by block the whole heads 8 * layer + x, then every eighth block of the heads that are
    // left over.  (Workgroup ids are dealt round-robin over the XCDs, each with its own L2: the rows that a head's blocks
    // share are fetched into a single L2, and all XCDs are in use however few heads there are.)
    const int nqb = (p.n + BM - 1) / BM, heads_all = p.batch * p.heads;
    const int xcd = blockIdx.x & 7, stride = (int)gridDim.x >> 3;
    const int whole = (heads_all >> 3) * nqb, left = (heads_all & 7) * nqb;
    const int list_end = whole + (left > xcd ? (left - xcd + 7) >> 3 : 0);
    int pos = (int)blockIdx.x >> 3;
    // a query block: its head, rows and columns
    struct Block {
        int bh, q0, n, ns;                  // q0: the workgroup's first row
        int64_t q_off, kv_off;              // element offsets of the head in Q / O and in K / V
        const byte* idx;                    // the column set of the block's group
    };
    // the block at `pos`, or the next one behind it that has rows (variable-length batches); false: none
    auto find_block = [&](Block& k) {
        for (; pos < list_end; pos += stride) {
            int qblk;
            if (pos < whole) {
                const int layer = pos / nqb;
                qblk = pos - layer * nqb;
                k.bh = layer * 8 + xcd;
            } else {
                const int i = (pos - whole) * 8 + xcd, hh = i / nqb;
                qblk = i - hh * nqb;
                k.bh = (heads_all & ~7) + hh;
            }
            int b, h;
            split_head(k.bh, p.batch, p.heads, &b, &h);
            k.q0 = qblk * BM;
            k.n = p.n;
            k.ns = p.ns;
            if (p.varlen != nullptr) {
                // the batch element's own length, and the leading `kept` entries of its sets
                k.n = p.varlen[b];
                const int kept = p.varlen[p.batch + b];
                k.ns = kept < k.ns ? kept : k.ns;
                if (k.q0 >= k.n) continue;          // a block of padding rows
            }
            k.q_off = (int64_t)b * p.td.sb + (int64_t)h * p.td.sh;
            // grouped-query layout: query head h reads K/V head h / (heads / kv_heads)
            k.kv_off = (int64_t)b * p.td_kv.sb + (int64_t)kv_head_of(h, p.heads, p.kv_heads) * p.td_kv.sh;
            // group_size is a multiple of BM
            const int group = p.groups > 1 ? k.q0 / p.group_size : 0;
            k.idx = (const byte*)(p.idx + ((int64_t)k.bh * p.groups + group) * p.ns);
            return true;
        }
        return false;
    };
    Block cur, next;
    if (!find_block(cur)) return;
    const uint32_t row_bytes = (uint32_t)p.td_kv.sn * 2u, q_row_bytes = (uint32_t)p.td.sn * 2u;
    byte* const lds_k = lds_all + team * TEAM_BYTES;
    byte* const lds_v = lds_k + NBUF * TILE_BYTES;

    W w;
    w.lq = lq;
    w.lh = lh;
    w.c2 = p.scale * kLog2e;                // exp(z*scale) = exp2(z*c2)
    // ---- gather geometry: chunk i of the wave covers tile rows (wave*CH + i)*RPC + lrow, lrow = lane/PIECES, and
    // takes the positions wave*16*.. + lrow*CH + i of the tile, K and V alike: a lane's CH positions are then
    // consecutive entries of the pattern.
    const int lrow = lane / PIECES;
    const int first_pos = wave * CH * RPC + lrow * CH;
    uint32_t koff[CH], voff[CH];
#pragma unroll
    for (int i = 0; i < CH; ++i) {
        const int row = (wave * CH + i) * RPC + lrow;
        koff[i] = (uint32_t)((lane % PIECES) ^ swizzle_k<PIECES>(row)) * 16u;
        voff[i] = (uint32_t)((lane % PIECES) ^ swizzle_v<PIECES>(row)) * 16u;
    }
    // position inside its tile of the key in LDS tile row `row`
    auto tile_pos = [&](int row) {
        const int chunk = row / RPC;
        return (chunk / CH) * CH * RPC + (row % RPC) * CH + chunk % CH;
    };
    // Row numbers of the team's tile t for this lane's chunks.  Positions past the end of the pattern (ragged tail,
    // tiles past the last one) take the pattern's last entry: a valid row, whose scores the tail mask removes or
    // whose slot is never read.
    auto load_rows = [&](const Block& k, int t, int (&dst)[CH]) {
        const uint32_t start = (uint32_t)(t * KS + team) * BN + first_pos, end = (uint32_t)(k.ns - 1);
#pragma unroll
        for (int i = 0; i < CH; ++i) dst[i] = *(const int*)(k.idx + (start + i < end ? start + i : end) * 4u);    // 32-bit offsets from the uniform base
    };
    // The lane's number, hidden from the compiler's loop-invariant hoisting: it would compute every address of a block's
    // start and end that follows from it in front of the loop over the blocks and, with no registers for them, keep
    // them in scratch.
    auto fresh_lane = [] {
        int l = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        asm volatile("" : "+v"(l));
        return l;
    };
    // This wave's own part of the tile slots, where its 32 rows of Q arrive and its output tile is turned around: chunk
    // range `wave` of NW slots, 32 / NW rows in each: the K slots, then V slot `vslot`; for the first block's Q
    // (vslot = -1) the V slots, then the last K slot, so that the first K tiles need not wait for it.
    constexpr int OWN = TILE_BYTES / NW;                 // bytes per slot
    constexpr int OWN_ROWS = 32 / NW;
    auto own_part = [&](int i, int vslot) {              // byte offset of part i from the team's first slot
        const int slot = vslot < 0 ? (i < NBUF ? NBUF + i : NBUF - 1) : (i < NBUF ? i : NBUF + vslot);
        return slot * TILE_BYTES + wave * OWN;
    };
    static_assert(NW <= NBUF + 1, "K slots and one V slot");
    static_assert(!LATE_V || (NW <= 2 && !LIST && KS == 1), "Q and O pass through two slots of an operand");
    // Q rows of a block: CH loads per part, RPC rows each, piece (lane % PIECES) ^ swizzle(row) of a row
    auto request_q = [&](const Block& k, int vslot) {
        const int lane = fresh_lane(), lrow = lane / PIECES;
        const byte* Q = (const byte*)((const __bf16*)p.q + k.q_off);
#pragma unroll
        for (int i = 0; i < NW; ++i)
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const int r = i * OWN_ROWS + c * RPC + lrow;             // 0 .. 31
                int row = k.q0 + wave * 32 + r;
                row = row < k.n ? row : k.n - 1;
                // both factors are below 2^24 and the product below 2^32 (checked on the host)
                const uint32_t off = __umul24((uint32_t)row, q_row_bytes) + (uint32_t)(((lane % PIECES) ^ swizzle_k<PIECES>(r)) << 4);
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(Q + off),
                                                 (PULSECOL_LDS void*)(lds_k + own_part(i, vslot) + c * 1024), 16, 0, 0);
            }
    };
    constexpr int Q_LOADS = NW * CH;
    // ... and their fragments, B operand: [query lq][d = kk*16 + 8*lh .. +7]
    auto read_q = [&](int vslot) {
        const int lane = fresh_lane(), lq = lane & 31, lh = lane >> 5;
        const int i = lq / OWN_ROWS;
        const byte* row = lds_k + own_part(i, vslot) + (lq % OWN_ROWS) * ROW_BYTES;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) w.qf[kk] = *(const bf16x8*)(row + (((2 * kk + lh) ^ swizzle_k<PIECES>(lq)) << 4));
    };

    // ---- fragment addresses in slot 0: what differs between slots and between the halves of a tile are constants,
    // which the reads carry as instruction offsets
    const uint32_t k0 = lds_address(lds_k), v0 = lds_address(lds_v);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) w.kaddr[kk] = k0 + (uint32_t)(lq * ROW_BYTES + (((2 * kk + lh) ^ swizzle_k<PIECES>(lq)) << 4));
    // the transposing read takes the address of row 4*lh + j16/4 (then +8, and +16 for the second half: rows with
    // the same swizzle), 8 bytes at d = db*32 + 16*((lane/16)&1) + 4*(j16%4), j16 = lane%16
    {
        const int j16 = lane & 15;
        const int row0 = 4 * lh + (j16 >> 2);
        const int colpiece = ((lane >> 4) & 1) * 2 + ((j16 & 3) >> 1);   // 16-byte piece inside the 64-byte d-block
        const int inpiece = (j16 & 1) * 8;                               // byte inside the piece
        static_assert(PIECES >= 8, "rows 8 and 16 apart share a swizzle");
#pragma unroll
        for (int db = 0; db < DB; ++db)
            w.vaddr[db] = v0 + (uint32_t)(row0 * ROW_BYTES + inpiece + (((db * 4 + colpiece) ^ swizzle_v<PIECES>(row0)) << 4));
    }
    // ---- Loads.  Iteration t reads K(t+1) and V(t-1) and issues K(t+3) and V(t+1), which replace K(t) and V(t-2),
    // both read in iteration t-1 (two V slots: V(t) and K(t+3); V(t) replaces V(t-2)).  rows_a .. rows_d: row numbers of
    // the tiles t+1 .. t+4 (V of t+1 now, K of t+3 now); rows_0, two V slots: of tile t.
    int rows_0[CH], rows_a[CH], rows_b[CH], rows_c[CH], rows_d[CH];
    const byte* K;
    const byte* V;
    // Row numbers of a block's first four tiles.
    auto request_rows = [&](const Block& k) {
        load_rows(k, 0, rows_0);
        load_rows(k, 1, rows_a);
        load_rows(k, 2, rows_b);
        load_rows(k, 3, rows_c);
    };
    // (named in front of the first direct-to-LDS load that uses them: behind one the compiler would wait for everything
    // in flight to have these)
    auto rows_arrived = [&] {
#pragma unroll
        for (int i = 0; i < CH; ++i) asm volatile("" : "+v"(rows_0[i]), "+v"(rows_a[i]), "+v"(rows_b[i]), "+v"(rows_c[i]));
    };
    // The same for the workgroup's first block, from assembly, and named in the wait that covers them: the compiler does
    // not know that vector memory returns in issue order where direct-to-LDS loads are in flight, and would wait for
    // the Q rows behind them too.
    auto request_first_rows = [&] {
        int (&r0)[CH] = rows_0, (&r1)[CH] = rows_a, (&r2)[CH] = rows_b, (&r3)[CH] = rows_c;
        const byte* const idx = cur.idx;
        const uint32_t end = (uint32_t)(cur.ns - 1) * 4u;
        auto offset = [&](int t, int i) {
            const uint32_t off = ((uint32_t)(t * KS + team) * BN + first_pos + i) * 4u;
            return off < end ? off : end;
        };
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            asm volatile("global_load_dword %0, %1, %2" : "=&v"(r0[i]) : "v"(offset(0, i)), "s"(idx));
            asm volatile("global_load_dword %0, %1, %2" : "=&v"(r1[i]) : "v"(offset(1, i)), "s"(idx));
            asm volatile("global_load_dword %0, %1, %2" : "=&v"(r2[i]) : "v"(offset(2, i)), "s"(idx));
            asm volatile("global_load_dword %0, %1, %2" : "=&v"(r3[i]) : "v"(offset(3, i)), "s"(idx));
        }
    };
    auto first_rows_arrived = [&](auto newer_c) {
        int (&r0)[CH] = rows_0, (&r1)[CH] = rows_a, (&r2)[CH] = rows_b, (&r3)[CH] = rows_c;
#pragma unroll
        for (int i = 0; i < CH; ++i)
            asm volatile("s_waitcnt vmcnt(%4)" : "+v"(r0[i]), "+v"(r1[i]), "+v"(r2[i]), "+v"(r3[i]) : "n"(decltype(newer_c)::value));
    };
    auto request_k01 = [&](const Block& k) {
        K = (const byte*)((const __bf16*)p.k + k.kv_off);
        V = (const byte*)((const __bf16*)p.v + k.kv_off);
        issue_tile<CH>(lds_k, K, rows_0, koff, row_bytes, wave);                       // K(0)
        issue_tile<CH>(lds_k + TILE_BYTES, K, rows_a, koff, row_bytes, wave);          // K(1)
    };
    auto request_k2v0 = [&] {
        issue_tile<CH>(lds_k + 2 * TILE_BYTES, K, rows_b, koff, row_bytes, wave);      // K(2)
        issue_tile<CH>(lds_v, V, rows_0, voff, row_bytes, wave);                       // V(0)
    };
    // ---- the first block
    request_first_rows();
    memory_order_point();
    request_q(cur, -1);
    memory_order_point();
    first_rows_arrived(std::integral_constant<int, Q_LOADS>{});
    memory_order_point();
    request_k01(cur);
    wait_vmcnt_at_most<2 * CH>();
    memory_order_point();
    read_q(-1);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) asm volatile("" : "+v"(w.qf[kk]));         // (read before tiles replace it)
    memory_order_point();
    request_k2v0();
    int newer_stores = 0;                   // stores of the block before, issued behind this block's first tiles

    for (;;) {
    const int n = cur.n, ns = cur.ns;
    // iterations: the tiles of this team are team, team + KS, ...; a team that runs out one early works on a tile
    // past the end, all of whose weights are zero
    const int tiles = ((ns + BN - 1) / BN + KS - 1) / KS;
    w.l_run = 0.f;
#pragma unroll
    for (int db = 0; db < DB; ++db) {
#pragma unroll
        for (int r = 0; r < 16; ++r) w.o_acc[db][r] = 0.f;
        asm volatile("" : "+v"(w.o_acc[db]));
    }
    bool more = false;
    // What the next block needs first, requested while the last tile of this one is worked on: no wave reads K any more,
    // nor the V slot of the tile in front of the last two.
    auto begin_next = [&](int vslot) {
        if constexpr (LIST) {
            pos += stride;
            more = find_block(next);
            if (more) {
                request_rows(next);
                memory_order_point();
                request_q(next, vslot);
                memory_order_point();
            }
        }
    };
    // ragged tail of the last tile, or a tile past the end: positions past ns get weight zero
    auto mask_tail = [&](int t, f32x16& s) {
        const int valid = ns - (t * KS + team) * BN;
        if (valid < BN) {
            const int lh = fresh_lane() >> 5;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (tile_pos(acc_row(r, lh)) >= valid) s[r] = -INFINITY;
        }
    };
    f32x16 sa, sb;
    u32x4 pa[2], pb[2];
    typename W::Sums sm{0.f, 0.f, 0.f};
    const int last = tiles - 1;
    // ---- S(0), which sets the reference: from the maximum of the first tile
    if (newer_stores == NW * CH) wait_vmcnt_at_most<3 * CH + NW * CH>();
    else wait_vmcnt_at_most<3 * CH>();
    memory_order_point();
    __builtin_amdgcn_s_barrier();
    memory_order_point();
    {
        typename W::Fragment fr[KK + W::NPV];
        w.template request_first<true, false, 0, 0>(fr);
        w.template slots<true, false, false, 0, 0>(fr, sb, sa, pb, pa, sm, std::make_integer_sequence<int, KK>{});
    }
    if (last == 0) mask_tail(0, sa);
    {
        float mx = sa[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sa[r]);
        w.ref = fmaxf(half_max(mx) * w.c2 + kAttnHeadroom, kNoReference);
    }
    // Two teams: both weigh against the reference that team 0 takes from the block's first tile, handed over behind the
    // next barrier.  A weight then has the same bits whichever team forms it, in this form of the kernel or in the one
    // with a single team, as a raise moves the reference by whole log2 units: the forms differ in the order of fp32 sums alone.
    // (Each team with a reference of its own rounded half of the weights to other 16-bit values.)
    const uint32_t ref_at = lds_address(lds_all) + (uint32_t)(KS * TEAM_BYTES + (wave * 32 + lq) * 4);
    if (KS > 1 && team == 0) asm volatile("ds_write_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : : "v"(ref_at), "v"(w.ref) : "memory");
    auto common_reference = [&] {
        if constexpr (KS > 1) asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(w.ref) : "v"(ref_at) : "memory");
    };

    // Iteration t, U = t % NBUF: S(t) in s -> P(t) in P, S(t+1) in s_next, P(t-1) in P_prev.  K(t+1) and V(t-1) have
    // landed in every wave once this wave's loads of the iteration before are the only ones it still may have in
    // flight (two V slots: its K loads; vector memory completes in issue order, and whatever this iteration issues comes
    // later still) and all waves have said so at the barrier.  Loads are issued for tiles past the end as well (valid rows, slots never
    // read), so the count in flight is the same at every iteration but the first, in front of which K(2) and V(0)
    // stand in the place of two iterations' loads.  E = (t - 1) % 2, the slot of V(t-1) where there are two.
    auto iterate = [&](auto u_c, auto e_c, auto qk_c, auto pv_c, int t, f32x16& s, f32x16& s_next, u32x4 (&P_prev)[2], u32x4 (&P)[2]) {
        constexpr int U = decltype(u_c)::value, E = decltype(e_c)::value;
        constexpr bool QK = decltype(qk_c)::value, PV = decltype(pv_c)::value;
        constexpr int KOFF = (U + 1) % NBUF * TILE_BYTES, VOFF = (LATE_V ? E : (U + 2) % NBUF) * TILE_BYTES;
        wait_vmcnt_at_most<(LATE_V && PV ? 1 : 2) * CH>();
        memory_order_point();
        __builtin_amdgcn_s_barrier();
        memory_order_point();
        if constexpr (!PV) common_reference();              // the first tile's weights come next
        typename W::Fragment fr[KK + W::NPV];
        w.template request_first<QK, PV, KOFF, VOFF>(fr);
        memory_order_point();
        if constexpr (!QK) begin_next((t + 1) % NBUF);
        if constexpr (!QK && LATE_V) {
            issue_tile<CH>(lds_v + (t & 1) * TILE_BYTES, V, rows_0, voff, row_bytes, wave);             // V(t), the last one
            memory_order_point();
        }
        if constexpr (QK) {
            // (in front of this iteration's loads, so that the next iteration's wait covers the row numbers)
            load_rows(cur, t + 4, rows_d);
            memory_order_point();
            // (V(0) of two slots went out in front of the first iteration)
            if constexpr (LATE_V && PV) issue_tile<CH>(lds_v + (1 - E) * TILE_BYTES, V, rows_0, voff, row_bytes, wave);        // V(t)
            issue_tile<CH>(lds_k + U * TILE_BYTES, K, rows_c, koff, row_bytes, wave);                   // K(t+3)
            if constexpr (!LATE_V) issue_tile<CH>(lds_v + (U + 1) % NBUF * TILE_BYTES, V, rows_a, voff, row_bytes, wave);      // V(t+1)
            memory_order_point();
        }
        w.template slots<QK, PV, true, KOFF, VOFF>(fr, s, s_next, P_prev, P, sm, std::make_integer_sequence<int, W::template count<QK, PV>()>{});
        w.close_tile(s, P, sm);
        if constexpr (QK) {
#pragma unroll
            for (int i = 0; i < CH; ++i) { if (LATE_V) rows_0[i] = rows_a[i]; rows_a[i] = rows_b[i]; rows_b[i] = rows_c[i]; rows_c[i] = rows_d[i]; }
        }
    };
    using Yes = std::true_type;
    using No = std::false_type;
    using Even = std::integral_constant<int, 0>;
    using Odd = std::integral_constant<int, 1>;
    if (last > 0) {
        iterate(std::integral_constant<int, 0>{}, Odd{}, Yes{}, No{}, 0, sa, sb, pb, pa);
        if (last == 1) mask_tail(1, sb);
        for (int t = 1; t < last; t += 6) {
            // six iterations: the slots repeat after three, the roles of the registers after two
            iterate(std::integral_constant<int, 1>{}, Even{}, Yes{}, Yes{}, t, sb, sa, pa, pb);
            if (t + 1 >= last) break;
            iterate(std::integral_constant<int, 2>{}, Odd{}, Yes{}, Yes{}, t + 1, sa, sb, pb, pa);
            if (t + 2 >= last) break;
            iterate(std::integral_constant<int, 0>{}, Even{}, Yes{}, Yes{}, t + 2, sb, sa, pa, pb);
            if (t + 3 >= last) break;
            iterate(std::integral_constant<int, 1>{}, Odd{}, Yes{}, Yes{}, t + 3, sa, sb, pb, pa);
            if (t + 4 >= last) break;
            iterate(std::integral_constant<int, 2>{}, Even{}, Yes{}, Yes{}, t + 4, sb, sa, pa, pb);
            if (t + 5 >= last) break;
            iterate(std::integral_constant<int, 0>{}, Odd{}, Yes{}, Yes{}, t + 5, sa, sb, pb, pa);
        }
        // ---- the last tile: S in sa, the tile before's P in pb, whichever iteration the loop ended with
        if (last & 1) {
            sa = sb;
            pb[0] = pa[0];
            pb[1] = pa[1];
        }
        if (last > 1) mask_tail(last, sa);
        // slot 0 of the addresses becomes the slot of V(last - 1) as iteration 2 of an unrolled run reads it
#pragma unroll
        for (int db = 0; db < DB; ++db) w.vaddr[db] += (uint32_t)((last - 1) % NBUF_V) * TILE_BYTES;
        iterate(std::integral_constant<int, 1>{}, Even{}, No{}, Yes{}, last, sa, sb, pb, pa);
#pragma unroll
        for (int db = 0; db < DB; ++db) w.vaddr[db] += (uint32_t)(last % NBUF_V - (last - 1) % NBUF_V) * TILE_BYTES;
    } else {
        __builtin_amdgcn_s_barrier();                       // every wave has read K(0)
        memory_order_point();
        common_reference();
        begin_next(1);
#pragma unroll
        for (int r = 0; r < 16; ++r) w.weight(r, sa, pa, sm);
        w.close_tile(sa, pa, sm);
    }
    // ---- O += V(last) P(last)
    if (more) wait_vmcnt_at_most<Q_LOADS>();      // (the next block's Q is newer)
    else wait_vmcnt_at_most<0>();
    memory_order_point();
    __builtin_amdgcn_s_barrier();
    memory_order_point();
    typename W::Fragment fr[KK + W::NPV];
    w.template request_first<false, true, 0, 0>(fr);
    w.template slots<false, true, false, 0, 0>(fr, sa, sb, pa, pb, sm, std::make_integer_sequence<int, W::NPV>{});

#pragma unroll
    for (int db = 0; db < DB; ++db) w.vaddr[db] -= (uint32_t)(last % NBUF_V) * TILE_BYTES;       // the next block starts from slot 0 again

    // ---- epilogue: O = diag(l)^-1 acc; hand-over to the next block
    const int vslot = (last + 1) % NBUF;
    if (more) {
        wait_vmcnt_at_most<0>();
        memory_order_point();
        read_q(vslot);
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) asm volatile("" : "+v"(w.qf[kk]));     // (read before the output replaces it)
    }
    mfma_settle(w.o_acc);
    float l_tot = half_sum(w.l_run);
    // d-blocks db0 .. db1-1 of this wave's rows, 1/l applied, turned around in its own part of the slots: in the
    // accumulator a lane holds one row in 8-byte runs; stored from there every instruction would touch 32 rows
    auto stage = [&](auto db0_c, auto db1_c) {
        constexpr int db0 = decltype(db0_c)::value, db1 = decltype(db1_c)::value;
        const int lane = fresh_lane(), lq = lane & 31, lh = lane >> 5;
        const float inv = 1.0f / l_tot;
        const int i = lq / OWN_ROWS;
        byte* const row = lds_k + own_part(i, vslot) + (lq % OWN_ROWS) * ROW_BYTES;
#pragma unroll
        for (int db = db0; db < db1; ++db)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                bf16x4 o4;
#pragma unroll
                for (int e = 0; e < 4; ++e) o4[e] = (__bf16)(w.o_acc[db][r4 * 4 + e] * inv);
                *(bf16x4*)(row + (((db * 4 + r4) ^ swizzle_k<PIECES>(lq)) << 4) + 8 * lh) = o4;
            }
    };
    const int first_row = cur.q0 + wave * 32;
    byte* const O = (byte*)((__bf16*)p.o + cur.q_off);
    // whole rows, 16 bytes per lane; `part` of the pieces only where two teams share the rows
    u32x4 rows_out[NW * CH];
    const int lane_out = fresh_lane();
    auto read_back = [&] {
#pragma unroll
        for (int i = 0; i < NW; ++i)
#pragma unroll
            for (int c = 0; c < CH; ++c) {
                const int r = i * OWN_ROWS + c * RPC + lane_out / PIECES;
                rows_out[i * CH + c] = *(const u32x4*)(lds_k + own_part(i, vslot) + (c * RPC + lane_out / PIECES) * ROW_BYTES +
                                                       (((lane_out % PIECES) ^ swizzle_k<PIECES>(r)) << 4));
            }
    };
    auto store = [&](int i, int c) {
        const int r = i * OWN_ROWS + c * RPC + lane_out / PIECES;
        *(u32x4*)(O + (int64_t)(first_row + r) * q_row_bytes + (lane_out % PIECES) * 16) = rows_out[i * CH + c];
    };
    if constexpr (KS == 1) {
        stage(std::integral_constant<int, 0>{}, std::integral_constant<int, DB>{});
        read_back();
#pragma unroll
        for (int i = 0; i < NW * CH; ++i) asm volatile("" : "+v"(rows_out[i]));
        memory_order_point();
        if (more) {
            rows_arrived();
            __builtin_amdgcn_s_barrier();                   // every wave has read its last V fragments
            memory_order_point();
            request_k01(next);
            request_k2v0();
            memory_order_point();
        }
        // (all of them or none without a test: the next block's first wait counts them)
        if (first_row + 32 <= n) {
#pragma unroll
            for (int i = 0; i < NW; ++i)
#pragma unroll
                for (int c = 0; c < CH; ++c) store(i, c);
            newer_stores = NW * CH;
        } else {
#pragma unroll
            for (int i = 0; i < NW; ++i)
#pragma unroll
                for (int c = 0; c < CH; ++c)
                    if (first_row + i * OWN_ROWS + c * RPC + lane_out / PIECES < n) store(i, c);
            newer_stores = 0;
        }
        if (!LIST || !more) return;
        cur = next;
    } else {
        // The two teams hold the same rows: each hands the other one half of its d-blocks, its reference and its
        // sum, and finishes the other half.
        static_assert(KS == 2 && DB % 2 == 0, "two teams, two halves");
        constexpr int HALF = DB / 2;
        constexpr int WAVE_BYTES = HALF * 4 * 64 * 16;
        static_assert(2 * NW * (WAVE_BYTES + 512) <= KS * TEAM_BYTES, "the exchange fits the tile slots");
        byte* const mine = lds_all + (team * NW + wave) * (WAVE_BYTES + 512);
        const byte* const theirs = lds_all + ((1 - team) * NW + wave) * (WAVE_BYTES + 512);
        __syncthreads();                                    // every wave has read its last V fragments
        auto give = [&](auto db0_c) {
            constexpr int db0 = decltype(db0_c)::value;
#pragma unroll
            for (int i = 0; i < HALF * 4; ++i) {
                f32x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = w.o_acc[db0 + i / 4][(i % 4) * 4 + e];
                *(f32x4*)(mine + (i * 64 + lane) * 16) = v;
            }
            float* const rl = (float*)(mine + WAVE_BYTES);
            rl[lane] = w.ref;
            rl[64 + lane] = l_tot;
        };
        auto take = [&](auto db0_c) {
            constexpr int db0 = decltype(db0_c)::value;
            const float* const rl = (const float*)(theirs + WAVE_BYTES);
            const float their_ref = rl[lane], top = fmaxf(w.ref, their_ref);
            const float a = fast_exp2(w.ref - top), c = fast_exp2(their_ref - top);
            l_tot = l_tot * a + rl[64 + lane] * c;
#pragma unroll
            for (int i = 0; i < HALF * 4; ++i) {
                const f32x4 v = *(const f32x4*)(theirs + (i * 64 + lane) * 16);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int r = (i % 4) * 4 + e;
                    w.o_acc[db0 + i / 4][r] = w.o_acc[db0 + i / 4][r] * a + v[e] * c;
                }
            }
        };
        if (team == 0) give(std::integral_constant<int, HALF>{});
        else give(std::integral_constant<int, 0>{});
        __syncthreads();
        if (team == 0) take(std::integral_constant<int, 0>{});
        else take(std::integral_constant<int, HALF>{});
        __syncthreads();                                    // the exchange has been read
        if (team == 0) stage(std::integral_constant<int, 0>{}, std::integral_constant<int, HALF>{});
        else stage(std::integral_constant<int, HALF>{}, std::integral_constant<int, DB>{});
        read_back();
        // this team's half of the pieces of every row
#pragma unroll
        for (int i = 0; i < NW; ++i)
#pragma unroll
            for (int c = 0; c < CH; ++c)
                if (lane_out % PIECES / (PIECES / 2) == team && first_row + i * OWN_ROWS + c * RPC + lane_out / PIECES < n) store(i, c);
        return;
    }
    }
}

// workgroups of 128-row blocks that one CU holds at a time (registers)
template <int D> constexpr int resident_per_cu() { return D == 128 ? 2 : 3; }

template <int D, int NW, int KS>
hipError_t launch(const AttnParams& p, hipStream_t s) {
    const int64_t blocks = (int64_t)((p.n + 32 * NW - 1) / (32 * NW)) * p.batch * p.heads;
    int64_t grid = (int64_t)compute_units() * resident_per_cu<D>();
    // A workgroup per block for the others, and where every block has a set of its own: lists start the blocks of a head
    // in step, which costs the gathers 2% there (32 heads of 8192 rows, groups of 128: 138 against 136 us) and is worth
    // as much with one set per head.
    if (NW < 4 || KS > 1 || p.groups > 1 || blocks < grid) grid = blocks;
    hipLaunchKernelGGL((attn_bf16_group_kernel<D, NW, KS>), dim3((unsigned)((grid + 7) / 8 * 8)), dim3(64 * NW * KS), 0, s, p);
    return hipGetLastError();
}

template <int D>
hipError_t launch_by_block(const AttnParams& p, int block_m, hipStream_t s) {
    if (block_m == 128) {
        // Two teams where every block can have a CU to itself (two waves per SIMD either way): 4 heads of 8192 rows
        // 22 -> 19 us.  With fewer than four tiles there is nothing to share out.
        const int64_t items = (int64_t)((p.n + 127) / 128) * p.batch * p.heads;
        return items <= compute_units() && p.ns >= 4 * BN ? launch<D, 4, 2>(p, s) : launch<D, 4, 1>(p, s);
    }
    if (block_m == 64) return launch<D, 2, 1>(p, s);
    if (block_m == 32) return launch<D, 1, 1>(p, s);
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_attn_bf16_group(const AttnParams& p, int head_dim, int block_m, hipStream_t s) {
    if (p.idx == nullptr || p.v == nullptr || p.o == nullptr) return hipErrorInvalidValue;
    if (p.groups > 1 && p.group_size % block_m != 0) return hipErrorInvalidValue;
    if (head_dim == 128) return launch_by_block<128>(p, block_m, s);
    if (head_dim == 64) return launch_by_block<64>(p, block_m, s);
    return hipErrorInvalidValue;
}

}  // namespace pulsecol
