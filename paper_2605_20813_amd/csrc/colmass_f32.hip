// Column softmax mass, fp32 inputs (Sec. 3.3, score equation, per query group G_u of a head):
//   s_{u,j} = (1/|G_u|) sum_{i in G_u} exp2(z_ij * scale * log2(e) - lse2_i)
// with lse2_i = log2 sum_j exp(z_ij * scale) from the row pass (attn_f32.hip, lse-only mode).
//
// K-stationary like the bf16 kernel, on v_mfma_f32_32x32x2_f32: a workgroup owns 128 key
// columns (4 waves x 32 keys held in registers as the A operand) and streams 32-row Q tiles
// through padded LDS; for grids that would leave the chip idle, a workgroup = 32 key columns whose Q tiles are shared
// out among its waves.  Fixed summation order, no floating-point atomics.
#include "pulsecol_device.h"
#include "pulsecol_kernels.h"

namespace pulsecol {
namespace {

constexpr int NTHREADS = 256;
constexpr int KEYS_PER_WG = 128;
constexpr int QT = 32;
constexpr int PAD = 4;
constexpr int FLUSH = 16;

template <int D>
__global__ void __launch_bounds__(NTHREADS) colmass_f32_kernel(ScoreParams p) {
    constexpr int PIECES = D / 4;
    constexpr int KK = D / 2;
    constexpr int CH = QT * PIECES / NTHREADS;
    constexpr int LDW = D + PAD;

    __shared__ __attribute__((aligned(16))) float lds_q[QT * LDW];
    __shared__ float lds_lse[QT];

    const int nkb = (p.n + KEYS_PER_WG - 1) / KEYS_PER_WG;
    int bh, kblk;
    if (!xcd_tile(blockIdx.x, nkb, p.batch * p.heads, &bh, &kblk)) return;
    const int b = bh / p.heads, h = bh - b * p.heads;
    // variable-length batches: queries and keys of this batch element end at its own length
    const int n = p.varlen != nullptr ? p.varlen[b] : p.n;
    if (kblk * KEYS_PER_WG >= n) return;    // a block of padding keys: its scores are left untouched
    const int64_t head_off = (int64_t)b * p.td.sb + (int64_t)h * p.td.sh;
    // grouped-query layout: query head h reads K/V head h / (heads / kv_heads)
    const int64_t kv_off = (int64_t)b * p.td_kv.sb + (int64_t)(h / (p.heads / p.kv_heads)) * p.td_kv.sh;
    const float* __restrict__ Q = (const float*)p.q + head_off;
    const float* __restrict__ K = (const float*)p.k + kv_off;
    const float* __restrict__ lse = p.lse + (int64_t)bh * p.n;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int lq = lane & 31, lh = lane >> 5;
    const int key0 = kblk * KEYS_PER_WG + wave * 32;

    float kf[KK];    // A operand: K[key lq][d = 2*kk + lh]
    {
        int row = key0 + lq;
        row = row < n ? row : n - 1;
        const float* src = K + (int64_t)row * p.td_kv.sn + lh;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) kf[kk] = src[2 * kk];
    }

    f32x4 stage[CH];
    float stage_lse = 0.f;
    auto fetch = [&](int t) {
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            const int c = tid + NTHREADS * j;
            int row = t * QT + c / PIECES;
            row = row < n ? row : n - 1;
            stage[j] = *(const f32x4*)(Q + (int64_t)row * p.td.sn + (c % PIECES) * 4);
        }
        if (tid < QT) {
            const int row = t * QT + tid;
            stage_lse = row < n ? lse[row] : INFINITY;     // rows past the end contribute exp2(-inf) = 0
        }
    };
    auto commit = [&]() {
#pragma unroll
        for (int j = 0; j < CH; ++j) {
            const int c = tid + NTHREADS * j;
            *(f32x4*)(lds_q + (c / PIECES) * LDW + (c % PIECES) * 4) = stage[j];
        }
        if (tid < QT) lds_lse[tid] = stage_lse;
    };

    const int ntiles = (n + QT - 1) / QT;
    const float c2 = p.scale * kLog2e;
    f32x16 acc_short, acc_long;
#pragma unroll
    for (int r = 0; r < 16; ++r) { acc_short[r] = 0.f; acc_long[r] = 0.f; }

    fetch(0);
    for (int t = 0; t < ntiles; ++t) {
        __syncthreads();
        commit();
        __syncthreads();
        if (t + 1 < ntiles) fetch(t + 1);

        f32x16 s;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
        const float* qrow = lds_q + lq * LDW + lh;     // B operand: Q[query lq][d = 2*kk + lh]
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) s = mfma_f32(kf[kk], qrow[2 * kk], s);
        const float l2 = lds_lse[lq];
#pragma unroll
        for (int r = 0; r < 16; ++r) acc_short[r] += exp2f(__builtin_fmaf(s[r], c2, -l2));
        if ((t % FLUSH) == FLUSH - 1) {
#pragma unroll
            for (int r = 0; r < 16; ++r) { acc_long[r] += acc_short[r]; acc_short[r] = 0.f; }
        }
        // ---- last tile of a query group: combine lanes (fixed butterfly), divide by the group's
        // size, store the group's score row, start over
        const int rows_done = (t + 1) * QT;
        const bool group_end = t + 1 == ntiles || (p.groups > 1 && rows_done % p.group_size == 0);
        if (group_end) {
            const int u = p.groups > 1 ? (t * QT) / p.group_size : 0;
            const int g_first = p.groups > 1 ? u * p.group_size : 0;
            const int g_rows = (rows_done < n ? rows_done : n) - g_first;
            const float inv = 1.0f / (float)g_rows;
            float* __restrict__ out = p.scores + ((int64_t)bh * p.groups + u) * p.n;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float v = acc_long[r] + acc_short[r];
#pragma unroll
                for (int m = 1; m < 32; m <<= 1) v += __shfl_xor(v, m, 64);
                const int key = key0 + acc_row(r, lh);
                if (lq == 0 && key < n) out[key] = v * inv;
                acc_long[r] = 0.f;
                acc_short[r] = 0.f;
            }
        }
    }
}

// ---- Few keys: a workgroup owns 32 of them, held as the B operand (lane = key column, so a column's sum is an in-lane
// sum), wave w of KS takes the 32-row Q tiles w, w + KS, ... of every query group, straight from memory as A fragments
// (half of the wave h holds the columns h*D/2 .. of a row; the same permutation of the contraction index on the K side),
// the next tile requested behind the last product that reads the running one.  The waves' sums meet in LDS once per group.
template <int D>
__device__ __forceinline__ void load_half_row(const float* __restrict__ base, uint32_t row, uint32_t row_bytes, int lh, float (&f)[D / 2]) {
    const char* src = (const char*)base + (row * row_bytes + (uint32_t)lh * (D / 2 * 4));        // 32-bit offset from the uniform base
#pragma unroll
    for (int i = 0; i < D / 8; ++i) {
        const f32x4 v = *(const f32x4*)(src + i * 16);
#pragma unroll
        for (int e = 0; e < 4; ++e) f[4 * i + e] = v[e];
    }
}

template <int D, int KS>
__global__ void __launch_bounds__(64 * KS) colmass_f32_split_kernel(ScoreParams p) {
    constexpr int HALF = D / 2;
    __shared__ float lds_sum[KS][32];

    int bh, kblk, b, h;
    if (!head_and_block(blockIdx.z * kLayersPerZ + blockIdx.y, p.batch * p.heads, (p.n + 31) / 32, &bh, &kblk)) return;
    split_head(bh, p.batch, p.heads, &b, &h);
    // variable-length batches: queries and keys of this batch element end at its own length
    const int n = p.varlen != nullptr ? p.varlen[b] : p.n;
    if (kblk * 32 >= n) return;             // a block of padding keys: its scores are left untouched
    const int64_t head_off = (int64_t)b * p.td.sb + (int64_t)h * p.td.sh;
    // grouped-query layout: query head h reads K/V head h / (heads / kv_heads)
    const int64_t kv_off = (int64_t)b * p.td_kv.sb + (int64_t)kv_head_of(h, p.heads, p.kv_heads) * p.td_kv.sh;
    const float* __restrict__ Q = (const float*)p.q + head_off;
    const float* __restrict__ K = (const float*)p.k + kv_off;
    const float* __restrict__ lse = p.lse + (int64_t)bh * p.n;
    const uint32_t q_bytes = (uint32_t)p.td.sn * 4u;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lq = lane & 31, lh = lane >> 5;
    const int key = kblk * 32 + lq;
    const int ntiles = (n + QT - 1) / QT;
    const int group_tiles = p.groups > 1 ? p.group_size / QT : ntiles;        // groups are multiples of 128 rows
    const float c2 = p.scale * kLog2e;

    float kf[HALF], qf[HALF];
    typedef f32x4 unaligned_f32x4 __attribute__((aligned(4)));
    f32x4 l2[4];
    // Q rows and log-sum-exp values of tile t; rows past the end read the last one, the caller gives them weight zero
    auto load_tile = [&](int t) {
        const int row = t * QT + lq < n ? t * QT + lq : n - 1;
        load_half_row<D>(Q, (uint32_t)row, q_bytes, lh, qf);
        if (t * QT + QT <= n) {
#pragma unroll
            for (int g = 0; g < 4; ++g) l2[g] = *(const unaligned_f32x4*)(lse + t * QT + 8 * g + 4 * lh);
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = t * QT + acc_row(r, lh);
                l2[r >> 2][r & 3] = lse[row < n ? row : n - 1];
            }
        }
    };
    load_half_row<D>(K, (uint32_t)(key < n ? key : n - 1), (uint32_t)p.td_kv.sn * 4u, lh, kf);
    if (wave < ntiles) load_tile(wave);

    const int groups = (ntiles + group_tiles - 1) / group_tiles;
    for (int u = 0; u < groups; ++u) {
        const int first = u * group_tiles, last = first + group_tiles < ntiles ? first + group_tiles : ntiles;
        float acc_short[4] = {0.f, 0.f, 0.f, 0.f}, acc_long[4] = {0.f, 0.f, 0.f, 0.f};
        int done = 0;
        for (int t = first + wave; t < last; t += KS) {
            f32x16 s;
#pragma unroll
            for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
            for (int kk = 0; kk < HALF; ++kk) s = mfma_f32(qf[kk], kf[kk], s);
            f32x4 l2_now[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) l2_now[g] = l2[g];
            // this wave's next tile: in this group, or its first one of the next
            const int next = t + KS < last ? t + KS : last + wave;
            if (next < ntiles) load_tile(next);
            const int valid = n - t * QT;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float e = exp2f(__builtin_fmaf(s[r], c2, -l2_now[r >> 2][r & 3]));
                acc_short[r & 3] += acc_row(r, lh) < valid ? e : 0.f;
            }
            if (++done == FLUSH) {
                done = 0;
#pragma unroll
                for (int c = 0; c < 4; ++c) { acc_long[c] += acc_short[c]; acc_short[c] = 0.f; }
            }
        }
        const float sum = half_sum(((acc_long[0] + acc_short[0]) + (acc_long[1] + acc_short[1])) +
                                   ((acc_long[2] + acc_short[2]) + (acc_long[3] + acc_short[3])));
        if (lh == 0) lds_sum[wave][lq] = sum;
        __syncthreads();
        if (wave == 0 && lh == 0 && key < n) {
            float all = lds_sum[0][lq];
#pragma unroll
            for (int w = 1; w < KS; ++w) all += lds_sum[w][lq];
            const int rows = (last * QT < n ? last * QT : n) - first * QT;
            p.scores[((int64_t)bh * p.groups + u) * p.n + key] = all * (1.0f / (float)rows);
        }
        __syncthreads();
    }
}

template <int D>
hipError_t launch(const ScoreParams& p, hipStream_t s) {
    const int64_t heads = (int64_t)p.batch * p.heads;
    // Where workgroups of 128 keys leave CUs idle; eight waves to share the tiles where every CU has room for all 32-key
    // workgroups at once.  Both scoring passes, before / after: 2 heads of 256, D = 64, 36.6 / 14.3 us; 8 of 1500,
    // D = 128, 249 / 130 (in groups of 128 280 / 148); 15 of 2048, D = 128, just below the line, 334 / 323.
    const int64_t blocks = (int64_t)((p.n + 31) / 32) * heads;
    if ((int64_t)((p.n + KEYS_PER_WG - 1) / KEYS_PER_WG) * heads < (int64_t)compute_units()) {
        if (blocks <= compute_units()) hipLaunchKernelGGL((colmass_f32_split_kernel<D, 8>), head_grid(heads, (p.n + 31) / 32), dim3(512), 0, s, p);
        else hipLaunchKernelGGL((colmass_f32_split_kernel<D, 4>), head_grid(heads, (p.n + 31) / 32), dim3(256), 0, s, p);
        return hipGetLastError();
    }
    const int nkb = (p.n + KEYS_PER_WG - 1) / KEYS_PER_WG;
    const int bh_pad = (p.batch * p.heads + 7) / 8 * 8;
    hipLaunchKernelGGL((colmass_f32_kernel<D>), dim3(nkb * bh_pad), dim3(NTHREADS), 0, s, p);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_colmass_f32(const ScoreParams& p, int head_dim, hipStream_t s) {
    if (head_dim == 128) return launch<128>(p, s);
    if (head_dim == 64) return launch<64>(p, s);
    return hipErrorInvalidValue;
}

}  // namespace pulsecol
