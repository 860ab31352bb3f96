// Variable-length batches: a padded batch whose elements have their own sequence lengths.
// The kernels read two words per batch element from a small device array, varlen[2 * batch]:
// the element's length (rows 0 .. len-1 of its slabs are real, the rest is padding) and `kept`, the
// number of leading entries of its column sets that count.  The kernels here maintain that array
// without any host-to-device copy: lengths travel inside the launch arguments, and `kept` is read off
// the column sets themselves (whose unused tail is filled with -1).
#include "pulsecol_kernels.h"

namespace pulsecol {
namespace {

__global__ void varlen_store_kernel(int32_t* __restrict__ varlen, int32_t first, int32_t count, VarlenChunk values) {
    const int i = threadIdx.x;
    if (i < count) varlen[first + i] = values.v[i];
}

__global__ void varlen_kept_from_idx_kernel(int32_t* __restrict__ varlen, int32_t batch, const int32_t* __restrict__ idx,
                                            int64_t per_batch, int32_t k) {
    const int b = blockIdx.x, lane = threadIdx.x;          // a wave per batch element
    const int32_t* row = idx + (int64_t)b * per_batch;
    const int len = varlen[b];
    const int most = k < len ? k : len;
    // valid entries come first, the padding (-1) behind them: the first negative entry, 64 evenly spaced ones looked at at a time
    // (each look is a trip to memory: 450 entries take two instead of nine by halving; select and attention of four elements of up to 3000 rows
    // 102.0 -> 101.0 us, little more than two runs of one side differ)
    int lo = 0, hi = most;                       // the answer lies in [lo, hi]
    while (lo < hi) {
        const int step = (hi - lo + 63) >> 6, at = lo + lane * step;
        const uint64_t padding = __ballot(at >= hi || row[at] < 0);
        const int valid = padding != 0ull ? __builtin_ctzll(padding) : 64;          // leading ones among those looked at
        const int end = lo + valid * step;
        if (valid == 0) break;                   // (the first entry, or one behind a valid one)
        lo = end - step + 1;
        hi = end < hi ? end : hi;
    }
    if (lane == 0) varlen[batch + b] = lo < 1 ? 1 : lo;         // at least one column (an all-padding row is the caller's error; keep the kernels in bounds)
}

}  // namespace

hipError_t launch_varlen_store(int32_t* varlen, int32_t first, int32_t count, const VarlenChunk& values, hipStream_t s) {
    if (count < 1 || count > 64) return hipErrorInvalidValue;
    hipLaunchKernelGGL(varlen_store_kernel, dim3(1), dim3(64), 0, s, varlen, first, count, values);
    return hipGetLastError();
}

hipError_t launch_varlen_kept_from_idx(int32_t* varlen, int32_t batch, const int32_t* idx, int64_t per_batch, int32_t k,
                                       hipStream_t s) {
    hipLaunchKernelGGL(varlen_kept_from_idx_kernel, dim3(batch), dim3(64), 0, s, varlen, batch, idx, per_batch, k);
    return hipGetLastError();
}

}  // namespace pulsecol
