// Stand-ins of the HIP runtime and of the kernel launchers behind csrc/pulsecol_api.hip: two devices with different
// numbers of compute units.  The launchers compare what a pass would touch with the allocations it was given; the
// 256-row attention kernel looks at its counters and leaves them as a launch does that has used them up.  What
// is launched on a stream under capture runs when the capture is replayed.
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <vector>

#include "pulsecol_kernels.h"

namespace {
int current = 0;
const int kUnits[2] = {64, 256};
std::map<char*, size_t> blocks;
int row_splits = 0, outside = 0, length_stores = 0, stale = 0, scheduled = 0, fail_after = -1, waits = 0;
bool capturing = false;
std::vector<std::function<void()>> graph;

hipError_t run(std::function<void()> kernel) {
    if (fail_after == 0) return hipErrorInvalidValue;
    if (fail_after > 0) --fail_after;
    if (capturing) graph.push_back(kernel); else kernel();
    return hipSuccess;
}

// counts accesses [p, p + bytes) that no allocation holds
void touch(const void* p, size_t bytes) {
    char* c = (char*)p;
    auto it = blocks.upper_bound(c);
    if (it == blocks.begin()) { ++outside; return; }
    --it;
    if (c + bytes > it->first + it->second) ++outside;
}
}  // namespace

hipError_t hipMalloc(void** p, size_t bytes) {
    *p = std::malloc(bytes);
    std::memset(*p, 0xA5, bytes);
    blocks[(char*)*p] = bytes;
    return hipSuccess;
}
hipError_t hipFree(void* p) { blocks.erase((char*)p); std::free(p); return hipSuccess; }
hipError_t hipMemset(void* p, int value, size_t bytes) { ++waits; std::memset(p, value, bytes); return hipSuccess; }
hipError_t hipMemcpyAsync(void* to, const void* from, size_t bytes, hipMemcpyKind, hipStream_t) { std::memcpy(to, from, bytes); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { ++waits; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* status) {
    *status = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = current; return hipSuccess; }
hipError_t hipSetDevice(int d) { current = d; return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 2; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* symbol) { *p = (void*)symbol; return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }

extern "C" {
int fake_row_splits() { return row_splits; }
int fake_outside() { return outside; }
int fake_device() { return current; }
int fake_stale() { return stale; }
int fake_waits() { return waits; }            // host waits, and work on the default stream
int fake_scheduled() { return scheduled; }
void fake_fail_after(int launches) { fail_after = launches; }
void fake_capture(int on) { capturing = on != 0; if (on) graph.clear(); }
void fake_replay() { for (auto& kernel : graph) kernel(); }
int fake_length_stores() { return length_stores; }
void fake_set_device(int d) { current = d; }
int fake_splits(int blocks, int longest, int head_dim, int units) { return pulsecol::score_splits(blocks, longest, head_dim, units); }
int fake_segments(int n) { return pulsecol::ScoreSegments(n).count; }
int fake_first_tile(int n, int i) { return pulsecol::ScoreSegments(n).first_tile(i); }
int fake_first_of_run(int n, int r, int runs) { return pulsecol::ScoreSegments(n).first_of_run(r, pulsecol::run_reciprocal(runs)); }
}

namespace pulsecol {
int compute_units() { return kUnits[current]; }
hipError_t launch_rowlse_bf16(const ScoreParams& p, int, hipStream_t) {
    const size_t rows = (size_t)p.batch * p.heads * p.n;
    row_splits = p.row_splits;
    touch(p.lse, rows * 4);
    if (p.row_splits > 1) touch(p.part, 2 * (size_t)ScoreSegments(p.n).count * rows * 4);
    return hipSuccess;
}
hipError_t launch_colmass_bf16(const ScoreParams& p, int, hipStream_t) {
    const size_t rows = (size_t)p.batch * p.heads * p.n;
    if (p.col_splits > 1 && p.groups == 1) touch(p.part, (size_t)ScoreSegments(p.n).count * rows * 4);
    return hipSuccess;
}
hipError_t launch_colmass_f32(const ScoreParams&, int, hipStream_t) { return hipSuccess; }
hipError_t launch_attn_bf16(const AttnParams& p, int, AttnMode, hipStream_t) {
    touch(p.work, kWorkWords * 4);
    if (p.work_next) touch(p.work_next, kWorkWords * 4);
    return run([=] {
        ++scheduled;
        for (int i = 0; i < kWorkCounters; ++i) stale += p.work[i * kWorkStride] != 0;
        for (int i = 0; i < kWorkCounters; ++i) p.work[i * kWorkStride] += 1000;
        for (int i = 0; i < kWorkCounters; ++i) if (p.work_next) p.work_next[i * kWorkStride] = 0;
    });
}
hipError_t launch_work_clear(uint32_t* work, int sets, hipStream_t) {
    touch(work, (size_t)sets * kWorkWords * 4);
    return run([=] { for (int i = 0; i < sets * kWorkCounters; ++i) work[i * kWorkStride] = 0; });
}
hipError_t launch_attn_bf16_group(const AttnParams&, int, int, hipStream_t) { return hipSuccess; }
hipError_t launch_attn_f32(const AttnParams&, int, AttnMode, hipStream_t) { return hipSuccess; }
hipError_t launch_topk(const TopkParams&, hipStream_t) { return hipSuccess; }
hipError_t launch_block_sums(const float*, float*, int32_t, int32_t, int64_t, int32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_index_range_check(const int32_t*, int64_t, int32_t, int32_t*, const int32_t*, int32_t, int64_t, int32_t, hipStream_t) { return hipSuccess; }
hipError_t launch_varlen_store(int32_t* varlen, int32_t first, int32_t count, const VarlenChunk&, hipStream_t) {
    ++length_stores;
    touch(varlen + first, (size_t)count * 4);
    return hipSuccess;
}
hipError_t launch_varlen_kept_from_idx(int32_t*, int32_t, const int32_t*, int64_t, int32_t, hipStream_t) { return hipSuccess; }
}  // namespace pulsecol
