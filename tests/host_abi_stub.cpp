// A GPU that is host memory, for tests of the order and the bookkeeping of abi.hip's launches on the CPU: the HIP calls it
// makes and the launchers it calls, each as little as the test needs.  Linked against abi.hip's host code.
#include <stdlib.h>
#include <string.h>

#include "common.hpp"

extern "C" {
// what the test sets ...
int stub_fail_preprocess_bwd = 0;   // the next launch of k_preprocess_bwd fails
size_t stub_fail_malloc_of = 0;     // allocations of this size fail (0: none does)
int64_t stub_pairs = 0;             // pairs of every view
int64_t stub_longest = 1;           // its longest list
int stub_queue = 0;                 // words for the host arrive when the stream has been asked this often whether it is done (0: at once)
int stub_never = 0;                 // ... or, of 1: the totals, 2: the loss, 3: an ordering in one launch, never: the stream is done without
// ... and reads: flags found set when k_render_bwd is launched, waits for the whole stream, allocations
// and how many launches went by bands of tiles: counts, placements, splits; how many counts there were
int64_t stub_stale_flags = -1;
int stub_syncs = 0, stub_mallocs = 0;
int stub_bands[3] = {0, 0, 0};
int stub_counts = 0;
// and orderings in one launch: their first launches, their second ones
int stub_small[2] = {0, 0};
// and forward and backward passes with a record of blended pairs
int stub_blends[2] = {0, 0};

hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipMalloc(void** p, size_t bytes)
{
    stub_mallocs++;
    if (bytes == stub_fail_malloc_of) return hipErrorOutOfMemory;
    *p = malloc(bytes);
    memset(*p, 1, bytes);   // (fresh device memory holds anything)
    return hipSuccess;
}
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t bytes, unsigned) { *p = calloc(1, bytes); return hipSuccess; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemset(void* p, int v, size_t bytes) { memset(p, v, bytes); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t bytes, hipMemcpyKind, hipStream_t) { memcpy(d, s, bytes); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { stub_syncs++; return hipSuccess; }
static struct { uint64_t* at; uint64_t value; } late[8];
static int late_count = 0, asked = 0;
hipError_t hipStreamQuery(hipStream_t)
{
    if (late_count == 0) return hipSuccess;
    if (++asked < stub_queue) return hipErrorNotReady;
    for (int k = 0; k < late_count; k++) *late[k].at = late[k].value;
    late_count = 0;
    return hipErrorNotReady;   // (what is enqueued behind them still runs)
}
hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.f; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* s) { *p = const_cast<void*>(s); return hipSuccess; }
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
}

namespace fs {

// a kernel's words for the host
static void words(int of, uint64_t* dst, const uint64_t* src, int count)
{
    if (stub_never == of) return;
    asked = 0;
    for (int k = 0; k < count; k++) {
        if (stub_queue) late[late_count++] = {dst + k, src[k]};
        else dst[k] = src[k];
    }
}

size_t scan_tmp_bytes(int64_t) { return 64; }
int photo_blocks(int, int) { return 1; }
int mask_partials() { return 1; }
AdamArgs adam_args(float, float, float, float, int, float) { return {}; }
int tile_sort_variants(int64_t, bool, int) { return 1; }

hipError_t launch_fill_u32(hipStream_t, uint32_t* p, uint32_t v, int64_t n)
{
    for (int64_t i = 0; i < n; i++) p[i] = v;
    return hipSuccess;
}
hipError_t launch_preprocess(hipStream_t, int64_t, int, const fs_gaussians&, bool, const CamDev&, const CfgDev&, const fs_projected&)
{
    return hipSuccess;
}
hipError_t launch_tile_count(hipStream_t, int64_t, const fs_projected&, const CfgDev&, int, int, uint32_t*, uint32_t*, uint2*, uint32_t*,
                             uint64_t* totals, uint32_t*, uint32_t*, uint64_t*, float*, bool bands)
{
    stub_bands[0] += bands;
    stub_counts++;
    const uint64_t pairs = (uint64_t)stub_pairs, four[4] = {pairs, pairs, pairs, (uint64_t)stub_longest};
    words(1, totals, four, 4);
    return hipSuccess;
}
hipError_t launch_small_frame(hipStream_t, int64_t, const fs_projected&, const CfgDev&, int, int, uint32_t, uint32_t*, uint32_t, uint2*,
                              uint32_t*, uint64_t* totals, uint32_t*, uint32_t*, float*, uint64_t*, uint64_t*, uint32_t*)
{
    const uint64_t pairs = (uint64_t)stub_pairs, four[4] = {pairs, pairs, pairs, (uint64_t)stub_longest};
    stub_small[totals == nullptr]++;
    if (totals && stub_never != 3) words(1, totals, four, 4);
    return hipSuccess;
}
hipError_t launch_tile_scatter(hipStream_t, int64_t, const fs_projected&, const CfgDev&, int, int, uint32_t, const uint2*, uint32_t*,
                               uint64_t*, const BandPlaces& places)
{
    stub_bands[1] += places.band != nullptr;
    return hipSuccess;
}
hipError_t launch_tile_sorts(hipStream_t, int, int variants, uint32_t, const uint2*, const uint32_t*, uint64_t*, uint64_t*, uint32_t*,
                             const BandPlaces&)
{
    stub_bands[2] += (variants & TS_SPLIT) != 0;
    return hipSuccess;
}
hipError_t launch_exclusive_scan(hipStream_t, const uint32_t*, uint32_t*, int64_t, void*, uint64_t*) { return hipSuccess; }
hipError_t launch_emit_pairs(hipStream_t, int64_t, const fs_projected&, const CfgDev&, const uint32_t*, int, uint64_t*, uint32_t*, float*)
{
    return hipSuccess;
}
hipError_t launch_radix_sort(hipStream_t, int64_t, int, uint64_t*[2], uint32_t*[2], uint32_t*, void*, uint64_t*, int* result)
{
    *result = 1;
    return hipSuccess;
}
hipError_t launch_tile_ranges(hipStream_t, int64_t, const uint64_t*, int, uint32_t*, uint32_t*) { return hipSuccess; }
hipError_t launch_render_fwd(hipStream_t, const CamDev&, const CfgDev&, const uint32_t*, const uint32_t*, const uint32_t*, const float*,
                             float*, float*, uint32_t*, const ScoreRecord&, const BlendRecord& blends)
{
    stub_blends[0] += blends.entries != nullptr;
    return hipSuccess;
}
hipError_t launch_photo_loss(hipStream_t, const float*, const float*, int, int, float, float*, double*, float*, double* out3)
{
    const double three[3] = {0.25, 0.5, 0.75};
    uint64_t bits[3];
    memcpy(bits, three, sizeof(bits));
    words(2, reinterpret_cast<uint64_t*>(out3), bits, 3);
    return hipSuccess;
}

// every pair's flag is set, as where every pair has received something
hipError_t launch_render_bwd(hipStream_t, const CamDev&, const CfgDev&, const uint32_t*, const uint32_t*, const uint32_t*, const float*,
                             const float*, const uint32_t*, const float*, float*, uint8_t* rec_valid, bool, bool, const BlendRecord& blends)
{
    stub_blends[1] += blends.entries != nullptr;
    if (!rec_valid) return hipSuccess;
    stub_stale_flags = 0;
    for (int64_t i = 0; i < stub_pairs; i++) { stub_stale_flags += rec_valid[i]; rec_valid[i] = 1; }
    return hipSuccess;
}
static hipError_t clear_flags(uint8_t* rec_valid)
{
    if (stub_fail_preprocess_bwd) { stub_fail_preprocess_bwd = 0; return hipErrorUnknown; }
    if (rec_valid) memset(rec_valid, 0, (size_t)stub_pairs);
    return hipSuccess;
}
hipError_t launch_preprocess_bwd(hipStream_t, int64_t, int, const fs_gaussians&, const CamDev&, const CfgDev&, const uint8_t*, const uint32_t*,
                                 const uint32_t*, const uint32_t*, const float*, uint8_t* rec_valid, const fs_grads&)
{
    return clear_flags(rec_valid);
}
hipError_t launch_preprocess_bwd_train(hipStream_t, int64_t, int, const fs_gaussians&, const CamDev&, const CfgDev&, const uint8_t*,
                                       const uint32_t*, const uint32_t*, const uint32_t*, const float*, uint8_t* rec_valid, BwdOut,
                                       const TrainDev&)
{
    return clear_flags(rec_valid);
}

}  // namespace fs
