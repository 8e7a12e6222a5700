// A stand-in for the HIP runtime and the kernels, so that the host engine
// (included whole, after this) runs on the CPU: device memory is host memory,
// copies are done at once, streams and events are logged, and the launchers
// hand their arguments to hooks that a scenario sets.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <functional>
#include <mutex>
#include <string>
#include <vector>

#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "amq_internal.h"

namespace fake {

constexpr int kCus = 256;
std::recursive_mutex mu;
std::vector<std::string> log;          // stream and event calls, in order
intptr_t next_handle = 0x1000;

inline void note(const char *what, const void *a, const void *b)
{
    char buf[96];
    snprintf(buf, sizeof buf, "%s %p %p", what, a, b);
    std::lock_guard<std::recursive_mutex> lk(mu);
    log.push_back(buf);
}
template <typename H> hipError_t handle(H *out)
{
    std::lock_guard<std::recursive_mutex> lk(mu);
    *out = (H)(next_handle += 16);
    return hipSuccess;
}

inline hipError_t get_device(int *d) { *d = 0; return hipSuccess; }
inline hipError_t set_device(int) { return hipSuccess; }
inline hipError_t device_attribute(int *v, hipDeviceAttribute_t a, int)
{
    *v = a == hipDeviceAttributeMultiprocessorCount ? kCus : 1;
    return hipSuccess;
}
template <typename P> hipError_t alloc(P **p, size_t n) { return (*p = (P *)aligned_alloc(256, (n + 255) / 256 * 256)) ? hipSuccess : hipErrorOutOfMemory; }
template <typename P> hipError_t host_alloc(P **p, size_t n, unsigned) { return alloc(p, n); }
inline hipError_t release(void *p) { free(p); return hipSuccess; }
inline hipError_t copy(void *d, const void *s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
inline hipError_t copy_async(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
inline hipError_t stream_create(hipStream_t *s, unsigned) { return handle(s); }
inline hipError_t stream_destroy(hipStream_t) { return hipSuccess; }
inline hipError_t stream_wait_event(hipStream_t s, hipEvent_t e, unsigned) { note("wait", s, e); return hipSuccess; }
hipStream_t capturing = nullptr;       // the stream under capture
inline hipError_t stream_capturing(hipStream_t s, hipStreamCaptureStatus *c)
{
    *c = s == capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
inline hipError_t stream_sync(hipStream_t) { return hipSuccess; }
inline hipError_t event_create(hipEvent_t *e) { return handle(e); }
inline hipError_t event_create_flags(hipEvent_t *e, unsigned) { return handle(e); }
inline hipError_t event_destroy(hipEvent_t) { return hipSuccess; }
inline hipError_t event_record(hipEvent_t e, hipStream_t s) { note("record", s, e); return hipSuccess; }
inline hipError_t event_ok(hipEvent_t) { return hipSuccess; }
inline hipError_t event_elapsed(float *ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
inline hipError_t begin_capture(hipStream_t s, hipStreamCaptureMode) { capturing = s; return hipSuccess; }
inline hipError_t end_capture(hipStream_t, hipGraph_t *g) { capturing = nullptr; return handle(g); }
inline hipError_t graph_instantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t) { return handle(x); }
inline hipError_t graph_launch(hipGraphExec_t x, hipStream_t s) { note("graph", s, x); return hipSuccess; }
inline hipError_t graph_destroy(hipGraph_t) { return hipSuccess; }
inline hipError_t graph_exec_destroy(hipGraphExec_t) { return hipSuccess; }
inline hipError_t symbol_address(void **p, const void *) { return alloc(p, 1); }

// what the batch launchers were given
std::function<void(const amq::BatchOpt *, const int32_t *, const amq::BatchGlobal &, int grid, int mode)> on_sweep_batch;
std::function<void(const amq::GenUnit *, int n, int max_seg_len)> on_generate_batch;
std::function<void(const amq::SweepArgs &)> on_sweep;
int small_groups_per_cu = 1, batch_groups_per_cu = 2, batch_sure_per_cu = 1;

}  // namespace fake

// direction numbers: copied to the "device", never evaluated
extern "C" const uint32_t amq_sobol_v32[amq::kMaxDates * 32] = {0};
extern "C" const uint32_t amq_sobol_v32_dims = amq::kMaxDates;

namespace amq {
hipError_t launch_generate(const GenArgs &a, int, hipStream_t)
{
    memset(a.sync, 0, kSyncWords * 4);
    return hipSuccess;
}
hipError_t preload_generate() { return hipSuccess; }
hipError_t launch_sweep(const SweepArgs &a, int, int, int, hipStream_t s)
{
    fake::note("sweep", s, nullptr);
    if (fake::on_sweep) fake::on_sweep(a);
    return hipSuccess;
}
int sweep_blocks_per_cu(int, int, int wg, int ppt, int) { return wg == 512 && ppt > 8 ? 1 : fake::small_groups_per_cu; }
hipError_t launch_paper(const PaperArgs &, int, hipStream_t) { return hipSuccess; }
hipError_t launch_generate_batch(const BatchOpt *, const GenUnit *u, int n, const uint32_t *, uint32_t *gsync, int max_seg_len,
                                 int, bool, hipStream_t)
{
    memset(gsync, 0, 64);
    if (fake::on_generate_batch) fake::on_generate_batch(u, n, max_seg_len);
    return hipSuccess;
}
hipError_t launch_sweep_batch(const BatchOpt *o, const int32_t *tile_opt, const BatchGlobal &g, int grid, int mode, int, int, bool,
                              hipStream_t s)
{
    fake::note("sweep", s, nullptr);
    if (fake::on_sweep_batch) fake::on_sweep_batch(o, tile_opt, g, grid, mode);
    return hipSuccess;
}
int sweep_batch_blocks_per_cu(int mode, int, int, int) { return mode & kAnyPlacement ? fake::batch_sure_per_cu : fake::batch_groups_per_cu; }
}  // namespace amq

#define hipGetDevice fake::get_device
#define hipSetDevice fake::set_device
#define hipDeviceGetAttribute fake::device_attribute
#define hipMalloc fake::alloc
#define hipHostMalloc fake::host_alloc
#define hipFree fake::release
#define hipHostFree fake::release
#define hipMemcpy fake::copy
#define hipMemcpyAsync fake::copy_async
#define hipStreamCreateWithFlags fake::stream_create
#define hipStreamDestroy fake::stream_destroy
#define hipStreamWaitEvent fake::stream_wait_event
#define hipStreamIsCapturing fake::stream_capturing
#define hipStreamSynchronize fake::stream_sync
#define hipEventCreate fake::event_create
#define hipEventCreateWithFlags fake::event_create_flags
#define hipEventDestroy fake::event_destroy
#define hipEventRecord fake::event_record
#define hipEventQuery fake::event_ok
#define hipEventSynchronize fake::event_ok
#define hipEventElapsedTime fake::event_elapsed
#define hipStreamBeginCapture fake::begin_capture
#define hipStreamEndCapture fake::end_capture
#define hipGraphInstantiate fake::graph_instantiate
#define hipGraphLaunch fake::graph_launch
#define hipGraphDestroy fake::graph_destroy
#define hipGraphExecDestroy fake::graph_exec_destroy
#define hipGetSymbolAddress fake::symbol_address
