// host_plan.cpp -- the library's host code with the HIP runtime and the kernel
// launches replaced: a compute device of 256 compute units and 160 KB of LDS
// that runs nothing, and launches that are recorded.  tests/test_plan.py
// builds it with dtr_sim.cpp and dtr_log.cpp into a library of its own and
// reads what a batch would have launched.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>
#include <cstring>
#include <vector>

#include "layout.h"
#include "layout_log.h"

struct PlanLaunch {
    int64_t group;           // -1: operator logs
    // (logs: sweep_chunks says whether any log is swept)
    int64_t sims, slots, slot_bytes, waves, sweep_chunks, small_n, lds_static, lds_dynamic;
    int64_t stream;          // 0: the caller's
    int64_t small_at;        // where the state words and stacks start in the dynamic LDS
};
static std::vector<PlanLaunch> launches;
static std::atomic<int64_t> streams, destroyed;     // so far
static hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
static std::vector<uint8_t> scratch(DTR_STATIC_SCRATCH_BYTES + 256);

extern "C" {

hipError_t hipGetDevice(int *dev) { *dev = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int)
{
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : a == hipDeviceAttributeMaxSharedMemoryPerBlock ? 160 << 10 : 0;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *to, const void *from, size_t n, hipMemcpyKind, hipStream_t)
{
    std::memcpy(to, from, n);
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)(uintptr_t)(int64_t)++streams; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { destroyed++; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *st) { *st = capturing; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = (hipEvent_t)(uintptr_t)64; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "no device"; }

hipError_t dtr_static_scratch(void **p, size_t *bytes)
{
    *p = (void *)(((uintptr_t)scratch.data() + 255) / 256 * 256);
    *bytes = DTR_STATIC_SCRATCH_BYTES;
    return hipSuccess;
}
hipError_t dtr_launch_reset(uint32_t *, hipStream_t) { return hipSuccess; }
hipError_t dtr_launch_group(const dtr::KernelArgs *a, int32_t group, hipStream_t st)
{
    launches.push_back({group, a->n_sims, a->n_slots, a->L.bytes, a->L.walk_waves, a->sweep_chunks,
                        a->small_n, dtr::static_lds_bytes(group),
                        dtr::dynamic_lds_bytes(group, a->sweep_chunks, a->L.walk_waves, a->small_n),
                        (int64_t)(uintptr_t)st, dtr::dynamic_lds_bytes(group, a->sweep_chunks, a->L.walk_waves, 0)});
    return hipSuccess;
}
hipError_t dtr_launch_log(const dtr::LogKernelArgs *a, hipStream_t)
{
    int64_t sweeps = 0;
    for (int32_t i = 0; i < a->n_sims; i++) sweeps |= a->progs[a->specs[i].trace].sweep;
    launches.push_back({-1, a->n_sims, a->n_slots, a->L.bytes, a->waves, sweeps, 0, 0, a->lds_bytes, 0, 0});
    return hipSuccess;
}

// streams created and destroyed so far, and what every stream says of captures
void plan_streams(int64_t *out) { out[0] = streams; out[1] = destroyed; }
void plan_capture(int32_t on) { capturing = on ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone; }

// the launches since the last call, at most max of them
int32_t plan_launches(PlanLaunch *out, int32_t max)
{
    const int32_t n = (int32_t)launches.size() < max ? (int32_t)launches.size() : max;
    for (int32_t i = 0; i < n; i++) out[i] = launches[i];
    launches.clear();
    return n;
}

}  // extern "C"
