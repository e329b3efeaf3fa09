// host_launch.cpp -- the launch functions of the kernel sources (built for the
// host only) with the HIP runtime replaced by a recorder, for
// tests/test_launch.py: each launch with its kernel, shape, dynamic LDS and
// the kernel's allowance of it at that moment.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <map>
#include <vector>

#include "dtr_sim.h"
#include "layout.h"
#include "layout_log.h"

struct Launch {
    int64_t kernel, grid, block, lds, allowed;
};
static std::vector<Launch> launches;
static std::map<const void *, int64_t> allowed;
static struct { dim3 grid, block; size_t lds; hipStream_t stream; } conf;

extern "C" {

void **__hipRegisterFatBinary(const void *) { static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, void *, void *, int *) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t st) { conf = {g, b, lds, st}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *st)
{
    *g = conf.grid;
    *b = conf.block;
    *lds = conf.lds;
    *st = conf.stream;
    return hipSuccess;
}
hipError_t hipGetDevice(int *dev) { *dev = 0; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **, const void *) { return hipErrorNoDevice; }
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute, int v) { allowed[f] = v; return hipSuccess; }
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t lds, hipStream_t)
{
    const auto it = allowed.find(f);
    launches.push_back({(int64_t)(uintptr_t)f, g.x, b.x, (int64_t)lds, it == allowed.end() ? 64 << 10 : it->second});
    return hipSuccess;
}

hipError_t dtr_launch_group(const dtr::KernelArgs *, int32_t, hipStream_t);
hipError_t dtr_launch_log(const dtr::LogKernelArgs *, hipStream_t);

// one launch of a trace group, or of the log kernel (its reset kernel is left
// out); the kernel's static LDS as the plan counts it is returned in `fixed`
int32_t launch_group(int32_t group, int32_t slots, int32_t waves, int32_t chunks, int32_t small_n, Launch *out, int64_t *fixed)
{
    dtr::KernelArgs a{};
    a.n_sims = a.n_slots = slots;
    a.L.walk_waves = waves;
    a.sweep_chunks = chunks;
    a.small_n = small_n;
    launches.clear();
    if (dtr_launch_group(&a, group, nullptr) != hipSuccess || launches.size() != 1) return -1;
    *out = launches[0];
    *fixed = dtr::static_lds_bytes(group);
    return 0;
}

int32_t launch_log(int32_t slots, int32_t waves, int32_t lds, Launch *out)
{
    dtr::LogKernelArgs a{};
    a.n_sims = a.n_slots = slots;
    a.waves = waves;
    a.lds_bytes = lds;
    launches.clear();
    if (dtr_launch_log(&a, nullptr) != hipSuccess || launches.size() != 2) return -1;
    *out = launches[1];
    return 0;
}

}  // extern "C"
