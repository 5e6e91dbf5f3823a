// Stand-in for the HIP runtime in host tests (test infrastructure): linked with the library's own objects, it takes
// their kernel launches, writes them down and runs nothing, so that what the host code would enqueue can be looked at
// without a GPU -- and a launch can be made to fail.  Built and used by tests/test_launches_host.py.
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "buzz_internal.h"

using namespace buzz;

namespace {

struct Launch {
    std::string kernel;
    dim3 grid, block;
    size_t lds;
    GatherArgs gather;      // of gather_rows_kernel
    ObsArgs obs;            // of the prompt-scoring kernels
};

std::map<const void*, std::string>& names() { static std::map<const void*, std::string> n; return n; }
std::vector<Launch> launches;
int fail_at = -1;                                          // the launch (counted from the last reset) that fails
hipError_t last_error = hipSuccess;
struct { dim3 grid, block; size_t lds; hipStream_t stream; } config;
alignas(256) char symbol_memory[16 << 20];                 // device variables live here

hipError_t note(hipError_t e) { if (e != hipSuccess) last_error = e; return e; }

hipError_t record(const void* fn, dim3 grid, dim3 block, void** args, size_t lds)
{
    if ((int)launches.size() == fail_at) { fail_at = -1; return note(hipErrorLaunchFailure); }
    // what the runtime refuses: an empty grid, more than 2^32 - 1 work-items in one dimension
    const uint64_t x = (uint64_t)grid.x * block.x, y = (uint64_t)grid.y * block.y, z = (uint64_t)grid.z * block.z;
    if (!x || !y || !z || x > UINT32_MAX || y > UINT32_MAX || z > UINT32_MAX || lds > 65536) return note(hipErrorInvalidConfiguration);
    Launch l{};
    l.kernel = names()[fn]; l.grid = grid; l.block = block; l.lds = lds;
    if (l.kernel.find("gather_rows_kernel") != std::string::npos) l.gather = *(const GatherArgs*)args[0];
    if (l.kernel.find("obs_") != std::string::npos) l.obs = *(const ObsArgs*)args[0];
    launches.push_back(l);
    return hipSuccess;
}

}  // namespace

extern "C" {

// ---- what the tests call
void rec_reset(int fail) { launches.clear(); fail_at = fail; last_error = hipSuccess; }
int rec_count() { return (int)launches.size(); }
const char* rec_kernel(int i) { return launches[i].kernel.c_str(); }
long long rec_value(int i, const char* what)
{
    const Launch& l = launches[i];
    const std::string w = what;
    if (w == "grid_x") return l.grid.x;
    if (w == "grid_y") return l.grid.y;
    if (w == "grid_z") return l.grid.z;
    if (w == "block_x") return l.block.x;
    if (w == "lds") return (long long)l.lds;
    if (w == "n_rows") return l.gather.n_rows;
    if (w == "key_parts") return l.obs.key_parts;
    if (w == "key_part_len") return l.obs.key_part_len;
    if (w == "item_parts") return l.obs.item_parts;
    if (w == "item_part_len") return l.obs.item_part_len;
    if (w == "t_begin") return l.obs.t_begin;
    if (w == "t_count") return l.obs.t_count;
    if (w == "heads") return l.obs.heads;
    if (w == "units") return l.obs.units;
    if (w == "stats_cap") return (long long)l.obs.stats_cap;
    if (w == "partial_cap") return (long long)l.obs.partial_cap;
    if (w == "places") return l.obs.place.on;
    return -1;
}

// ---- what the library calls
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* fn, char*, const char* name, unsigned, void*, void*, void*, void*, int*) { names()[fn] = name; }
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t st) { config = {grid, block, lds, st}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* st)
{
    *grid = config.grid; *block = config.block; *lds = config.lds; *st = config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* fn, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t) { return record(fn, grid, block, args, lds); }
hipError_t hipExtLaunchKernel(const void* fn, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t, hipEvent_t, hipEvent_t, int) { return record(fn, grid, block, args, lds); }
hipError_t hipGetLastError() { const hipError_t e = last_error; last_error = hipSuccess; return e; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = kDefaultCUs; return hipSuccess; }
hipError_t hipFuncGetAttributes(hipFuncAttributes* f, const void*) { *f = hipFuncAttributes{}; f->sharedSizeBytes = 8000; return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int block, size_t) { *n = 3 * 256 / block; return hipSuccess; }   // 3 waves per SIMD
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = symbol_memory; return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return hipErrorInvalidValue; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float*, hipEvent_t, hipEvent_t) { return hipErrorInvalidValue; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipErrorInvalidValue; }

}  // extern "C"
