/*
 * dsr_static.hip -- the library's fixed device workspace, for callers that
 * cannot allocate device memory (code under HIP graph capture, tight
 * serving loops, harnesses that forbid hipMalloc).
 *
 * `scratch` is a file-scope device array of DSR_STATIC_SCRATCH_BYTES that
 * every GPU the library runs on holds until the process ends.  In host code
 * its name is only a host-side stand-in, so nothing here passes it to a
 * kernel or a copy: the device address is looked up once per device, with
 * that device current, through hipGetSymbolAddress, and every use goes
 * through the address kept for that device.  Calls that overlap on one GPU
 * share the array and race; the entry point that uses it says so.
 *
 * It starts out zero, and its first bytes are the result block of every
 * launch that uses it.  Each launch leaves the block's counters at zero for the
 * next one, unless another ran beside it; then they may hold anything, and no
 * later launch may rely on them.  Launches of one stream follow one another, so
 * while one stream alone has used the workspace none has to clear the counters
 * first.  From the first launch of another stream on (or one recorded into a
 * graph, whose replays may run at any time), every launch clears them: nothing
 * tells here when a launch of the other stream, which should have ended by then,
 * does end.  64 teams, per launch in a row of them: 7.6 us without the clearing
 * kernel, 9.5 us with it, 9.1 us in a graph.  One launch in 256 of the one stream clears as well: a
 * new stream may have the handle of one that was destroyed with work left.
 */
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "dsr.h"
#include "dsr_internal.h"

static __device__ __align__(256) uint8_t scratch[DSR_STATIC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
uint8_t *g_ptr[kMaxDevices];
bool g_have[kMaxDevices];

/* The streams that have used a device's workspace. */
struct users {
    void *stream;
    bool several;
    uint32_t calls;
};
users g_users[kMaxDevices];
std::mutex g_users_lock;

__global__ void clear_words(uint32_t *p, uint32_t words)
{
    for (uint32_t k = blockIdx.x * blockDim.x + threadIdx.x; k < words; k += gridDim.x * blockDim.x) p[k] = 0;
}

}  // namespace

/* The workspace's device address on `device` (looked up with the device
 * current, the first time, then kept). */
extern "C" int dsr_static_workspace(int device, uint8_t **out)
{
    if (!out || device < 0 || device >= kMaxDevices) return DSR_E_INVAL;
    *out = nullptr;
    if (!g_have[device]) {
        int prev = 0;
        if (hipGetDevice(&prev) != hipSuccess) return DSR_E_HIP;
        if (hipSetDevice(device) != hipSuccess) return DSR_E_HIP;
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        (void)hipSetDevice(prev);
        if (e != hipSuccess || !p) return DSR_E_HIP;
        g_ptr[device] = (uint8_t *)p;
        g_have[device] = true;
    }
    *out = g_ptr[device];
    return DSR_OK;
}

extern "C" int dsr_static_counters_open(int device, void *stream, int captured)
{
    const std::lock_guard<std::mutex> hold(g_users_lock);
    users &u = g_users[device];
    /* (a per-thread stream has the same handle in every thread) */
    if (captured || stream == (void *)hipStreamPerThread || (u.calls && stream != u.stream)) u.several = true;
    u.stream = stream;
    return u.calls++ % 256u == 0 || u.several;
}

extern "C" int dsr_static_clear(void *p, uint32_t words, void *stream)
{
    hipLaunchKernelGGL(clear_words, dim3((words + 255u) / 256u), dim3(256), 0, (hipStream_t)stream, (uint32_t *)p,
                       words);
    return hipGetLastError() == hipSuccess ? DSR_OK : DSR_E_HIP;
}
