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
 * launch that uses it: each launch leaves the block's counters at zero for the
 * next one, so none has to clear them first.
 */
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dsr.h"
#include "dsr_internal.h"

static __device__ __align__(256) uint8_t scratch[DSR_STATIC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
uint8_t *g_ptr[kMaxDevices];
bool g_have[kMaxDevices];

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
