// rsr_eval_unknown_noalloc: Stage-2 evaluation with its scratch memory (the
// list of unclassified samples) in a file-scope device array
// instead of the context's workspace, so the call never allocates.
//
// `scratch` exists once per device that loads the library and lives until
// the process ends.  Host code never passes the array's name to a kernel (on
// the host it is only a stand-in symbol): each device's address is looked up
// once with hipGetSymbolAddress, with that device current, when the first
// context on the device is created, and every kernel argument uses that
// address.
#include <mutex>

#include "rsr_internal.h"

namespace rsr {
namespace {

// A SampleList: the regions' extents (two u32 each) followed by up to
// kNoAllocMaxSamples sample indices.
constexpr size_t kScratchWords = 2 * kListRegions + static_cast<size_t>(kNoAllocMaxSamples);

__device__ __align__(256) uint32_t scratch[kScratchWords];

std::mutex g_lock;
void* g_addr[RSR_MAX_DEVICES] = {};

}  // namespace

hipError_t noalloc_scratch(int device, void** out) {
    *out = nullptr;
    if (device < 0 || device >= RSR_MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_lock);
    if (!g_addr[device]) {
        int prev = -1;
        hipError_t e = hipGetDevice(&prev);
        if (e != hipSuccess) return e;
        if (prev != device && (e = hipSetDevice(device)) != hipSuccess) return e;
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (prev != device) (void)hipSetDevice(prev);
        if (e != hipSuccess) return e;
        g_addr[device] = p;
    }
    *out = g_addr[device];
    return hipSuccess;
}

}  // namespace rsr

extern "C" rsr_status rsr_eval_unknown_noalloc(rsr_ctx* ctx, const rsr_system* sys,
                                               const uint32_t* d_samples, int64_t N,
                                               const uint8_t* d_flags, int32_t which,
                                               uint8_t* d_Y, uint64_t* d_n_evaluated) {
    if (!ctx) return RSR_EINVAL;
    if (!sys || !d_samples || !d_Y) return rsr::set_error(ctx, RSR_EINVAL, "NULL argument");
    if (N <= 0) return rsr::set_error(ctx, RSR_EINVAL, "N must be > 0");
    if (N > rsr::kNoAllocMaxSamples)
        return rsr::set_error(ctx, RSR_EINVAL,
                              "N exceeds the scratch of rsr_eval_unknown_noalloc (2^22 samples)");
    if (which != RSR_UNKNOWN_ONLY && which != RSR_ALL)
        return rsr::set_error(ctx, RSR_EINVAL, "bad which");
    if (which == RSR_UNKNOWN_ONLY && !d_flags)
        return rsr::set_error(ctx, RSR_EINVAL, "d_flags is NULL with RSR_UNKNOWN_ONLY");
    if (sys->kind == RSR_SYS_HOST_CALLBACK)
        return rsr::set_error(ctx, RSR_EUNSUPPORTED,
                              "host-callback systems stage samples in allocated memory");
    if (!ctx->noalloc_scratch)
        return rsr::set_error(ctx, RSR_EHIP, "no scratch address for this device");
    int prev = -1;
    if (hipGetDevice(&prev) != hipSuccess) return rsr::set_error(ctx, RSR_EHIP, "hipGetDevice");
    if (prev != ctx->device && hipSetDevice(ctx->device) != hipSuccess)
        return rsr::set_error(ctx, RSR_EHIP, "hipSetDevice");
    const rsr::SampleList list(ctx->noalloc_scratch);
    const rsr::SegSrc seg = rsr::single_src(d_samples, N, const_cast<uint8_t*>(d_flags), d_Y);
    hipError_t e = hipSuccess;
    if (which == RSR_UNKNOWN_ONLY) e = rsr::launch_label(ctx->stream, seg, list);
    if (e == hipSuccess)
        e = rsr::launch_eval(ctx->stream, sys, seg, list, which, d_n_evaluated, ctx->cu_count);
    if (prev != ctx->device) (void)hipSetDevice(prev);
    if (e != hipSuccess) return rsr::hip_error(ctx, e, "rsr_eval_unknown_noalloc launch");
    return RSR_OK;
}
