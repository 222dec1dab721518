// Forward foveation without any allocation: up to kArgFrames frames, whose
// descriptors travel in the kernel arguments, so the launch needs no device
// memory of the library's own.  Same kernel as foveate_forward, so outputs are
// bitwise the same.  Sigma maps that lie in the output are read from copies in a
// fixed array that the code object holds.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <string>

#include "host.h"

using namespace fov;

namespace {
// Largest call taken, by the size that its fragments' plans (radius, taps and queue slots of every fragment) and its
// frame table would have written out, as an earlier form of the launch did: programs rely on the refusal as on the
// rest.  A 3840x2160 frame in 32 px fragments at radius 150 (the widest window a workgroup can stage) comes to about 10 MiB.
constexpr size_t kPlanLimit = (size_t)16 << 20;

size_t plan_bytes(const ForwardPlan& fp, int in_dtype) {
    const auto up = [](size_t v, size_t m) { return (v + m - 1) / m * m; };
    const FwdLaunch& a = fp.a;
    const size_t nfrag = a.nfrag, pad = 8 * (size_t)std::min(a.r_cap + 1, 1024);
    const bool by_channel = fp.cfg.chan_split != 0 && fp.cfg.split_log2 == 0 && a.cmax > 1 && a.cmax <= 16 && nfrag < ((size_t)1 << 26);
    const size_t slots = by_channel ? a.cmax * (nfrag + pad) : (nfrag << (2 * fp.cfg.split_log2)) + pad;
    const size_t taps = nfrag * up(2 * (size_t)a.r_cap + 1, 16) * (in_dtype == FOV_F64 ? 8 : 4);
    return up(2 * up(nfrag * 4, 16) + up(slots * 8, 16) + 256 + taps, 256) + up(148 * (size_t)a.nframes + 4, 256);
}

// Entries that the copies of a call's maps may have: a fragment counts at least 80 bytes of kPlanLimit.
constexpr size_t kMapEntries = (size_t)1 << 18;
static_assert(kMapEntries >= kPlanLimit / 80, "a call within the limit has room for its maps");
static __device__ __align__(256) float g_maps[kMapEntries];  // one array per device

// Who uses the array: calls of a device take turns, by an event that each records behind its kernel and the
// next one's stream waits for.  (Not under capture, where replays can't: they must not overlap.)
constexpr int kMaxDevices = 64;
struct MapTurns {
    std::mutex mu;
    float* at = nullptr;
    hipEvent_t last = nullptr;
};
MapTurns g_turns[kMaxDevices];

fov_status launch_with_copies(FrameDesc* frames, int nf, const fov_tensor& in, const fov_tensor& out, ForwardPlan& fp,
                              hipStream_t stream) {
    size_t entries = 0;
    for (int i = 0; i < nf; ++i) entries += frames[i].p.sigma_map ? (size_t)frames[i].p.nbx * frames[i].nby : 0;
    if (entries > kMapEntries) return set_error(FOV_EINVAL, "too many fragments for copies of the sigma maps");
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_error(e, "hipGetDevice");
    if (dev < 0 || dev >= kMaxDevices) return set_error(FOV_EINVAL, "device index beyond 63");
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    e = hipStreamIsCapturing(stream, &capture);
    if (e != hipSuccess) return hip_error(e, "hipStreamIsCapturing");
    const bool live = capture == hipStreamCaptureStatusNone;
    MapTurns& t = g_turns[dev];
    std::lock_guard<std::mutex> hold(t.mu);
    if (!t.at) {
        void* at = nullptr;
        e = hipGetSymbolAddress(&at, HIP_SYMBOL(g_maps));
        if (e != hipSuccess) return hip_error(e, "hipGetSymbolAddress(g_maps)");
        t.at = static_cast<float*>(at);
    }
    if (live) {
        e = t.last ? hipStreamWaitEvent(stream, t.last, 0) : hipEventCreateWithFlags(&t.last, hipEventDisableTiming);
        if (e != hipSuccess) return hip_error(e, "event of the sigma maps' array");
    }
    float* to = t.at;
    for (int i = 0; i < nf; ++i) {
        if (!frames[i].p.sigma_map) continue;
        const size_t n = (size_t)frames[i].p.nbx * frames[i].nby;
        e = hipMemcpyAsync(to, frames[i].p.sigma_map, n * sizeof(float), hipMemcpyDeviceToDevice, stream);
        if (e != hipSuccess) return hip_error(e, "hipMemcpyAsync(sigma map)");
        frames[i].p.sigma_map = to;
        to += n;
    }
    const fov_status s = launch_planned(frames, nf, in.dtype, out.dtype, fp, nullptr, stream, false);
    if (s != FOV_OK || !live) return s;
    e = hipEventRecord(t.last, stream);
    return e == hipSuccess ? FOV_OK : hip_error(e, "hipEventRecord(sigma maps' array)");
}
}  // namespace

extern "C" fov_status foveate_forward_noalloc(const fov_tensor* in, const fov_tensor* out, const fov_params* p,
                                              int32_t np, void* stream) {
    bool empty = false;
    fov_status s = prepare(in, out, p, np, false, &empty);
    if (s != FOV_OK || empty) return s;
    if (in->n > kArgFrames)
        return set_error(FOV_EINVAL, "foveate_forward_noalloc takes at most " + std::to_string(kArgFrames) +
                                         " frames per call (their descriptors travel in the kernel arguments)");
    FrameDesc frames[kArgFrames];
    for (int i = 0; i < in->n; ++i) frames[i] = make_frame_desc(*in, *out, i, p[np == 1 ? 0 : i]);
    ForwardPlan fp;
    if ((s = plan_forward(frames, in->n, in->dtype, out->dtype, nullptr, &fp)) != FOV_OK) return s;
    const size_t size = plan_bytes(fp, in->dtype);
    if (size > kPlanLimit)
        return set_error(FOV_EINVAL, "the call is too large: by its size in bytes of plan workspace, " + std::to_string(size) +
                                         ", foveate_forward_noalloc takes up to " + std::to_string(kPlanLimit) +
                                         " (use foveate_forward)");
    if (maps_in_outputs(frames, in->n, out->dtype)) return launch_with_copies(frames, in->n, *in, *out, fp, (hipStream_t)stream);
    return launch_planned(frames, in->n, in->dtype, out->dtype, fp, nullptr, (hipStream_t)stream, false);
}
