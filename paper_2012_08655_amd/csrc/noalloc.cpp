// Forward foveation without any allocation: up to kArgFrames frames, whose
// descriptors travel in the kernel arguments, so the launch needs no device
// memory of the library's own.  Same kernel as foveate_forward, so outputs are
// bitwise the same.
#include <hip/hip_runtime.h>

#include <string>

#include "host.h"

using namespace fov;

namespace {
// Largest call taken, by the size of its fragment plans (ForwardPlan::plan_bytes).  A 3840x2160 frame in
// 32 px fragments at radius 150 (the widest window a workgroup can stage) needs about 10 MiB.
constexpr size_t kPlanLimit = (size_t)16 << 20;
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
    if (maps_in_outputs(frames, in->n, out->dtype))
        return set_error(FOV_EALIAS, "a sigma map overlaps the output; foveate_forward_noalloc has no memory for a copy of it "
                                     "(use foveate_forward)");
    ForwardPlan fp;
    if ((s = plan_forward(frames, in->n, in->dtype, out->dtype, nullptr, &fp)) != FOV_OK) return s;
    if (fp.plan_bytes > kPlanLimit)
        return set_error(FOV_EINVAL, "this call needs " + std::to_string(fp.plan_bytes) +
                                         " bytes of plan workspace; foveate_forward_noalloc takes calls of up to " +
                                         std::to_string(kPlanLimit) + " (use foveate_forward)");
    return launch_planned(frames, in->n, in->dtype, out->dtype, fp, nullptr, (hipStream_t)stream, false);
}
