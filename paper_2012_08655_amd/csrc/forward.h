// Launch interface of the forward kernels.
#pragma once

#include "common.h"

namespace fov {

// One frame of a forward launch: where it lives, its shape and parameters.
struct FrameDesc {
    const void* in;  // first element of this frame's input
    void* out;       // first element of this frame's output
    int64_t isc, ish, isw, osc, osh, osw;  // element strides
    int32_t c, h, w, nby;
    FrameParams p;  // p.nbx filled in
    // The order of its fragments (order.h): on each axis, how many lines lie farther from the fixation than all
    // lines on its other side (of the frame, or with merge of the rectangle low_*).
    int32_t ahead_x, ahead_y;
    // With merge: the pairs that may not be merged, columns low_x .. low_x + low_w - 1 and rows low_y .. low_y + low_h - 1
    // (whole pairs).
    int32_t low_x, low_y, low_w, low_h;
};

// Frames whose descriptors travel inside the kernel arguments; larger
// batches pass a device table instead.
constexpr int kArgFrames = 16;

// Kernel arguments of the forward and adjoint kernels.  Fragments of all
// frames are numbered consecutively: frame f owns fragments
// [prefix[f], prefix[f+1]).  Work item i of the forward belongs to fragment
// i >> (2 split_log2) of the launch order (see decode() in forward.hip).
// With merge a frame's numbers are those of its pairs, and one more for each pair that may not be merged.
struct FwdLaunch {
    int32_t nframes, nfrag;
    int32_t nitems;      // work items of the forward
    int32_t split_log2;  // each fragment is cut into (2^split_log2)^2 work items (output tiles of
                         // ceil(B / 2^split_log2) pixels a side); 0 = one item per fragment
    int32_t r_cap;       // largest radius the LDS allocation was sized for
    int32_t strip_rows;  // padded-tile rows staged in LDS at once
    int32_t from_args;   // 1: fr[]/kprefix[] hold the frames; 0: table/prefix were uploaded
    int32_t chan;        // 1: one work item per fragment and channel (cmax per fragment), so that
                         // small, latency-bound launches run their channels side by side;
                         // split_log2 must be 0
    int32_t cmax;        // largest channel count of the frames
    int32_t even;        // 1: every frame has the same number of fragments (items take the frames in
                         // turn)
    int32_t merge;       // 1: fragments of rows 2k and 2k + 1 whose sigmas both equal the cap are filtered
                         // as one rectangle (equal taps, so the halo rows they share are computed
                         // once); split_log2 must be 0
    int32_t fp32;        // 1: 8-bit output on the FP32 kernel whatever the radius (see forward_fixed())
    FrameDesc* table;    // device table of nframes entries (read by the main kernel)
    int32_t* prefix;     // device array of nframes+1 entries
    const int32_t* hdr;  // optional device header (BatchHeader): when set, the kernels read the
                         // counts, the split and merge there and the fields above are capacities (a launch
                         // sequence that can be captured once and replayed for many batches; the
                         // replayer sets the main kernel's grid to the batch's item count)
    int32_t kprefix[kArgFrames + 1];
    FrameDesc fr[kArgFrames];
};
static_assert(sizeof(FwdLaunch) <= 4000, "kernel arguments must fit the kernarg segment");

// Device header of a replayable batch (see FwdLaunch::hdr).
struct BatchHeader {
    int32_t nframes, merge, nitems, split_log2;
};

// The forward kernel of one launch.  persist selects its dispatch: a persistent
// grid striding over the work items, or one workgroup per item handed out by
// the hardware dispatcher.
// ev_start/ev_stop, when not null, are recorded on `stream` right before and
// right after the main kernel.
fov_status launch_forward(const FwdLaunch& a, int in_dtype, int out_dtype, size_t lds, hipStream_t stream,
                          size_t lds_limit, int cus, bool persist,
                          hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);

// The main forward kernel of a batch table launched one workgroup per item, for
// a dtype pair (to find its node in a captured graph); NULL for an unsupported
// pair.
const void* forward_main_kernel(int in_dtype, int out_dtype, int r_cap, bool fp32 = false);

// Whether launches of this dtype pair with radii up to r_cap run on the matrix
// cores (8-bit output; see fixed.h).
bool forward_fixed(int in_dtype, int out_dtype, int r_cap);

// Whether that kernel reads this frame byte by byte (interleaved channels other than three, spaced columns).
bool forward_fixed_bytewise(const FrameDesc& d);

// Whether that kernel can store this frame's output, whose rows may lie far apart (it forms
// a tile's offsets in 32 bits).
bool forward_fixed_reaches(const FrameDesc& d);

// Whether fragments of this side are split into a work item per tile there.  Each tile is staged and
// filtered by itself, so an item for each costs nothing more and fills the chip sooner.
bool forward_tiled(int in_dtype, int out_dtype, int r_cap, int block);
// Fragments of a call up to which that is done: a launch holds fewer than 2^32 threads, and there are four items each.
constexpr int64_t kTiledMax = (((int64_t)1 << 32) / kThreads - 1) / 4;

// Device plan for foveate_plan(): sigma and radius of every fragment.
fov_status launch_plan(const FrameParams& fp, int nblk, double* sigma_out, int32_t* r_out, hipStream_t stream);

// LDS bytes a forward workgroup needs for radius r_cap and output tiles of
// tile_w x tile_h pixels (the fragment side B divided by the split, rounded
// up; tile_h = 2B when vertical pairs are merged).
size_t forward_lds_bytes(int in_dtype, int out_dtype, int r_cap, int tile_w, int tile_h, int strip_rows, bool fp32 = false);

// Padded-tile rows of a tile tile_h pixels tall at radius r (what a strip
// height above it cannot change).
int forward_tile_rows(int r, int tile_h);

// Workgroups of the main kernel (one workgroup per work item) that one CU
// holds at once with `lds` bytes of dynamic LDS each.
int forward_occupancy(int in_dtype, int out_dtype, int r_cap, size_t lds, bool fp32 = false);

// Largest strip height the kernel stages at once.
int forward_strip_max();

// Let `kern` use all the dynamic LDS a workgroup may have on the current
// device (done once per device and kernel; safe to call from any thread).
fov_status allow_dyn_lds(const void* kern, size_t lds_limit);

// Workgroups of kThreads threads with `lds` bytes of dynamic LDS each that
// one CU of the current device holds at once; cached per device, kernel and
// size (safe from any thread); 0 if the query fails.
int occupancy_of(const void* kern, size_t lds);

}  // namespace fov
