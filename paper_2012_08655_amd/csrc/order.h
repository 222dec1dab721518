// The order of a launch's fragments: where the k-th item of a frame lies (device) and how many items there are
// (host).  Integer arithmetic and the ramp alone, for host and device alike.
#pragma once

#include <algorithm>
#include <cmath>

#include "forward.h"

namespace fov {

struct Place {
    int bx, by;
    bool box;  // one of a frame's FrameDesc::low_* fragments
};

// What a frame's order is worked out from.
struct Grid {
    int nbx, nby, ahead_x, ahead_y, low_x, low_y, low_w, low_h;
};
__host__ __device__ inline Grid grid_of(const FrameDesc& d) {
    return Grid{d.p.nbx, d.nby, d.ahead_x, d.ahead_y, d.low_x, d.low_y, d.low_w, d.low_h};
}

// The lines of an axis in an order: the first `ahead` of the n lines (ahead < 0: the last -ahead of them from the end),
// then the rest from both ends in turn.  The line-th of them, and the first of those that are left after `line`
// (they lie side by side).  (Any ahead in -n .. n visits every line once.)
__host__ __device__ inline int line_at(int line, int ahead, int n) {
    const int back = ahead >> 31, a = (ahead ^ back) - back, m = line - a, half = m >> 1;
    const int odd = -(m & 1), first = m >> 31;
    const int turn = ((a + half) & odd) | ((n - 1 - half) & ~odd);
    const int pos = (line & first) | (turn & ~first);
    return (pos ^ back) + (n & back);  // n - 1 - pos if ahead < 0
}
__host__ __device__ inline int left_from(int line, int ahead) {
    const int a = ahead < 0 ? -ahead : ahead, m = line - a;
    if (ahead < 0) return m > 0 ? (m + 1) >> 1 : 0;
    return m > 0 ? a + (m >> 1) : line;
}

struct Cell {
    int u, v;
};

// A square root to within one (the caller makes it exact).
__host__ __device__ inline float root(float x) {
#ifdef __HIP_DEVICE_COMPILE__
    return __builtin_amdgcn_sqrtf(x);
#else
    return std::sqrt(x);
#endif
}

// The rank-th cell of n1 x n2 (n1 >= n2), those far from the fixation on either axis first: lines of the longer axis
// until a square is left, then a line of each axis in turn.  With lines of the longer axis alone, the costly ends of the other
// axis came last; per call, so in brackets: 4 x 3 x 512 x 512 f32, 16 px, radii up to 27 60 us (79), 100 389 (505); u8 to float,
// 3 x 1080 x 1920, 24 px, 48 115 (138); f64, 256 x 256, 4 px, 100 56 (90); u8, 3 x 1080 x 1920, 16 px 39.4 (40.8).
// Where every item costs the same the longer way to a place shows: 32 x 3 x 224 x 224 f32, 32 px, 3 34.4 (33.6).
__host__ __device__ inline Cell shell_at(int n1, int n2, int ahead1, int ahead2, int rank) {
    const int more = n1 - n2, head = more * n2;
    if (rank < head) {
        const int line = rank / n2;
        return Cell{line_at(line, ahead1, n1), rank - line * n2};
    }
    // of the square's n2^2 cells left^2 are left before the line that this one is on: left is the root, rounded up
    const int rest = n2 * n2 - (rank - head);
    int left = (int)root((float)rest);
    left += left * left < rest;
    left -= (left - 1) * (left - 1) >= rest;
    const int done = n2 - left, at = left * left - rest;
    if (at < left) return Cell{line_at(more + done, ahead1, n1), left_from(done, ahead2) + at};
    return Cell{left_from(more + done + 1, ahead1) + at - left, line_at(done, ahead2, n2)};
}

// The rank-th item of a frame, the costliest first (sigma grows with the distance from the fixation).
//
// With pairs (rows 2k and 2k + 1): outside the rectangle low_* every pair is merged and its upper
// fragment stands for it (and for a last row without a pair); these come first, being costliest.  In it each
// fragment has a rank.  Of a pair that is merged there one is empty, the upper or the lower by the parity of the bits of
// its place: where every second item was empty, the compute units to which the dispatcher gives every second workgroup
// had no work.  Per call, with an empty item for every merged pair in brackets: u8 to float, 3 x 2160 x 3840, 32 px, radii up
// to 48 261 us (467), 100 1170 (2250); 3 x 1080 x 1920, 16 px, radii up to 60 283 us (505).
__host__ __device__ inline Place item_place(const Grid& g, int rank, bool pairs) {
    int x0 = 0, y0 = 0, w = g.nbx, h = g.nby;
    if (__builtin_expect(pairs, 0)) {
        const int rows = (g.nby + 1) >> 1, high = g.low_h >> 1;
        const int beside = (g.nbx - g.low_w) * rows, per = rows - high, outside = beside + g.low_w * per;
        if (rank < outside) {
            const bool clear = rank < beside;  // a column that does not meet the rectangle
            const int num = clear ? rank : rank - beside, n = clear ? rows : per;
            const int col = num / n, at = num - col * n;
            return Place{clear ? (col < g.low_x ? col : col + g.low_w) : g.low_x + col, 2 * (clear || 2 * at < g.low_y ? at : at + high),
                         false};
        }
        rank -= outside;
        x0 = g.low_x, y0 = g.low_y, w = g.low_w, h = g.low_h;
    }
    const bool cols = w >= h;
    const Cell c = shell_at(cols ? w : h, cols ? h : w, cols ? g.ahead_x : g.ahead_y, cols ? g.ahead_y : g.ahead_x, rank);
    return Place{x0 + (cols ? c.u : c.v), y0 + (cols ? c.v : c.u), pairs};
}

// The rank-th fragment in the order of memory.
__host__ __device__ inline Place row_place(int nbx, int rank) {
    const int by = rank / nbx;
    return Place{rank - by * nbx, by, false};
}

// Ahead of the others on an axis of n fragments from `origin` on: how many more lie on one side of the fixation than on
// the other.
inline int lines_ahead(double fix, double origin, int block, int n) {
    const double v = 2.0 * (fix - origin + 0.5) / block - n;
    return (int)std::min(std::max(v, (double)-n), (double)n);
}

// low_* of a frame: the pairs of fragments (rows 2k and 2k + 1) that may not be merged.  A pair is not merged if one of
// the two lies nearer to the fixation than where the ramp reaches the
// cap; the margin is far above the rounding of that distance, as a pair outside has no item for its lower fragment.
// Any of them if sigmas come from a map, or the cap is 0 (such fragments are copied one by one).
inline void set_low(FrameDesc* d) {
    const FrameParams& p = d->p;
    int x0 = 0, x1 = p.nbx, y0 = 0, y1 = d->nby;
    const double reach = p.e0 + p.cap / p.slope;
    const double lim = reach + 1.0 + 1e-9 * (std::fabs(reach) + std::fabs(p.e0) + std::fabs(p.fix_x) + std::fabs(p.fix_y));
    if (!p.sigma_map && p.cap > 0.0 && std::isfinite(lim)) {
        // fragments lo .. hi - 1 of an axis of n: all with midpoints within lim of the fixation
        const auto within = [&](double fix, int origin, int n, int* lo, int* hi) {
            const double mid0 = origin + (p.block - 1) / 2.0, B = p.block;
            *lo = (int)std::min(std::max(std::floor((fix - lim - mid0) / B), 0.0), (double)n);
            *hi = (int)std::min(std::max(std::ceil((fix + lim - mid0) / B) + 1.0, 0.0), (double)n);
            *hi = lim < 0.0 ? *lo : std::max(*lo, *hi);
        };
        within(p.fix_x, p.origin_x, p.nbx, &x0, &x1);
        within(p.fix_y, p.origin_y, d->nby, &y0, &y1);
    }
    // whole pairs; none if either side is empty
    const int last = d->nby & ~1;
    d->low_x = x0;
    d->low_y = std::min(y0 & ~1, last);
    d->low_w = x1 - x0;
    d->low_h = std::min((y1 + 1) & ~1, last) - d->low_y;
    if (d->low_w <= 0 || y1 <= y0 || d->low_h <= 0) d->low_w = d->low_h = 0;
}

// Whether merging pairs pays in a launch of `items` fragments (or fragments and channels) without it, `slots` of
// which the chip holds at once: where it holds them all, a pair's item is only a longer one; and where few
// pairs are merged, finding an item's place costs more.  Per call without / with pairs, slots = 1024: u8 to
// float, 256 x 256, 64 items 6.2 / 7.8 us, 1024 items 6.7 / 7.2; 1080 x 1920, radii up to 12, 510 items 13 / 18, 920 15.7 / 17.8, 2040 15.4 / 16.4,
// 3600 24 / 21, 8160 42 / 28; 4 x 3 x 512 x 512 f32, hardly any pairs merged 43 / 44.
inline bool merge_pays(const FrameDesc* frames, int nf, int64_t items, int64_t slots) {
    if (items <= slots) return false;
    double pairs = 0.0, apart = 0.0;  // all; not merged, counted in some of the rows
    for (int i = 0; i < nf; ++i) {
        const FrameDesc& d = frames[i];
        const int rows = d.nby / 2, step = 1 + rows / 16;
        pairs += (double)rows * d.p.nbx;
        if (d.p.sigma_map) continue;  // not known here
        const double reach = d.p.e0 + d.p.cap / d.p.slope, half = (d.p.block - 1) / 2.0, B = d.p.block;
        for (int k = step / 2; k < rows; k += step) {
            const double dy = d.p.origin_y + (2 * k + 1) * B - 0.5 - d.p.fix_y, at = (d.p.fix_x - d.p.origin_x - half) / B;
            const double chord = reach > std::fabs(dy) ? std::sqrt(reach * reach - dy * dy) / B : 0.0;
            const double n = std::min(at + chord, d.p.nbx - 1.0) - std::max(at - chord, 0.0);
            if (!(n <= 0.0)) apart += step * n;  // (all of them if there is no reach)
        }
    }
    return apart < 0.875 * pairs;
}

// Numbers the items of a launch's frames (see FwdLaunch) in prefix[0 .. nf], and sets the frames' ahead_* and, with merge,
// low_*; returns their count.
inline int64_t number_items(FrameDesc* frames, int nf, bool merge, int32_t* prefix) {
    bool alike = merge;  // frames of one grid get equal counts, so that they can take turns
    int w = 0, h = 0;
    for (int i = 0; i < nf && merge; ++i) {
        set_low(&frames[i]);
        alike &= frames[i].p.nbx == frames[0].p.nbx && frames[i].nby == frames[0].nby;
        w = std::max(w, frames[i].low_w);
        h = std::max(h, frames[i].low_h);
    }
    int64_t total = 0;
    for (int i = 0; i < nf; ++i) {
        FrameDesc& d = frames[i];
        const FrameParams& p = d.p;
        prefix[i] = (int32_t)total;
        if (!merge) {
            d.ahead_x = lines_ahead(p.fix_x, p.origin_x, p.block, p.nbx);
            d.ahead_y = lines_ahead(p.fix_y, p.origin_y, p.block, d.nby);
            total += (int64_t)p.nbx * d.nby;
            continue;
        }
        if (alike) {
            d.low_w = w;
            d.low_h = h;
            d.low_x = std::min(d.low_x, p.nbx - w);
            d.low_y = std::min(d.low_y, (d.nby & ~1) - h);
        }
        d.ahead_x = lines_ahead(p.fix_x, p.origin_x + (double)d.low_x * p.block, p.block, d.low_w);
        d.ahead_y = lines_ahead(p.fix_y, p.origin_y + (double)d.low_y * p.block, p.block, d.low_h);
        total += (int64_t)p.nbx * ((d.nby + 1) / 2) + (int64_t)d.low_w * (d.low_h / 2);
    }
    prefix[nf] = (int32_t)total;
    return total;
}

}  // namespace fov
