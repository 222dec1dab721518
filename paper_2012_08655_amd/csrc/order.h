// The order of a launch's fragments: where the k-th item of a frame lies (device) and how many items there are
// (host).  Integer arithmetic and the ramp alone, for host and device alike.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdlib>

#include "forward.h"

namespace fov {

struct Place {
    int bx, by;
};

// What a frame's order is worked out from.
struct Grid {
    int nbx, nby, ahead, low_lines, low_at, low_span;
};
__host__ __device__ inline Grid grid_of(const FrameDesc& d) {
    return Grid{d.p.nbx, d.nby, d.ahead, d.low_lines, d.low_at, d.low_span};
}

// The line-th of n lines: the first `ahead` of them in order (ahead < 0: the last -ahead of them from the end), then the
// rest from both ends in turn.  (Any ahead in -n .. n visits every line once.)
__host__ __device__ inline int line_at(int line, int ahead, int n) {
    // (masks, not branches: this is in the way of an item's first load)
    const int back = ahead >> 31, a = (ahead ^ back) - back, m = line - a, half = m >> 1;
    const int odd = -(m & 1), first = m >> 31;
    const int turn = ((a + half) & odd) | ((n - 1 - half) & ~odd);
    const int pos = (line & first) | (turn & ~first);
    return (pos ^ back) + (n & back);  // n - 1 - pos if ahead < 0
}

// The rank-th fragment of a frame, the costliest lines first (sigma grows with the distance from the fixation).
__host__ __device__ inline Place ranked_place(const Grid& g, int rank) {
    const bool cols = g.nbx >= g.nby;
    const int n1 = cols ? g.nbx : g.nby, n2 = cols ? g.nby : g.nbx;  // lines, fragments in each
    const int line = rank / n2, at = rank - line * n2, pos = line_at(line, g.ahead, n1);
    return cols ? Place{pos, at} : Place{at, pos};
}

// The same for pairs of fragments (rows 2k and 2k + 1; by of a lower one may lie a row below the frame).  Outside the
// last low_lines lines' low_span pairs every pair is merged and its upper fragment stands for it; these pairs come
// first.  Then the others, both fragments of a pair one after the other; which one first is the parity of the bits of
// its place, as the lower item of those that are merged is empty: where every second item was, the compute units
// to which the dispatcher gives every second workgroup had no work.  Kernels' times, with an empty item for every
// merged pair in brackets: u8 to float, 3 x 2160 x 3840, 32 px, radii up to 48 277 us (474), 100 1190 (2260); 3 x 1080 x 1920, 16 px,
// radii up to 60 296 us (511).
__host__ __device__ inline Place paired_place(const Grid& g, int rank) {
    const int rows = (g.nby + 1) >> 1;
    const bool cols = g.nbx >= g.nby;
    const int n1 = cols ? g.nbx : rows, n2 = cols ? rows : g.nbx;
    const int first = n1 - g.low_lines, span = g.low_span, beside = n2 - span;
    const int head = first * n2, box = head + g.low_lines * beside;
    // (selections, not branches: this is in the way of an item's first load)
    const int start = rank < head ? 0 : (rank < box ? head : box), per = rank < head ? n2 : (rank < box ? beside : 2 * span);
    const int num = rank - start, q = num / per, m = num - q * per;
    const int line = rank < head ? q : q + first, k = g.low_at + (m >> 1);
    const int lower = rank < box ? 0 : (m ^ __builtin_popcount((unsigned)(k ^ line))) & 1;
    const int at = rank >= box ? k : (rank >= head && m >= g.low_at ? m + span : m);
    const int pos = line_at(line, cols ? g.ahead : g.ahead / 2, n1);
    return cols ? Place{pos, 2 * at + lower} : Place{at, 2 * pos + lower};
}

// FrameDesc::ahead of a frame: how many more lines lie on one side of the fixation than on the other.
inline int lines_ahead(const FrameDesc& d) {
    const bool cols = d.p.nbx >= d.nby;
    const int n = cols ? d.p.nbx : d.nby;
    const double v = 2.0 * ((cols ? d.p.fix_x - d.p.origin_x : d.p.fix_y - d.p.origin_y) + 0.5) / d.p.block - n;
    return (int)std::min(std::max(v, (double)-n), (double)n);
}

// Where a frame's pairs of fragments (rows 2k and 2k + 1) may not be merged: columns x0 .. x1 - 1 of the rows of pairs
// y0 .. y1 - 1.  A pair is not merged if one of the two lies nearer to the fixation than where the ramp reaches the
// cap; the margin is far above the rounding of that distance, as a pair outside has no item for its lower fragment.
// Any of them if sigmas come from a map, or the cap is 0 (such fragments are copied one by one).
struct PairBox {
    int x0, x1, y0, y1;
};
inline PairBox unmerged_pairs(const FrameDesc& d) {
    const FrameParams& p = d.p;
    const int rows = d.nby / 2;
    PairBox b{0, p.nbx, 0, rows};
    const double reach = p.e0 + p.cap / p.slope;
    const double lim = reach + 1.0 + 1e-9 * (std::fabs(reach) + std::fabs(p.e0) + std::fabs(p.fix_x) + std::fabs(p.fix_y));
    if (p.sigma_map || !(p.cap > 0.0) || !std::isfinite(lim)) return b;
    // fragments lo .. hi - 1 of an axis of n: all with midpoints within lim of the fixation
    const auto within = [&](double fix, int origin, int n, int* lo, int* hi) {
        const double mid0 = origin + (p.block - 1) / 2.0, B = p.block;
        *lo = (int)std::min(std::max(std::floor((fix - lim - mid0) / B), 0.0), (double)n);
        *hi = (int)std::min(std::max(std::ceil((fix + lim - mid0) / B) + 1.0, 0.0), (double)n);
        *hi = lim < 0.0 ? *lo : std::max(*lo, *hi);
    };
    within(p.fix_x, p.origin_x, p.nbx, &b.x0, &b.x1);
    within(p.fix_y, p.origin_y, d.nby, &b.y0, &b.y1);
    b.y0 = std::min(b.y0 / 2, rows);
    b.y1 = std::min((b.y1 + 1) / 2, rows);
    return b;
}

// low_* of a frame: the last lines in its order that hold all of those pairs.
inline void set_low(FrameDesc* d) {
    const PairBox b = unmerged_pairs(*d);
    const bool cols = d->p.nbx >= d->nby, back = d->ahead < 0;
    const int n = cols ? d->p.nbx : (d->nby + 1) / 2, ahead = std::abs(cols ? d->ahead : d->ahead / 2);
    int lo = cols ? b.x0 : b.y0, hi = cols ? b.x1 : b.y1;
    if (back) {
        std::swap(lo, hi);
        lo = n - lo;
        hi = n - hi;
    }
    d->low_at = cols ? b.y0 : b.x0;
    d->low_span = std::max((cols ? b.y1 : b.x1) - d->low_at, 0);
    d->low_lines = 0;
    if (hi <= lo || d->low_span == 0) {
        d->low_span = 0;
        return;
    }
    // of the lines from `ahead` on, m leave a window that starts m / 2 lines from one end and stops (m + 1) / 2 from the
    // other
    if (lo < ahead) d->low_lines = n - lo;
    else d->low_lines = n - ahead - std::min(std::min(2 * (lo - ahead) + 1, 2 * (n - hi)), n - ahead);
}

// Whether merging pairs pays in a launch of `items` fragments (or fragments and channels) without it, `slots` of
// which the chip holds at once: where it holds them all, a pair's item is only a longer one; and where few
// pairs are merged, finding an item's place costs more (0.3 us an item).  Kernels' times without / with pairs, slots = 1024: u8 to
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

// Numbers the items of a launch's frames (see FwdLaunch) in prefix[0 .. nf], and with merge sets the frames'
// low_*; returns their count.
inline int64_t number_items(FrameDesc* frames, int nf, bool merge, int32_t* prefix) {
    bool alike = merge;  // frames of one grid get equal counts, so that they can take turns
    int lines = 0, span = 0;
    for (int i = 0; i < nf && merge; ++i) {
        set_low(&frames[i]);
        alike &= frames[i].p.nbx == frames[0].p.nbx && frames[i].nby == frames[0].nby;
        lines = std::max(lines, frames[i].low_lines);
        span = std::max(span, frames[i].low_span);
    }
    int64_t total = 0;
    for (int i = 0; i < nf; ++i) {
        FrameDesc& d = frames[i];
        prefix[i] = (int32_t)total;
        if (!merge) {
            total += (int64_t)d.p.nbx * d.nby;
            continue;
        }
        const int rows = (d.nby + 1) / 2, n2 = d.p.nbx >= d.nby ? rows : d.p.nbx;
        if (alike) {
            d.low_lines = lines;
            d.low_span = span;
            d.low_at = std::min(d.low_at, n2 - span);
        }
        total += (int64_t)d.p.nbx * rows + (int64_t)d.low_lines * d.low_span;
    }
    prefix[nf] = (int32_t)total;
    return total;
}

}  // namespace fov
