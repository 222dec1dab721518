// Adjoint of block-wise foveation (the backward pass for training through the
// foveation), as a gather: no atomics, every element written once, a fixed
// summation order.
//
// Restricted to one fragment b, the forward map is separable: a horizontal
// then a vertical 1-D correlation with b's taps w_b over the clamped frame.
// Its transpose maps the fragment's output gradient g_b back over b's window
// (the fragment grown by r_b on every side), so
//     grad_in = sum_b Fold_x H_b^T Fold_y V_b^T g_b,
// where V_b^T / H_b^T correlate with w_b (the taps are symmetric) over the
// window's rows / columns, and Fold adds what lands outside the frame onto
// the edge row or column (the transpose of clamp-to-edge).  On an axis of
// length L the fold gives output 0 the extra weight
// cdf_b(-p-1) = sum_{i <= -p-1} w_b(i) for input p, and output L-1 the extra
// weight cdf_b(p-L).
//
// 32-bit gradients with fragment sides of 16 or 28 .. 32 take the matrix-core gather further below; the
// rest two kernels:
//  1. fov_adj_window_kernel — one workgroup per fragment and channel: the
//     fragment's sigma, radius and normalised taps (kept in LDS), then its
//     transposed window as the forward computes a fragment: the gradient is
//     staged in LDS (column-major, zero rows around it), the vertical
//     transpose writes the window's rows into a second LDS buffer (zero
//     columns around the data), and the horizontal transpose writes the
//     folded window to scratch, column by column (lanes take rows, so the
//     stores of a wave cover consecutive addresses).  It also records each
//     fragment's radius.
//  2. fov_adj_sum_kernel — one workgroup per output tile (the fragment grid)
//     adds up the windows of every fragment that reaches it, in a fixed
//     order (lanes test the candidate fragments, a ballot lists the hits),
//     reading window columns with buffer loads, and stores the tile along
//     rows through an LDS transpose.
// Both transposes are the forward's register-window correlations, run over
// the band of taps that meet the fragment.
#include "adjoint.h"

#include <hip/hip_runtime.h>

#include <algorithm>

#include "conv.h"

namespace fov {

namespace {

constexpr int kPadA = 12;  // zero columns before a window row (horizontal transpose)

// Folded window of fragment F at radius r: frame rows [y0, y1), columns [x0, x1].
struct Window {
    int y0, y1, x0, x1;
};

__device__ __forceinline__ Window window_of(const Frag& F, int r, int h, int w) {
    Window v;
    v.y0 = max(F.ya - r, 0);
    v.y1 = min(F.ya + F.bh + r, h);
    v.x0 = max(F.xa - r, 0);
    v.x1 = min(F.xa + F.bw - 1 + r, w - 1);
    return v;
}

// The fragment's taps in LDS: V copies (V = 16 / sizeof(T)), copy k holding tap i at element
// k * stride + kAdjWeightLead + k + i (stride a multiple of 4) with zeros around, so that a run of
// taps starting at any tap t >= -kAdjWeightLead + 1 starts on a 16-byte boundary in one of them and
// is read with 16-byte loads.
template <typename T>
__device__ __forceinline__ const T* taps_from(const T* taps, int stride, int t) {
    constexpr int V = 16 / sizeof(T);
    const int k = (-t) & (V - 1);
    return static_cast<const T*>(__builtin_assume_aligned(taps + k * stride + kAdjWeightLead + k + t, 16));
}

// Transposed window of fragment gid into scratch[gid][c][x - x0][y - ya + window_lead(r)]
// (column-major, column stride s.sh) for the frame columns x0..x1 and rows y0..y1-1 of its folded
// window: the fragment's own rows start on a 128-byte boundary, and so do those of the tiles above
// and below when the block size is a multiple of 128 bytes of elements.  Workgroup
// q takes fragment q / csplit and its channel share q % csplit (csplit workgroups per fragment).
// GV: gradient values a thread holds per channel (bh * bw <= 256 GV).
template <typename T, int GV, bool ARGS>
__global__ __launch_bounds__(kThreads) void fov_adj_window_kernel(const FwdLaunch a, const AdjShape s,
                                                                  const FrameDesc* __restrict__ table,
                                                                  const int32_t* __restrict__ prefix,
                                                                  int32_t* __restrict__ radius, T* __restrict__ scratch,
                                                                  int csplit) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int V = 16 / sizeof(T);  // elements per aligned 16-byte LDS load
    const int PB = s.pitch_b, PAD = s.pad_b, P = s.pitch_a;
    T* taps = reinterpret_cast<T*>(smem);  // V shifted copies of the taps (taps_from)
    T* G = taps + s.tap_elems;             // [bmax columns][PB rows]: one channel's gradient, rows PAD..
    T* R = G + (size_t)s.bmax * PB;        // [s.rows_r rows][P]: vertical transpose of a run of window
                                           // rows, columns kPadA..
    __shared__ double part_of_wave[kThreads / 64];
    const int gid = blockIdx.x / csplit, share = blockIdx.x - gid * csplit;
    const Frag F = frag_of<ARGS>(a, table, prefix, a.nframes, gid);
    const FrameDesc& d = *F.fd;
    const int per = (s.cmax + csplit - 1) / csplit;
    const int c_begin = share * per, c_end = min(d.c, c_begin + per);
    if (c_begin >= c_end) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_id();
    const global_ptr<const T> g = as_global(static_cast<const T*>(d.in));
    // One channel's gradient in registers, thread values i = tid + 256 k at row i / bmax, column
    // i % bmax (lanes along a row: coalesced reads); the next channel's loads are issued while this
    // channel is transposed.
    constexpr int kGv = GV;
    T gv[kGv];
    int gy[kGv], gx[kGv];  // row and column of each value (-1: none)
#pragma unroll
    for (int k = 0; k < kGv; ++k) {
        const int i = tid + k * kThreads;
        const int py = div_by(i, s.bdiv), x = i - py * s.bmax;
        const bool in = x < F.bw && py < F.bh;
        gy[k] = in ? py : -1;
        gx[k] = x;
    }
    auto load_g = [&](int c) {
#pragma unroll
        for (int k = 0; k < kGv; ++k)
            if (gy[k] >= 0)
                gv[k] = g[(int64_t)c * d.isc + (int64_t)(F.ya + gy[k]) * d.ish + (int64_t)(F.xa + gx[k]) * d.isw];
    };
    load_g(c_begin);
    // Radius and normalised taps of the fragment (its sigma from the midpoint's eccentricity, Sec. 2;
    // Eq. 1 cut at 3 sigma), as the forward's plan computes them.
    const FrameParams& fp = d.p;
    const double sigma = fragment_sigma(fp, F.lb, F.bx, F.by);
    const int r = min(radius_of(sigma), a.r_cap);
    const int N = 2 * r + 1;
    if (share == 0 && tid == 0) radius[gid] = r;  // for the sum kernel
    const double inv = r > 0 ? 1.0 / (2.0 * sigma * sigma) : 0.0;
    double part = 0.0, mine = 0.0;
    for (int j = tid; j < N; j += kThreads) {
        const double k = (double)(j - r);
        const double e = exp(-(k * k) * inv);
        part += e;
        if (j == tid) mine = e;
    }
    for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off, 64);
    if (lane == 0) part_of_wave[wave] = part;
    const Window win = window_of(F, r, d.h, d.w);
    const int RT = win.y1 - win.y0;
    const int CH = s.rows_r;  // window rows transposed per run (a multiple of 4)
    // Zeros: the taps' padding, and the staged gradient and transposed rows (whose data cells every
    // channel and run overwrite).
    for (int k = 0; k < V; ++k)
        for (int j = tid; j < s.tap_stride; j += kThreads) {
            const int t = j - kAdjWeightLead - k;
            if (t < 0 || t >= N) taps[k * s.tap_stride + j] = (T)0;
        }
    {
        using V16 = __attribute__((ext_vector_type(4))) uint32_t;
        V16* z = reinterpret_cast<V16*>(G);
        const int n16 = (s.bmax * PB + min(RT, CH) * P) / V;
        for (int i = tid; i < n16; i += kThreads) z[i] = V16{0, 0, 0, 0};
    }
    __syncthreads();
    part = 0.0;
#pragma unroll
    for (int q = 0; q < kThreads / 64; ++q) part += part_of_wave[q];
    for (int j = tid; j < N; j += kThreads) {
        const double k = (double)(j - r);
        const T v = (T)((j == tid ? mine : exp(-(k * k) * inv)) / part);
#pragma unroll
        for (int c = 0; c < V; ++c) taps[c * s.tap_stride + kAdjWeightLead + c + j] = v;
    }
    const T* __restrict__ w = taps + kAdjWeightLead;  // copy 0, w[i] = tap i (i = t + r)
    T* dst0 = scratch + (size_t)gid * s.cmax * s.sw * s.sh;
    const int G8 = (win.x1 - win.x0 + kPH) / kPH;
    // Barriers: one before each run's vertical transpose (the staged gradient and the taps are
    // visible; the previous run's rows are no longer read) and one after it (the rows are written;
    // the gradient is no longer read, so the next channel may be staged).
    for (int c = c_begin; c < c_end; ++c) {
        // the fragment's gradient, column-major
#pragma unroll
        for (int k = 0; k < kGv; ++k)
            if (gy[k] >= 0) G[gx[k] * PB + PAD + gy[k]] = gv[k];
        if (c + 1 < c_end) load_g(c + 1);
        for (int cr0 = win.y0; cr0 < win.y1; cr0 += CH) {
        const int rows = min(CH, win.y1 - cr0);  // window rows cr0 .. cr0 + rows - 1 in this run
        const int ngroups = (rows + kPV - 1) / kPV;
        const int ntask_v = s.bmax * ngroups;  // task i: column i % bmax, rows cr0 + 4 (i / bmax) .. +3
        __syncthreads();
        // Vertical transpose Fold_y V^T g into R: a wave's 64 tasks share one band of taps (the taps
        // that meet the fragment's rows from some row of the wave).
        for (int i0 = wave * 64; i0 < ntask_v; i0 += kThreads) {
            const int gA = div_by(i0, s.bdiv), gB = min(div_by(i0 + 63, s.bdiv), ngroups - 1);
            const int ymin = cr0 + kPV * gA, ymax = min(cr0 + kPV * gB + kPV - 1, cr0 + rows - 1);
            int t_lo = max(-r, F.ya - ymax);
            const int t_hi = min(r, F.ya + F.bh - 1 - ymin);
            if (t_lo <= t_hi) t_lo -= (cr0 + kPV * gA + t_lo - F.ya + PAD) & (V - 1);  // aligned start
            const int i = i0 + lane;
            const int gr = div_by(i, s.bdiv), x = i - gr * s.bmax;
            if (x >= F.bw || gr >= ngroups) continue;
            const int y0 = cr0 + kPV * gr;
            T acc[kPV];
#pragma unroll
            for (int p = 0; p < kPV; ++p) acc[p] = 0;
            const T* col = G + x * PB + PAD - F.ya;  // col[y]: the gradient at frame row y (zero outside)
            if (t_lo <= t_hi) vconv(acc, col + y0 + t_lo, t_hi - t_lo + 1, taps_from(taps, s.tap_stride, t_lo + r));
            if (y0 == 0) {  // row 0 collects the taps off the top edge
                T cdf = 0, corr = 0;
                for (int m = -r; m <= -F.ya - 1; ++m) {
                    cdf += w[m + r];
                    const int py = -m - 1;
                    if (py < F.ya + F.bh) corr = fma(cdf, col[py], corr);
                }
                acc[0] += corr;
            }
            const int pr = d.h - 1 - y0;  // row h-1 collects those off the bottom edge
            if (pr >= 0 && pr < kPV) {
                T cdf = 0, corr = 0;
                for (int m = -r; m <= -1; ++m) {
                    cdf += w[m + r];
                    const int py = m + d.h;
                    if (py >= F.ya && py < F.ya + F.bh) corr = fma(cdf, col[py], corr);
                }
#pragma unroll
                for (int p = 0; p < kPV; ++p)
                    if (p == pr) acc[p] += corr;
            }
            T* rr = R + (y0 - cr0) * P + kPadA + x;
#pragma unroll
            for (int p = 0; p < kPV; ++p)
                if (y0 + p < cr0 + rows) rr[p * P] = acc[p];
        }
        __syncthreads();
        // Horizontal transpose Fold_x H^T of the window rows into scratch: lanes take rows, a wave
        // shares one group of 8 output columns, so the taps that meet the fragment form one
        // wave-uniform range.
        T* dstc = dst0 + (size_t)c * s.sw * s.sh + (cr0 - F.ya + window_lead(r, (int)sizeof(T)));
        for (int ch = 0; ch * 64 < rows; ++ch)
        for (int gi = wave; gi < G8; gi += kThreads / 64) {
            const int X = win.x0 + gi * kPH;
            // taps t with X + p + t inside the fragment for some p in 0..7
            int t_lo = max(-r, F.xa - X - (kPH - 1));
            const int t_hi = min(r, F.xa + F.bw - 1 - X);
            const int row = ch * 64 + lane;
            if (row >= rows) continue;
            const T* rr = R + row * P + kPadA - F.xa;  // rr[x]: this row at frame column x
            T acc[kPH];
#pragma unroll
            for (int p = 0; p < kPH; ++p) acc[p] = 0;
            if (t_lo <= t_hi) {
                t_lo -= (X + t_lo - F.xa + kPadA) & (V - 1);  // aligned window start; taps below -r are zero
                hconv(acc, rr + X + t_lo, t_hi - t_lo + 1, taps_from(taps, s.tap_stride, t_lo + r));
            }
            if (win.x0 == 0 && gi == 0) {  // column 0 collects the taps that fell off the left edge
                T cdf = 0, corr = 0;
                for (int m = -r; m <= -F.xa - 1; ++m) {
                    cdf += w[m + r];
                    const int x = -m - 1;
                    if (x < F.xa + F.bw) corr = fma(cdf, rr[x], corr);
                }
                acc[0] += corr;
            }
            const int jr = d.w - 1 - X;
            if (win.x1 == d.w - 1 && jr >= 0 && jr < kPH) {  // column w-1 collects those off the right edge
                T cdf = 0, corr = 0;
                for (int m = -r; m <= -1; ++m) {
                    cdf += w[m + r];
                    const int x = m + d.w;
                    if (x >= F.xa && x < F.xa + F.bw) corr = fma(cdf, rr[x], corr);
                }
#pragma unroll
                for (int p = 0; p < kPH; ++p)
                    if (p == jr) acc[p] += corr;
            }
            T* dst = dstc + (size_t)(X - win.x0) * s.sh + row;
#pragma unroll
            for (int p = 0; p < kPH; ++p)
                if (X + p <= win.x1) dst[(size_t)p * s.sh] = acc[p];
        }
        }
    }
}

// Output tile gid: grad_in over the fragment's rectangle, the sum of the windows of every fragment
// that reaches it, in a fixed order (fragment rows, then columns).  Pixel i of the tile is column
// i / bh, row i % bh, so the lanes of a wave read consecutive rows of a window column.  Up to
// kSumCh channels are summed together, and the windows are read kSumBatch at a time, all their loads
// in flight before the values are added in order (PIX: pixels per thread, bh * bw <= 256 PIX).
constexpr int kSumCh = 3;
// Windows in flight per batch, sized so that the loaded values stay within the register budget of
// four waves per SIMD.
template <typename T, int PIX>
constexpr int sum_batch() {
    return PIX * (int)sizeof(T) <= 16 ? 4 : (PIX * (int)sizeof(T) <= 64 ? 2 : 1);
}

struct SumNb {
    int b;      // fragment
    int ybase;  // frame row of the first element of its window columns
    Window w;
};

// Raw buffer descriptor (dword 3 as gfx9 expects for untyped access).
constexpr int kBufferWord3 = 0x00020000;
// Byte offset past any window plane: a buffer load there returns 0.
constexpr uint32_t kOutside = 0x7fffffffu;

template <typename T>
__device__ __forceinline__ T buffer_load(__amdgpu_buffer_rsrc_t rsrc, uint32_t voff) {
    if constexpr (sizeof(T) == 8)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)voff, 0, 0));
    else
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)voff, 0, 0));
}

// The values of window n at this thread's pixels, channels c0 .. c0 + kSumCh - 1 (zero outside the
// window and for channels >= c0 + cc): one buffer descriptor per channel plane of the window, so a
// pixel outside it reads 0 through the descriptor's range check.
template <typename T, int PIX>
__device__ __forceinline__ void load_window(T (&v)[kSumCh][PIX], const SumNb& n, const T* __restrict__ scratch,
                                            const AdjShape& s, int c0, int cc, const int (&px)[PIX],
                                            const int (&py)[PIX]) {
    const uint32_t wx = (uint32_t)(n.w.x1 - n.w.x0), wy = (uint32_t)(n.w.y1 - n.w.y0);
    uint32_t voff[PIX];
#pragma unroll
    for (int k = 0; k < PIX; ++k) {
        const uint32_t dx = (uint32_t)(px[k] - n.w.x0), dy = (uint32_t)(py[k] - n.w.y0);
        voff[k] = (dx <= wx && dy < wy) ? (dx * (uint32_t)s.sh + (uint32_t)(py[k] - n.ybase)) * (uint32_t)sizeof(T)
                                        : kOutside;
    }
    const int plane = s.sw * s.sh;
#pragma unroll
    for (int ch = 0; ch < kSumCh; ++ch) {
        if (ch < cc) {
            const T* src = scratch + ((size_t)n.b * s.cmax + c0 + ch) * plane;
            const __amdgpu_buffer_rsrc_t rsrc =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(src), 0, plane * (int)sizeof(T), kBufferWord3);
#pragma unroll
            for (int k = 0; k < PIX; ++k) v[ch][k] = buffer_load<T>(rsrc, voff[k]);
        } else {
#pragma unroll
            for (int k = 0; k < PIX; ++k) v[ch][k] = (T)0;
        }
    }
}

__device__ __forceinline__ int lane_value(int v, int j) { return __builtin_amdgcn_readlane(v, j); }

template <typename T, int PIX, bool ARGS>
__global__ __launch_bounds__(kThreads) void fov_adj_sum_kernel(const FwdLaunch a, const AdjShape s,
                                                               const FrameDesc* __restrict__ table,
                                                               const int32_t* __restrict__ prefix,
                                                               const int32_t* __restrict__ radius,
                                                               const T* __restrict__ scratch) {
    const int gid = blockIdx.x;
    const Frag Q = frag_of<ARGS>(a, table, prefix, a.nframes, gid);
    const FrameDesc& d = *Q.fd;
    const FrameParams& fp = d.p;
    const int nbx = fp.nbx, nby = d.nby;
    const int first = gid - Q.lb;
    const int K = (a.r_cap + fp.block - 1) / fp.block;  // fragments within reach on each side
    const int by_lo = max(Q.by - K, 0), by_hi = min(Q.by + K, nby - 1);
    const int bx_lo = max(Q.bx - K, 0), bx_hi = min(Q.bx + K, nbx - 1);
    const int nx = bx_hi - bx_lo + 1, ncand = nx * (by_hi - by_lo + 1);
    const float rnx = 1.0f / (float)nx;  // candidate j is row j / nx of the neighbourhood
    const int lane = threadIdx.x & 63;
    const int B = fp.block;
    int px[PIX], py[PIX];  // frame column and row of each pixel (-1: none)
#pragma unroll
    for (int k = 0; k < PIX; ++k) {
        const int i = threadIdx.x + k * kThreads;
        const int col = div_by(i, s.bdiv), row = i - col * s.bmax;
        const bool in = col < Q.bw && row < Q.bh;
        px[k] = in ? Q.xa + col : -1;
        py[k] = in ? Q.ya + row : -1;
    }
    const global_ptr<T> out = as_global(static_cast<T*>(d.out));
    extern __shared__ __align__(16) unsigned char smem[];
    T* tile = reinterpret_cast<T*>(smem);
    const int LP = s.bmax + 1;
    constexpr int kSumBatch = sum_batch<T, PIX>();
    for (int c0 = 0; c0 < d.c; c0 += kSumCh) {
        const int cc = min(kSumCh, d.c - c0);
        T acc[kSumCh][PIX];
#pragma unroll
        for (int ch = 0; ch < kSumCh; ++ch)
#pragma unroll
            for (int k = 0; k < PIX; ++k) acc[ch][k] = 0;
        for (int j0 = 0; j0 < ncand; j0 += 64) {
            // Candidates j0 .. j0 + 63 (row-major over the fragments within reach), one per lane: the
            // ballot of those whose window meets the tile lists them in the fixed summation order.
            const int j = j0 + lane;
            int b = 0, y0 = 0, y1 = 0, x0 = 0, x1 = 0, yb = 0;
            bool hit = false;
            if (j < ncand) {
                const int jy = (int)(((float)j + 0.5f) * rnx);
                const int by = by_lo + jy, bx = bx_lo + (j - jy * nx);
                const int lb = by * nbx + bx;
                b = first + lb;
                const int rb = radius[b];
                // its folded window (as window_of gives it for that fragment)
                const int X0 = fp.origin_x + bx * B, Y0 = fp.origin_y + by * B;
                x0 = max(X0 - rb, 0);
                x1 = min(X0 + B - 1 + rb, d.w - 1);
                y0 = max(Y0 - rb, 0);
                y1 = min(Y0 + B + rb, d.h);
                yb = max(Y0, 0) - window_lead(rb, (int)sizeof(T));
                hit = x1 >= Q.xa && x0 < Q.xa + Q.bw && y1 > Q.ya && y0 < Q.ya + Q.bh;
            }
            uint64_t m = __ballot(hit);
            while (m) {
                // the next kSumBatch of them: all their loads in flight, then added in order
                SumNb nb[kSumBatch];
                int cnt = 0;
#pragma unroll
                for (int q = 0; q < kSumBatch; ++q) {
                    if (m) {
                        const int l = __builtin_ctzll(m);
                        m &= m - 1;
                        nb[q].b = lane_value(b, l);
                        nb[q].ybase = lane_value(yb, l);
                        nb[q].w.y0 = lane_value(y0, l);
                        nb[q].w.y1 = lane_value(y1, l);
                        nb[q].w.x0 = lane_value(x0, l);
                        nb[q].w.x1 = lane_value(x1, l);
                        ++cnt;
                    }
                }
                T v[kSumBatch][kSumCh][PIX];
#pragma unroll
                for (int q = 0; q < kSumBatch; ++q)
                    if (q < cnt) load_window(v[q], nb[q], scratch, s, c0, cc, px, py);
#pragma unroll
                for (int q = 0; q < kSumBatch; ++q)
                    if (q < cnt) {
#pragma unroll
                        for (int ch = 0; ch < kSumCh; ++ch)
#pragma unroll
                            for (int k = 0; k < PIX; ++k) acc[ch][k] += v[q][ch][k];
                    }
            }
        }
        // Through LDS (tile[ch][row][col], pitch bmax + 1) so that the stores run along rows.
        if (c0 > 0) __syncthreads();  // the previous channels' tile is read
#pragma unroll
        for (int ch = 0; ch < kSumCh; ++ch)
#pragma unroll
            for (int k = 0; k < PIX; ++k)
                if (ch < cc && px[k] >= 0) tile[(ch * s.bmax + py[k] - Q.ya) * LP + px[k] - Q.xa] = acc[ch][k];
        __syncthreads();
        int tx = threadIdx.x;
        asm volatile("" : "+v"(tx));  // store addresses computed here, not held through the sums
#pragma unroll
        for (int k = 0; k < PIX; ++k) {
            const int i = tx + k * kThreads;
            const int row = div_by(i, s.bdiv), col = i - row * s.bmax;
            if (row >= Q.bh || col >= Q.bw) continue;
#pragma unroll
            for (int ch = 0; ch < kSumCh; ++ch)
                if (ch < cc)
                    out[(int64_t)(c0 + ch) * d.osc + (int64_t)(Q.ya + row) * d.osh + (int64_t)(Q.xa + col) * d.osw] =
                        tile[(ch * s.bmax + row) * LP + col];
        }
    }
}

// ---- matrix-core gather for 32-bit gradients, fragment sides 16 and 28 .. 32 ----------------------
// grad_in over an output tile is the sum, over the fragments b that reach it, of Ay_b^T g_b Ax_b: two dense
// products of at most 32 x 32 x 32 per channel with Ax_b[c][x] = w_b(x - c) (plus the edge folds), which
// v_mfma_f32_16x16x4_f32 forms in FP32 like the vector units.  Nothing but the gradient and the taps is
// read and nothing but grad_in written: the window and sum kernels move every fragment's transposed window,
// (32 + 2r)^2 values a channel, through scratch and back, and were bound by that.  Measured per call, with the
// window kernels in brackets: 4 x 3 x 512 x 512, radii up to 36, 32 px fragments 57 us (85), 16 px 122 (347);
// 32 x 3 x 224 x 224 55.5 us (73); 3 x 1080 x 1920, radii up to 48 165 us (301).  Of a SIMD's time the matrix
// instructions take 36 %, scalar instructions (a tile's and a hit's set-up, the skips) 40 %, vector ones 29 %; a
// wave waits 40 % of its own.  Slower were: the next hit's loads ahead of this one's products (65 us: a second set of
// addresses and weights costs more than the wait), and one or two waves a tile (67 and 63 us).
//  1. fov_adj_plan_kernel: one wave per fragment: radius, taps and the running sums of the taps.
//  2. fov_adj_gather_kernel: one workgroup per output tile (as many fragments as fit 32 pixels a side) and
//     channel; its waves take the fragments that reach the tile in turn, and their sums meet in LDS in a
//     fixed order.  Steps of the products whose weights are all zero are skipped (16 x 16 results, 16 rows or
//     8 columns of the fragment at a time).

// Taps of fragment gid in `taps`: w(t) at [gid][t + r_cap] for |t| <= r, then C(t) = sum_{i <= t} w(i)
// at [gid][2 r_cap + 1 + t + r_cap] for -r <= t <= -1.
__host__ __device__ inline int adj_tap_stride(int r_cap) { return 3 * r_cap + 1; }

template <bool ARGS>
__global__ __launch_bounds__(64) void fov_adj_plan_kernel(const FwdLaunch a, const FrameDesc* __restrict__ table,
                                                          const int32_t* __restrict__ prefix,
                                                          int32_t* __restrict__ radius, float* __restrict__ taps) {
    const int gid = blockIdx.x, lane = threadIdx.x;
    const Frag F = frag_of<ARGS>(a, table, prefix, a.nframes, gid);
    const double sigma = fragment_sigma(F.fd->p, F.lb, F.bx, F.by);
    const int r = min(radius_of(sigma), a.r_cap);
    if (lane == 0) radius[gid] = r;
    const Taps tp(sigma, r, lane);
    float* w = taps + (size_t)gid * adj_tap_stride(a.r_cap) + a.r_cap;
    float* c = w + 2 * a.r_cap + 1;
    double carry = 0.0;
    for (int q = 0; 64 * q < 2 * r + 1; ++q) {
        const int j = 64 * q + lane;
        const double v = j < 2 * r + 1 ? tp.tap(q, r, lane) : 0.0;
        if (j < 2 * r + 1) w[j - r] = (float)v;
        if (64 * q >= r) continue;  // the sums end at t = -1
        double incl = v;
        for (int off = 1; off < 64; off <<= 1) {
            const double t = __shfl_up(incl, off, 64);
            if (lane >= off) incl += t;
        }
        incl += carry;
        if (j < r) c[j - r] = (float)incl;
        carry = __shfl(incl, 63, 64);
    }
}

constexpr int kGatherTile = 32;
constexpr int kGatherPitch = kGatherTile + 1;  // LDS row pitch of the waves' sums
constexpr int kGatherWaves = 4;                // waves per output tile and channel

// One axis of a fragment and a tile: tile position 0 is at fragment position d; n positions of the tile,
// frag_n of the fragment, radius r.
struct Axis {
    int d, n, frag_n, r;
    bool first, last;  // the tile holds the frame's first, last position

    // The fragment positions that reach the tile's positions 16 k .. 16 k + 15: bit g for those of the g-th
    // group of 2^size.
    __device__ __forceinline__ uint32_t band(int k, int size) const {
        const int lo = max(d + 16 * k - r, 0), hi = min(d + min(16 * k + 15, n - 1) + r, frag_n - 1);
        return 16 * k < n && lo <= hi ? (2u << ((uint32_t)hi >> size)) - (1u << ((uint32_t)lo >> size)) : 0u;
    }
};

__device__ __forceinline__ Axis axis_of(int tile0, int tile_n, int frag0, int frag_n, int r, int len) {
    return Axis{tile0 - frag0, tile_n, frag_n, r, tile0 == 0, tile0 + tile_n == len};
}

// The weights of an axis by t = tile position - fragment position, t + 31 - d in lw: w(t), and for a tile at
// the frame's first or last position the folds onto it.  `lw` is 3 x 64 words of this wave's LDS.  load()
// issues every read at a valid place (both axes' are in flight together), store() drops what is outside.
struct AxisLoads {
    float w, first, last;
    __device__ __forceinline__ void load(const Axis& x, const float* __restrict__ taps, const float* __restrict__ c, int lane) {
        const int t = x.d - 31 + lane, r = x.r;
        w = taps[clampi(t, -r, r)];
        first = last = 0.0f;
        if (r > 0 && x.first) first = c[clampi(t - 1, -r, -1)];
        if (r > 0 && x.last) last = c[clampi(-t - 1, -r, -1)];
    }
    __device__ __forceinline__ void store(const Axis& x, float* lw, int lane) const {
        const int t = x.d - 31 + lane, r = x.r;
        lw[lane] = t >= -r && t <= r ? w : 0.0f;
        if (x.first) lw[64 + lane] = t - 1 >= -r && t <= 0 ? first : 0.0f;
        if (x.last) lw[128 + lane] = t >= 0 && -t - 1 >= -r ? last : 0.0f;
    }
};

// A lane's weights of tile position pos for fragment positions base + at(i), i = 0 .. 7.
template <typename At>
__device__ __forceinline__ void lane_weights(float (&A)[8], const Axis& x, const float* lw, int pos, int base, At at) {
    const float* p = lw + (31 + pos - base - at(7));
#pragma unroll
    for (int i = 0; i < 8; ++i) A[i] = p[at(7) - at(i)];
    if (!x.first && !x.last) return;
    if (x.first && pos == 0) {
#pragma unroll
        for (int i = 0; i < 8; ++i) A[i] += p[64 + at(7) - at(i)];
    }
    if (x.last && pos == x.n - 1) {
#pragma unroll
        for (int i = 0; i < 8; ++i) A[i] += p[128 + at(7) - at(i)];
    }
}

typedef float v4f __attribute__((ext_vector_type(4)));

// A step of v_mfma_f32_16x16x4_f32 takes one fragment position from each quarter h4 of the wave.  Columns
// (first product): step i, 8 (i / 2) + 2 h4 + i % 2.  Rows (second product): step i, 16 (i / 4) + 4 h4 + i % 4,
// the rows in which the first product's result lies.
__device__ __forceinline__ constexpr int gather_col(int i) { return 8 * (i >> 1) + (i & 1); }
__device__ __forceinline__ constexpr int gather_row(int i) { return 16 * (i >> 2) + (i & 3); }

template <bool ARGS>
__global__ __launch_bounds__(64 * kGatherWaves, 4) void fov_adj_gather_kernel(const FwdLaunch a, const FrameDesc* __restrict__ table,
                                                                     const int32_t* __restrict__ prefix,
                                                                     const int32_t* __restrict__ radius,
                                                                     const float* __restrict__ taps) {
    __shared__ float sums[kGatherWaves][kGatherTile * kGatherPitch];
    // The way to a hit's loads runs at a raised wave priority: other waves' products can wait for it (57.6 -> 56.7, 16 px
    // 124.3 -> 121.8 us; the products raised instead, no change).
    __builtin_amdgcn_s_setprio(2);
    const int item = blockIdx.x / a.cmax, ch = blockIdx.x - item * a.cmax;
    int frame, rank;
    ranked_frame<ARGS>(a, prefix, a.nframes, item, &frame, &rank);
    const Frag Q = ranked_at(frame_of<ARGS>(a, table, frame), frame, rank);
    const FrameDesc& d = frame_of<ARGS>(a, table, Q.f);
    const FrameParams& fp = d.p;
    const int B = fp.block, m = B <= kGatherTile / 2 ? 2 : 1;  // fragments per tile side
    if (ch >= d.c || (m == 2 && ((Q.bx | Q.by) & 1))) return;
    const int nbx = fp.nbx, nby = d.nby, first = ARGS ? a.kprefix[Q.f] : prefix[Q.f];
    const int X0 = fp.origin_x + Q.bx * B, Y0 = fp.origin_y + Q.by * B;
    const int tw = min(X0 + m * B, d.w) - Q.xa, th = min(Y0 + m * B, d.h) - Q.ya;
    const int K = (a.r_cap + B - 1) / B;  // fragments within reach on each side
    const int by_lo = max(Q.by - K, 0), by_hi = min(Q.by + m - 1 + K, nby - 1);
    const int bx_lo = max(Q.bx - K, 0), bx_hi = min(Q.bx + m - 1 + K, nbx - 1);
    const int nx = bx_hi - bx_lo + 1, ncand = nx * (by_hi - by_lo + 1);
    const float rnx = 1.0f / (float)nx;
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_id(), l = lane & 15, h4 = lane >> 4;
    float* lx = &sums[wave][0];  // this wave's axis weights; its sums later
    float* ly = lx + 192;
    const int stride = adj_tap_stride(a.r_cap);
    const global_ptr<const float> in = as_global(static_cast<const float*>(d.in)) + (int64_t)ch * d.isc;
    // a fragment's offsets fit 31 bits of bytes
    const bool near = (kGatherTile - 1) * (d.ish + d.isw) < (int64_t)(kOutside / 4);
    v4f acc[2][2];
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i >> 1][i & 1] = v4f{};
    // Each fragment that reaches the tile, in a fixed order; wave v takes hits v, v + kGatherWaves, ...
    const auto for_hits = [&](auto&& f) {
        int turn = 0;
        for (int j0 = 0; j0 < ncand; j0 += 64) {
            const int j = j0 + lane, jy = (int)(((float)j + 0.5f) * rnx);
            const int cy = by_lo + jy, cx = bx_lo + (j - jy * nx);
            int rb = 0;
            bool hit = false;
            if (j < ncand) {
                rb = radius[first + cy * nbx + cx];
                const int x0 = fp.origin_x + cx * B, y0 = fp.origin_y + cy * B;
                hit = x0 + B - 1 + rb >= Q.xa && x0 - rb < Q.xa + tw && y0 + B - 1 + rb >= Q.ya && y0 - rb < Q.ya + th;
            }
            for (uint64_t hits = __ballot(hit); hits; hits &= hits - 1, ++turn) {
                if (turn % kGatherWaves != wave) continue;
                const int src = __builtin_ctzll(hits);
                const int bx = lane_value(cx, src), by = lane_value(cy, src), r = lane_value(rb, src);
                const int xb = max(fp.origin_x + bx * B, 0), yb = max(fp.origin_y + by * B, 0);
                const int bw = min(fp.origin_x + (bx + 1) * B, d.w) - xb, bh = min(fp.origin_y + (by + 1) * B, d.h) - yb;
                const float* w = taps + (size_t)(first + by * nbx + bx) * stride + a.r_cap;
                const Axis ax = axis_of(Q.xa, tw, xb, bw, r, d.w), ay = axis_of(Q.ya, th, yb, bh, r, d.h);
                f(ax, ay, w, w + 2 * a.r_cap + 1, in + (int64_t)yb * d.ish + (int64_t)xb * d.isw);
            }
        }
    };
    for_hits([&](const Axis& ax, const Axis& ay, const float* w, const float* c, global_ptr<const float> gp) {
        // Columns 8 j .. of the fragment that tile columns 0 .. 15 and 16 .. want, and rows 16 k .. that tile rows
        // 0 .. 15 and 16 .. want, as bits j and k: a test of one is two scalar instructions (the scalar unit was
        // busier here than the matrix cores).
        const uint32_t x_0 = ax.band(0, 3), x_1 = ax.band(1, 3), y_0 = ay.band(0, 4), y_1 = ay.band(1, 4);
        __builtin_amdgcn_s_setprio(2);
        AxisLoads wx, wy;
        wx.load(ax, w, c, lane);
        wy.load(ay, w, c, lane);
        // The gradient where it has a weight, zero elsewhere: lane l's rows 16 k + l, columns gather_col().  A place
        // that is not wanted is given an offset that the range check turns into a zero without a read.
        float g[2][8];
        const int x0 = max(ax.d - ax.r, 0), x1 = min(ax.d + tw - 1 + ax.r, ax.frag_n - 1);
        const int y0 = max(ay.d - ay.r, 0), y1 = min(ay.d + th - 1 + ay.r, ay.frag_n - 1);
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float*>((const float*)gp), 0, (int)kOutside, kBufferWord3);
        if (d.isw == 1 && near && !(ax.frag_n & 1)) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int row = 16 * k + l;
                const uint32_t at = ((uint32_t)row * (uint32_t)d.ish + 2 * h4) * 4;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int col = 8 * j + 2 * h4;
                    const bool want = row >= y0 && row <= y1 && col + 1 >= x0 && col <= x1;
                    const auto v = __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)(want ? at + 32 * j : kOutside), 0, 0);
                    g[k][2 * j] = __builtin_bit_cast(float, (uint32_t)v[0]);
                    g[k][2 * j + 1] = __builtin_bit_cast(float, (uint32_t)v[1]);
                }
            }
        } else if (near) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const int row = 16 * k + l;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int col = gather_col(i) + 2 * h4;
                    const bool want = row >= y0 && row <= y1 && col >= x0 && col <= x1;
                    const uint32_t at = ((uint32_t)row * (uint32_t)d.ish + (uint32_t)col * (uint32_t)d.isw) * 4;
                    g[k][i] = buffer_load<float>(rsrc, want ? at : kOutside);
                }
            }
        } else {
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int row = 16 * k + l, col = gather_col(i) + 2 * h4;
                    const bool want = row >= y0 && row <= y1 && col >= x0 && col <= x1;
                    g[k][i] = want ? gp[(int64_t)row * d.ish + (int64_t)col * d.isw] : 0.0f;
                }
        }
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_wave_barrier();
        wx.store(ax, lx, lane);
        wy.store(ay, ly, lane);
        __builtin_amdgcn_wave_barrier();
        float Ax[2][8], Ay[2][8];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            lane_weights(Ax[k], ax, lx, 16 * k + l, 2 * h4, gather_col);
            lane_weights(Ay[k], ay, ly, 16 * k + l, 4 * h4, gather_row);
        }
        // The fragment's part on its own, then added: one chain over all fragments rounds more (rms error 8.5e-8
        // of the outputs' against 7.4e-8 for uniform gradients; the window kernels' is 7.6e-8).
        v4f part[2][2];
#pragma unroll
        for (int i = 0; i < 4; ++i) part[i >> 1][i & 1] = v4f{};
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (!((y_0 | y_1) >> k & 1)) continue;
            v4f G0{}, G1{};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (x_0 >> j & 1) {
                    G0 = __builtin_amdgcn_mfma_f32_16x16x4f32(g[k][2 * j], Ax[0][2 * j], G0, 0, 0, 0);
                    G0 = __builtin_amdgcn_mfma_f32_16x16x4f32(g[k][2 * j + 1], Ax[0][2 * j + 1], G0, 0, 0, 0);
                }
                if (x_1 >> j & 1) {
                    G1 = __builtin_amdgcn_mfma_f32_16x16x4f32(g[k][2 * j], Ax[1][2 * j], G1, 0, 0, 0);
                    G1 = __builtin_amdgcn_mfma_f32_16x16x4f32(g[k][2 * j + 1], Ax[1][2 * j + 1], G1, 0, 0, 0);
                }
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                if (!((i ? y_1 : y_0) >> k & 1)) continue;
                if (x_0) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        part[i][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(Ay[i][4 * k + e], G0[e], part[i][0], 0, 0, 0);
                }
                if (x_1) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        part[i][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(Ay[i][4 * k + e], G1[e], part[i][1], 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i >> 1][i & 1] += part[i >> 1][i & 1];
    });
    float probe = 0.0f;  // NaN if a sum is an infinity or a NaN
#pragma unroll
    for (int i = 0; i < 16; ++i) probe = fmaf(acc[i >> 3][(i >> 2) & 1][i & 3], 0.0f, probe);
    if (__ballot(probe != 0.0f)) {
        // An infinity or a NaN in the gradient, or an overflow, may have met a zero weight: this wave's hits
        // again, term by term over the weights that are not zero.
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[i >> 1][i & 1] = v4f{};
        for_hits([&](const Axis& ax, const Axis& ay, const float* w, const float* c, global_ptr<const float> gp) {
            AxisLoads wx, wy;
            wx.load(ax, w, c, lane);
            wy.load(ay, w, c, lane);
            __builtin_amdgcn_wave_barrier();
            wx.store(ax, lx, lane);
            wy.store(ay, ly, lane);
            __builtin_amdgcn_wave_barrier();
            const auto weight = [](const float* t, const Axis& x, int pos, int frag) {
                const int at = 31 + pos - frag;
                return t[at] + (x.first && pos == 0 ? t[64 + at] : 0.0f) + (x.last && pos == x.n - 1 ? t[128 + at] : 0.0f);
            };
#pragma unroll
            for (int xi = 0; xi < 2; ++xi)
#pragma unroll 1
                for (int p = 0; p < ay.frag_n; ++p) {
                    float s = 0.0f;
                    for (int q = 0; q < ax.frag_n; ++q) {
                        const float wt = 16 * xi + l < tw ? weight(lx, ax, 16 * xi + l, q) : 0.0f;
                        if (wt != 0.0f) s = fmaf(wt, gp[(int64_t)p * d.ish + (int64_t)q * d.isw], s);
                    }
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int y = 16 * (i >> 2) + 4 * h4 + (i & 3);
                        const float wt = y < th ? weight(ly, ay, y, p) : 0.0f;
                        if (wt != 0.0f) acc[i >> 2][xi][i & 3] = fmaf(wt, s, acc[i >> 2][xi][i & 3]);
                    }
                }
        });
    }
    // (a wave's weights are read before it stores its sums over them: LDS operations of a wave stay in order)
#pragma unroll
    for (int i = 0; i < 16; ++i)
        sums[wave][(16 * (i >> 3) + 4 * h4 + (i & 3)) * kGatherPitch + 16 * ((i >> 2) & 1) + l] = acc[i >> 3][(i >> 2) & 1][i & 3];
    __syncthreads();
    const global_ptr<float> out = as_global(static_cast<float*>(d.out)) + (int64_t)ch * d.osc + (int64_t)Q.ya * d.osh +
                                  (int64_t)Q.xa * d.osw;
    for (int i = tid; i < kGatherTile * kGatherTile; i += 64 * kGatherWaves) {
        const int y = i >> 5, x = i & 31, at = y * kGatherPitch + x;
        float s = sums[0][at];
#pragma unroll
        for (int v = 1; v < kGatherWaves; ++v) s += sums[v][at];
        if (x < tw && y < th) out[(int64_t)y * d.osh + (int64_t)x * d.osw] = s;
    }
}

template <bool ARGS>
fov_status launch_gather(const FwdLaunch& a, int32_t* radius, float* taps, hipStream_t stream) {
    hipLaunchKernelGGL(fov_adj_plan_kernel<ARGS>, dim3(a.nfrag), dim3(64), 0, stream, a, (const FrameDesc*)a.table,
                       (const int32_t*)a.prefix, radius, taps);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_error(e, "adjoint plan kernel launch");
    hipLaunchKernelGGL(fov_adj_gather_kernel<ARGS>, dim3(a.nfrag * a.cmax), dim3(64 * kGatherWaves), 0, stream, a,
                       (const FrameDesc*)a.table, (const int32_t*)a.prefix, (const int32_t*)radius, (const float*)taps);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_error(e, "adjoint gather kernel launch");
    return FOV_OK;
}

template <typename T, int GV, bool ARGS>
fov_status launch_kernels(const FwdLaunch& a, const AdjShape& s, int32_t* radius, T* sc, hipStream_t stream,
                          size_t lds_limit) {
    const auto kw = fov_adj_window_kernel<T, GV, ARGS>;
    fov_status st;
    if ((st = allow_dyn_lds((const void*)kw, lds_limit)) != FOV_OK) return st;
    // one window workgroup per fragment and channel (per fragment if the grid would be too large)
    const int csplit = (int64_t)a.nfrag * s.cmax * kThreads < ((int64_t)1 << 32) ? s.cmax : 1;
    hipLaunchKernelGGL(kw, dim3(a.nfrag * csplit), dim3(kThreads), adjoint_lds(s, sizeof(T)), stream, a, s,
                       (const FrameDesc*)a.table, (const int32_t*)a.prefix, radius, sc, csplit);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_error(e, "adjoint window kernel launch");
    const auto ks = fov_adj_sum_kernel<T, GV, ARGS>;
    const size_t sum_lds = (size_t)kSumCh * s.bmax * (s.bmax + 1) * sizeof(T);
    if (sum_lds + 64 > lds_limit) return set_error(FOV_ERANGE, "adjoint output tile does not fit in LDS");
    if ((st = allow_dyn_lds((const void*)ks, lds_limit)) != FOV_OK) return st;
    hipLaunchKernelGGL(ks, dim3(a.nfrag), dim3(kThreads), sum_lds, stream, a, s,
                       (const FrameDesc*)a.table, (const int32_t*)a.prefix, (const int32_t*)radius, (const T*)sc);
    e = hipGetLastError();
    if (e != hipSuccess) return hip_error(e, "adjoint sum kernel launch");
    return FOV_OK;
}

template <typename T>
fov_status launch_typed(const FwdLaunch& a, const AdjShape& s, int32_t* radius, void* scratch, hipStream_t stream,
                        size_t lds_limit) {
    // values per thread: 4 for fragments of at most 32 x 32 pixels, else kMaxBlock^2 / kThreads
    constexpr int kBig = kMaxBlock * kMaxBlock / kThreads;
    const bool small = s.bmax * s.bmax <= 4 * kThreads;
    T* sc = static_cast<T*>(scratch);
    if (a.from_args)
        return small ? launch_kernels<T, 4, true>(a, s, radius, sc, stream, lds_limit)
                     : launch_kernels<T, kBig, true>(a, s, radius, sc, stream, lds_limit);
    return small ? launch_kernels<T, 4, false>(a, s, radius, sc, stream, lds_limit)
                 : launch_kernels<T, kBig, false>(a, s, radius, sc, stream, lds_limit);
}

}  // namespace

AdjShape adjoint_shape(int es, int r_cap, int bmax, int cmax) {
    AdjShape s;
    s.bmax = bmax;
    s.sw = bmax + 2 * r_cap;
    s.sh = round_up(bmax + r_cap + window_lead(r_cap, es), 128 / es);
    s.cmax = cmax;
    s.pitch_a = tile_pitch(bmax + kPadA + 7, es);
    // rows one wave's tasks span in the vertical transpose, minus one
    const int span = std::min(kPV * (63 / bmax + 1) + kPV - 1, bmax + 2 * r_cap - 1);
    s.pad_b = round_up(span + 4, 4);
    s.pitch_b = inter_pitch(bmax + 2 * s.pad_b, es);
    s.tap_stride = round_up(2 * r_cap + 1 + kAdjWeightLead + 8, 4);
    s.tap_elems = (16 / es) * s.tap_stride;
    s.bdiv = div_magic((uint32_t)bmax);
    // window rows transposed per run: the whole window when the LDS stays within kAdjLdsBudget,
    // else as many rows (a multiple of 4, at least 4) as fit beside the staged gradient
    const size_t g = ((size_t)s.tap_elems + (size_t)bmax * s.pitch_b) * es, row = (size_t)s.pitch_a * es;
    const int fit = g + 4 * row <= kAdjLdsBudget ? (int)((kAdjLdsBudget - g) / row) / 4 * 4 : 4;
    s.rows_r = std::min(round_up(s.sw, 4), fit);
    return s;
}

size_t adjoint_lds(const AdjShape& s, int es) {
    return ((size_t)s.tap_elems + (size_t)s.bmax * s.pitch_b + (size_t)s.rows_r * s.pitch_a) * es;
}

size_t adjoint_scratch_elems(const AdjShape& s, int nfrag) { return (size_t)nfrag * s.cmax * s.sw * s.sh; }

// A tile is 32 x 32 whatever the fragments: sides that leave much of it empty do better with the windows.  Per
// call, gather / windows, 4 x 3 x 512 x 512 with radii up to 36 and then 3, 3 x 1080 x 1920 with radii up to 3: 16 px
// 128 / 347, 66 / 111 and 128 / 205 us; 17 px 303 / 282, 129 / 109 and 241 / 191; 24 px 106 / 155 but 59 / 64 and 107 / 104;
// 26 px 90 / 114, 51 / 58 and 95 / 95; 28 px 78 / 104, 47 / 56 and 84 / 86; 32 px 57 / 85, 37 / 44 and 67 / 71.  (Measured
// later, other fixation, 14 px 102 / 352, 70 / 145, 138 / 275 and 15 px 99 / 304, 69 / 132, 149 / 238, beside 16 px 82 / 280, 61 / 111,
// 106 / 205: two such sides fill a tile as 28 and 30 px do, but the rule does not take them.)
bool adjoint_gathers(int es, int block) {
    return es == 4 && (block == kGatherTile / 2 || (block >= 28 && block <= kGatherTile));
}

bool adjoint_gather_fits(int64_t nfrag, int cmax) { return nfrag * cmax * kThreads < ((int64_t)1 << 32); }

size_t adjoint_tap_elems(int r_cap, int nfrag) { return (size_t)nfrag * adj_tap_stride(r_cap); }

fov_status launch_adjoint_gather(const FwdLaunch& a, int32_t* radius, float* taps, hipStream_t stream) {
    if (a.nfrag <= 0) return FOV_OK;
    return a.from_args ? launch_gather<true>(a, radius, taps, stream) : launch_gather<false>(a, radius, taps, stream);
}

fov_status launch_adjoint(const FwdLaunch& a, const AdjShape& s, int es, int32_t* radius, void* scratch,
                          hipStream_t stream, size_t lds_limit) {
    if (a.nfrag <= 0) return FOV_OK;
    if (adjoint_lds(s, es) + 64 > lds_limit) return set_error(FOV_ERANGE, "adjoint tiles do not fit in LDS");
    return es == 8 ? launch_typed<double>(a, s, radius, scratch, stream, lds_limit)
                   : launch_typed<float>(a, s, radius, scratch, stream, lds_limit);
}

}  // namespace fov
