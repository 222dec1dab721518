// Forward block-wise foveation for gfx950: one launch per batch of frames, one workgroup per work item
// (Alg. 1).  A work item finds its fragment from its number (decode()), the fragment's sigma from its
// midpoint's eccentricity (Sec. 2, Fig. 1) or the sigma map, the radius r = ceil(3 sigma) and the normalised
// taps w_k = exp(-k^2/(2 sigma^2)) / sum (Eq. 1 cut at 3 sigma, Appendix "Methods"), the taps while its first
// samples are on their way.  Earlier forms ran a plan kernel (taps of every fragment) and an order kernel (a
// counting sort by radius) first; for small calls the three launches in series were the time (480p gray 17.7
// us a call, 10.7 without them; 1080p RGB 57.1 and 49.0), for large ones the order kernel's single workgroup
// (64 mixed frames 4280 us and 3503).  Calls of more than kArgFrames frames upload their frame table.
//
//  * fov_fwd_kernel: the padded tile (fragment plus r on each side, clamp-to-edge) is staged into LDS
//    with row-coalesced loads, 8-bit input as 16-bit integers; a horizontal
//    pass writes the fp32 intermediate into LDS; a vertical pass produces the
//    fragment (Appendix "Workload of the Block", "Shared Memory").  Each
//    thread computes 8 (horizontal) or 4 (vertical) outputs and slides the
//    filter window through registers (the register reuse of Appendix "Data
//    Reuse"); both passes read the weights as broadcast LDS loads.  For 8-bit input the horizontal
//    pass adds the two samples that share a weight (the taps are symmetric) exactly,
//    two sums per 32-bit integer add, before the FP32 multiply-add.  A
//    fragment with r = 0 is copied.
//  * fov_fwd_u8_kernel: 8-bit output with radii up to 48, the same bytes on the matrix cores (fixed.h).
//
// Every output sums its taps in the same order (k = -r .. r; for 8-bit input
// the horizontal pass goes k = 0, then the pairs +-1 .. +-r) whatever the
// strip height, output tile split or dispatch mode, so results do not depend
// on tuning choices.
#include "forward.h"

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include "conv.h"
#include "fixed.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace fov {

namespace {

struct Geom {
    int N;   // taps, 2r+1
    int G;   // horizontal-pass column groups
    int GV;  // vertical-pass row groups
    int TW;  // staged tile columns (8G + 2r)
    int TH;  // staged tile rows = intermediate rows (4GV + 2r)
};

__host__ __device__ inline Geom geom(int r, int bw, int bh) {
    Geom g;
    g.N = 2 * r + 1;
    g.G = (bw + kPH - 1) / kPH;
    g.GV = (bh + kPV - 1) / kPV;
    g.TW = g.G * kPH + g.N - 1;
    g.TH = g.GV * kPV + g.N - 1;
    return g;
}

// ---- element conversions ----------------------------------------------------------------------
template <typename TS, typename TIn>
__device__ __forceinline__ TS to_stage(TIn v) { return (TS)v; }

template <typename TOut, typename TC>
__device__ __forceinline__ TOut to_out(TC v) { return (TOut)v; }
template <>
__device__ __forceinline__ uint8_t to_out<uint8_t, float>(float v) {
    v = rintf(v);  // round half to even
    v = __builtin_amdgcn_fmed3f(v, 0.0f, 255.0f);  // clamp to [0, 255] (the value is never NaN)
    return (uint8_t)v;
}

template <typename TOut, typename TIn>
__device__ __forceinline__ TOut copy_out(TIn v) { return (TOut)v; }

// ---- staging of the padded tile ---------------------------------------------------------------
// The tile is staged into LDS in strips of at most kStripMax rows.  Each strip
// is loaded in two halves: issue() starts the global loads into registers
// (lanes walk columns, so loads coalesce along x; wave w owns rows w, w+4,
// ...), commit() converts the values and writes them to LDS.  The kernel
// issues strip k+1 before computing strip k, so load latency hides behind
// arithmetic.  Columns beyond the prefetched chunks are loaded and written
// inside commit().
constexpr int kStripMax = 64;
// Bytes of LDS before the tile: the symmetric horizontal pass may read (and ignore) up to three
// samples before a row's first one.
constexpr int kTileLead = 16;
constexpr int kRowsPerWave = kStripMax / (kThreads / 64);

// Raw buffer descriptor (dword 3 as gfx9 expects for untyped access).
constexpr int kBufferWord3 = 0x00020000;
// Byte offset past any descriptor's range: a buffer load there returns 0.
constexpr uint32_t kOutside = 0x7fffffffu;

// Rows are read with buffer loads: each lane's column offsets are fixed for the
// fragment (past the range beyond the tile, so that no lane predicate stands around the loads) and a row's
// offset is a wave-uniform scalar that steps inside the frame.  Per-row clamps, 64-bit products and lane
// predicates were most of the scalar instructions of a work item: FP32 kernel, 4 x 3 x 512 x 512 48.5 -> 44.0 us,
// 32 x 3 x 224 x 224 41.4 -> 37.7 us, 256 x 256 8.8 -> 8.3 us.  The offsets are from the frame's first byte where its bytes
// fit 31 bits, else (far) from each strip's first row; frames of which not even a strip does are loaded in commit().
template <typename TIn, typename TS>
struct Stager {
    static constexpr int KB = 2;  // prefetched 64-column chunks
    TIn v[kRowsPerWave][KB];
    uint32_t coff[KB];
    __amdgpu_buffer_rsrc_t rsrc;
    const TIn* base;
    const TIn* plane;
    int64_t ish, isw;
    int y0, rows, h, w, x_first, TW;
    bool near, far;

    __device__ __forceinline__ void setup(int x_first_, int TW_, int w_, int64_t isw_, int64_t ish_, int h_,
                                          const TIn* base_, int64_t span) {
        x_first = x_first_; TW = TW_; w = w_; isw = isw_; ish = ish_; h = h_;
        base = base_;
        far = span * (int64_t)sizeof(TIn) >= (int64_t)kOutside;
        near = !far || ((kStripMax - 1) * ish_ + (w_ - 1) * isw_ + 1) * (int64_t)sizeof(TIn) < (int64_t)kOutside;
        rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<TIn*>(base_), 0, (int)(span * sizeof(TIn)), kBufferWord3);
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const int tx = kb * 64 + lane;
            const uint32_t co = (uint32_t)clampi(x_first + tx, 0, w - 1) * (uint32_t)isw;
            coff[kb] = tx < TW ? co * (uint32_t)sizeof(TIn) : kOutside;
        }
    }
    __device__ __forceinline__ void issue(const TIn* plane_, int y0_, int rows_) {
        plane = plane_; y0 = y0_; rows = rows_;
        const int wave = wave_id();
        if (!near) return;
        const bool inside = y0 >= 0 && y0 + rows <= h;
        const uint32_t ib = (uint32_t)ish * (uint32_t)sizeof(TIn);
        uint32_t poff = (uint32_t)((plane - base) * sizeof(TIn));
        if (__builtin_expect(far, 0)) {
            const int first = clampi(y0, 0, h - 1);
            rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<TIn*>(plane + first * ish), 0, (int)kOutside, kBufferWord3);
            poff = 0u - (uint32_t)first * ib;
        }
        const uint32_t step = (uint32_t)(kThreads / 64) * ib;
        uint32_t so = poff + (uint32_t)(y0 + wave) * ib;
#pragma unroll
        for (int rb = 0; rb < kRowsPerWave; ++rb) {
            const int ty = wave + rb * (kThreads / 64);
            if (ty < rows) {
                if (!inside) so = poff + (uint32_t)clampi(y0 + ty, 0, h - 1) * ib;
#pragma unroll
                for (int kb = 0; kb < KB; ++kb) v[rb][kb] = load(coff[kb], so);
                so += step;
            }
        }
    }
    __device__ __forceinline__ TIn load(uint32_t voff, uint32_t soff) const {
        if constexpr (sizeof(TIn) == 8)
            return __builtin_bit_cast(TIn, __builtin_amdgcn_raw_buffer_load_b64(rsrc, (int)voff, (int)soff, 0));
        else
            return __builtin_bit_cast(TIn, __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)voff, (int)soff, 0));
    }
    __device__ __forceinline__ void commit(TS* tile, int TP) {
        const int wave = wave_id(), lane = threadIdx.x & 63;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            if (!near || kb * 64 + lane >= TW) continue;
            TS* dst = tile + wave * TP + kb * 64 + lane;
#pragma unroll
            for (int rb = 0; rb < kRowsPerWave; ++rb)
                if (wave + rb * (kThreads / 64) < rows) dst[rb * (kThreads / 64) * TP] = to_stage<TS, TIn>(v[rb][kb]);
        }
        for (int k0 = near ? 64 * KB : 0; k0 < TW; k0 += 64) {
            const int tx = k0 + lane;
            if (tx >= TW) continue;
            const int64_t co = (int64_t)clampi(x_first + tx, 0, w - 1) * isw;
            for (int ty = wave; ty < rows; ty += kThreads / 64)
                tile[ty * TP + tx] = to_stage<TS, TIn>(plane[(int64_t)clampi(y0 + ty, 0, h - 1) * ish + co]);
        }
    }
};

// 8-bit input staged as 16-bit integers, two columns per lane and one 32-bit
// LDS write per pair (b1 << 16 | b0).  Read as fp16, such a half is the
// subnormal b * 2^-24, which the symmetric horizontal pass multiplies by taps
// scaled by 2^24.  One 128-column chunk is prefetched.  Bytes are read with
// buffer loads over the frame (a descriptor covering its bytes): each lane's
// two column offsets are fixed for the fragment and a row's offset is a
// wave-uniform scalar, so no per-row address arithmetic runs on the vector
// unit; reads past the descriptor's range would return 0.
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ half2_t bytes_to_half2(uint32_t b0, uint32_t b1) {
    return __builtin_bit_cast(half2_t, (b1 << 16) | b0);
}

__device__ __forceinline__ uint32_t load_byte(__amdgpu_buffer_rsrc_t rsrc, uint32_t voff, uint32_t soff) {
    return (uint32_t)(uint8_t)__builtin_amdgcn_raw_buffer_load_b8(rsrc, (int)voff, (int)soff, 0);
}

template <>
struct Stager<uint8_t, _Float16> {
    uint32_t b0[kRowsPerWave], b1[kRowsPerWave];
    uint32_t c0, c1;
    bool cv;
    __amdgpu_buffer_rsrc_t rsrc;
    const uint8_t* base;
    uint32_t poff, ish;
    uint32_t isw;
    int y0, rows, h, w, x_first, TW;

    // base: the frame's first byte; span: bytes from base to its last byte + 1 (< 2^31)
    __device__ __forceinline__ void setup(int x_first_, int TW_, int w_, int64_t isw_, int64_t ish_, int h_,
                                          const uint8_t* base_, int64_t span) {
        x_first = x_first_; TW = TW_; w = w_; isw = (uint32_t)isw_; ish = (uint32_t)ish_; h = h_;
        base = base_;
        rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(base_), 0, (int)span, kBufferWord3);
        const int tx = 2 * (threadIdx.x & 63);  // tx + 1 < TP always
        cv = tx < TW;
        c0 = (uint32_t)clampi(x_first + tx, 0, w - 1) * isw;
        c1 = (uint32_t)clampi(x_first + tx + 1, 0, w - 1) * isw;
    }
    __device__ __forceinline__ void issue(const uint8_t* plane_, int y0_, int rows_) {
        poff = (uint32_t)(plane_ - base);
        y0 = y0_; rows = rows_;
        if (!cv) return;  // one lane predicate for all rows (not one exec-mask region per row)
        const int wave = wave_id();
        if (y0 >= 0 && y0 + rows <= h) {
            // strip inside the frame: row offsets step by 4 rows, no clamping
            const uint32_t s0 = poff + (uint32_t)(y0 + wave) * ish, step = (uint32_t)(kThreads / 64) * ish;
            if (rows == kStripMax) {  // full strip: every row of every wave
#pragma unroll
                for (int rb = 0; rb < kRowsPerWave; ++rb) {
                    b0[rb] = load_byte(rsrc, c0, s0 + rb * step);
                    b1[rb] = load_byte(rsrc, c1, s0 + rb * step);
                }
                return;
            }
#pragma unroll
            for (int rb = 0; rb < kRowsPerWave; ++rb)
                if (wave + rb * (kThreads / 64) < rows) {
                    b0[rb] = load_byte(rsrc, c0, s0 + rb * step);
                    b1[rb] = load_byte(rsrc, c1, s0 + rb * step);
                }
            return;
        }
#pragma unroll
        for (int rb = 0; rb < kRowsPerWave; ++rb) {
            const int ty = wave + rb * (kThreads / 64);
            if (ty < rows) {
                const uint32_t soff = poff + (uint32_t)clampi(y0 + ty, 0, h - 1) * ish;
                b0[rb] = load_byte(rsrc, c0, soff);
                b1[rb] = load_byte(rsrc, c1, soff);
            }
        }
    }
    __device__ __forceinline__ void commit(_Float16* tile, int TP) {
        const int wave = wave_id(), lane = threadIdx.x & 63;
        if (cv) {
            half2_t* dst = reinterpret_cast<half2_t*>(tile + wave * TP + 2 * lane);
            const int step = (kThreads / 64) * TP / 2;  // half2 elements per 4 rows (TP is even)
            if (rows == kStripMax) {
#pragma unroll
                for (int rb = 0; rb < kRowsPerWave; ++rb) dst[rb * step] = bytes_to_half2(b0[rb], b1[rb]);
            } else {
#pragma unroll
                for (int rb = 0; rb < kRowsPerWave; ++rb)
                    if (wave + rb * (kThreads / 64) < rows) dst[rb * step] = bytes_to_half2(b0[rb], b1[rb]);
            }
        }
        for (int k0 = 128; k0 < TW; k0 += 128) {
            const int tx = k0 + 2 * lane;
            if (tx >= TW) continue;
            const uint32_t d0 = (uint32_t)clampi(x_first + tx, 0, w - 1) * isw;
            const uint32_t d1 = (uint32_t)clampi(x_first + tx + 1, 0, w - 1) * isw;
            for (int ty = wave; ty < rows; ty += kThreads / 64) {
                const uint32_t soff = poff + (uint32_t)clampi(y0 + ty, 0, h - 1) * ish;
                *reinterpret_cast<half2_t*>(tile + ty * TP + tx) =
                    bytes_to_half2(load_byte(rsrc, d0, soff), load_byte(rsrc, d1, soff));
            }
        }
    }
};

// ---- fragments of a launch ---------------------------------------------------------------------
// Narrow a fragment to output tile `sub` of its L-level split: tiles of
// T = ceil(B / 2^L) pixels a side, row-major, clipped to the fragment and the
// frame.  Returns false for a tile that holds no pixel (ragged splits).
template <typename D>
__device__ __forceinline__ bool narrow_to_tile(Frag& F, const D& d, int L, int sub) {
    if (L == 0) return true;
    const FrameParams& fp = d.p;
    const int B = fp.block, T = (B + (1 << L) - 1) >> L;
    const int sx = sub & ((1 << L) - 1), sy = sub >> L;
    const int X0 = fp.origin_x + F.bx * B, Y0 = fp.origin_y + F.by * B;
    const int x0 = X0 + sx * T, y0 = Y0 + sy * T;
    const int x1 = min(min(x0 + T, X0 + B), d.w), y1 = min(min(y0 + T, Y0 + B), d.h);
    F.xa = max(x0, 0);
    F.ya = max(y0, 0);
    F.bw = x1 - F.xa;
    F.bh = y1 - F.ya;
    return F.bw > 0 && F.bh > 0;
}

// Foveal fragment: copied (Appendix "Workload of the Block").
template <typename TIn, typename TOut>
__device__ __forceinline__ void copy_fragment(const Frag& F, int c_lo, int c_hi) {
    const FrameDesc& d = *F.fd;
    const TIn* in = static_cast<const TIn*>(d.in);
    TOut* out = static_cast<TOut*>(d.out);
    const int wave = wave_id(), lane = threadIdx.x & 63;
    for (int c = c_lo; c < c_hi; ++c)
        for (int y = wave; y < F.bh; y += kThreads / 64)
            for (int x = lane; x < F.bw; x += 64) {
                const TIn v = in[c * d.isc + (int64_t)(F.ya + y) * d.ish + (int64_t)(F.xa + x) * d.isw];
                out[c * d.osc + (int64_t)(F.ya + y) * d.osh + (int64_t)(F.xa + x) * d.osw] = copy_out<TOut, TIn>(v);
            }
}

// ---- main kernel ---------------------------------------------------------------------------------
// One fragment: stage its padded tile strip by strip (the next strip's loads
// in flight while the current one is computed), horizontal pass into the
// column-major intermediate, vertical pass into the output.
template <typename TIn, typename TOut, typename TS, typename TC>
__device__ __forceinline__ void process_fragment(int r_cap, int strip_rows, int r, double sigma, const Frag& F, int c_lo,
                                                 int c_hi, unsigned char* smem) {
    const FrameDesc& d = *F.fd;
    if (r == 0) {
        copy_fragment<TIn, TOut>(F, c_lo, c_hi);
        return;
    }
    const int tid = threadIdx.x;
    const Geom g = geom(r, F.bw, F.bh);
    const int SR = min(min(strip_rows, kStripMax), g.TH);
    // 8-bit input: the symmetric horizontal pass wants each output's centre on a 4-sample group,
    // so the tile starts sh = (-r) mod 4 columns further left.
    constexpr bool kSym = std::is_same<TS, _Float16>::value;
    const int sh = kSym ? ((-r) & 3) : 0;
    const int TW = g.TW + sh;
    const int TP = tile_pitch(TW, sizeof(TS));
    const int IP = inter_pitch(g.TH, sizeof(TC));
    // The fragment's taps go to LDS once (read by the passes as broadcast LDS loads, so the inner
    // loops wait on LDS only): w[0 .. N-1] = w_{-r} .. w_r, then for the symmetric
    // pass ws[j] = 2^24 w_{j+1} (j = 0 .. r-1) at a 16-byte boundary (scaled for the 16-bit
    // integer samples, which it reads as fp16 subnormals; the scaling is exact).
    TC* w = reinterpret_cast<TC*>(smem + kTileLead);
    TC* ws = w + round_up(g.N, 4);
    TS* tile = reinterpret_cast<TS*>(smem + kTileLead + tap_lds_bytes(r_cap, sizeof(TC)));
    TC* inter = reinterpret_cast<TC*>(reinterpret_cast<unsigned char*>(tile) +
                                      align16((size_t)SR * TP * sizeof(TS)));  // [column][row]
    const TIn* in = static_cast<const TIn*>(d.in);
    const int nst = (g.TH + SR - 1) / SR;
    const int nunits = (c_hi - c_lo) * nst;  // (channel, strip) units, channels c_lo .. c_hi - 1
    // Tasks map to (row, column group) and (column, row group) with shifts: the column groups of a
    // 16-row block and the columns of the vertical pass are padded to powers of two (the padding
    // tasks idle; 32-pixel fragments have none).  LDS offsets stay below 2^24, so their products
    // are 24-bit multiplies.
    const int gsh = ceil_log2(g.G), xsh = ceil_log2(F.bw);
    const uint32_t IPH = (uint32_t)IP * kPH;
    // The way to the first strip runs at a raised wave priority, so that its loads are on their way before other
    // workgroups' multiply-adds (FP32, 4 x 3 x 512 x 512 45.0 -> 43.4 us, 32 x 3 x 224 x 224 34.8 -> 33.9; from the item's
    // start on, 43.6 and 33.9, but 8-bit to float 2 % slower).
    __builtin_amdgcn_s_setprio(2);
    Stager<TIn, TS> st;
    const int64_t span = (int64_t)(d.c - 1) * d.isc + (int64_t)(d.h - 1) * d.ish + (int64_t)(d.w - 1) * d.isw + 1;
    st.setup(F.xa - r - sh, TW, d.w, d.isw, d.ish, d.h, in, span);
    st.issue(in + c_lo * d.isc, F.ya - r, SR);
    // the taps, while the first strip's samples arrive
    Taps tp(sigma, r, tid & 63);
    for (int q = wave_id(); 64 * q < g.N; q += kThreads / 64) {
        const int i = 64 * q + (tid & 63);
        if (i >= g.N) continue;
        const TC v = (TC)tp.tap(q, r, tid & 63);
        w[i] = v;
        if (kSym && i > r) ws[i - r - 1] = v * kSymScale;
    }
    int cu = 0, sidx = 0;  // the current unit: channel c_lo + cu, strip sidx
    for (int u = 0; u < nunits; ++u) {
        st.commit(tile, TP);
        __builtin_amdgcn_s_setprio(0);
        __syncthreads();  // the strip is staged; every thread is past the previous vertical pass
        const int c = c_lo + cu;
        const int s0 = sidx * SR, rows = min(SR, g.TH - s0);
        int cn = cu, sn = sidx + 1;  // the next unit
        if (sn == nst) {
            sn = 0;
            ++cn;
        }
        if (u + 1 < nunits) st.issue(in + (c_lo + cn) * d.isc, F.ya - r + sn * SR, min(SR, g.TH - sn * SR));
        // Horizontal pass.  Task t: lanes of a 16-lane group take 16
        // consecutive rows of one column group (conflict-free row reads).
        const int ntask = round_up(rows, 16) << gsh;
        bool four = false;  // 8-bit strips of at most half a workgroup of tasks: 4-output tasks
        if constexpr (kSym) {
            if (ntask <= kThreads / 2) {
                four = true;
                for (int t = tid; t < 2 * ntask; t += kThreads) {
                    const int blk = t >> 4, gi = blk & ((2 << gsh) - 1);
                    const int ty = ((blk >> (gsh + 1)) << 4) | (t & 15);
                    if (ty >= rows || gi >= 2 * g.G) continue;
                    float a4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
                    const TS* row = tile + __umul24((uint32_t)ty, (uint32_t)TP) + gi * 4;
                    hconv_sym4(a4, row + r + sh, r, w[r] * kSymScale, ws);
                    TC* dst = inter + __umul24((uint32_t)gi, (uint32_t)(4 * IP)) + s0 + ty;
#pragma unroll
                    for (int p = 0; p < 4; ++p) dst[p * IP] = a4[p];
                }
            }
        }
        const int ntask8 = four ? 0 : ntask;
        for (int t = tid; t < ntask8; t += kThreads) {
            const int blk = t >> 4, gi = blk & ((1 << gsh) - 1);
            const int ty = ((blk >> gsh) << 4) | (t & 15);
            if (ty >= rows || gi >= g.G) continue;
            TC acc[kPH];
#pragma unroll
            for (int p = 0; p < kPH; ++p) acc[p] = 0;
            const TS* row = tile + __umul24((uint32_t)ty, (uint32_t)TP) + gi * kPH;
            if constexpr (kSym) hconv_sym(acc, row + r + sh, r, w[r] * kSymScale, ws);
            else hconv(acc, row, g.N, w);
            TC* dst = inter + __umul24((uint32_t)gi, IPH) + s0 + ty;
#pragma unroll
            for (int p = 0; p < kPH; ++p) dst[p * IP] = acc[p];
        }
        __syncthreads();  // the tile is free; the channel's intermediate may be complete
        if (sidx == nst - 1) {
            // Vertical pass over the complete intermediate of channel c.  Output rows step by the
            // row stride from one 64-bit address per task.
            const int64_t osh = d.osh, osw = d.osw;
            const global_ptr<TOut> oc =
                as_global(static_cast<TOut*>(d.out)) + c * d.osc + (int64_t)F.ya * osh + (int64_t)F.xa * osw;
            const int ntv = g.GV << xsh;
            for (int t = tid; t < ntv; t += kThreads) {
                const int x = t & ((1 << xsh) - 1), y0 = (t >> xsh) * kPV;
                if (x >= F.bw) continue;
                TC acc[kPV];
#pragma unroll
                for (int p = 0; p < kPV; ++p) acc[p] = 0;
                vconv(acc, inter + __umul24((uint32_t)x, (uint32_t)IP) + y0, g.N, w);
                global_ptr<TOut> o = oc + (int64_t)x * osw + (int64_t)y0 * osh;
                if ((F.bh & (kPV - 1)) == 0) {  // whole row groups (uniform): no per-row test
#pragma unroll
                    for (int p = 0; p < kPV; ++p) {
                        *o = to_out<TOut, TC>(acc[p]);
                        o += osh;
                    }
                } else {
#pragma unroll
                    for (int p = 0; p < kPV; ++p) {
                        if (y0 + p < F.bh) *o = to_out<TOut, TC>(acc[p]);
                        o += osh;
                    }
                }
            }
        }
        cu = cn;
        sidx = sn;
    }
}

// Counts of a launch: from the arguments or (replayed launches) the device header.
struct Counts {
    int nitems, nframes, split_log2, merge;
};

template <bool ARGS>
__device__ __forceinline__ Counts counts(const FwdLaunch& a) {
    Counts n{a.nitems, a.nframes, a.split_log2, a.merge};
    if (!ARGS && a.hdr) {
        n.nitems = __builtin_amdgcn_readfirstlane(a.hdr[2]);
        n.nframes = __builtin_amdgcn_readfirstlane(a.hdr[0]);
        n.merge = __builtin_amdgcn_readfirstlane(a.hdr[1]);
        n.split_log2 = __builtin_amdgcn_readfirstlane(a.hdr[3]);
    }
    return n;
}

// A work item: a rectangle (a fragment, a merged pair of them or an output tile of one) with the sigma and
// radius of its fragment, and its channels c_lo .. c_hi - 1.
struct Item {
    int r, c_lo, c_hi;
    double sigma;
    Frag F;
};

// Work item i of the launch; false if it holds nothing.  Items take the fragments in the order of
// ranked_frame(), dealt so that neighbours, which share halo samples, meet in one L2: workgroup b runs on XCD
// b mod 8, each with an L2 of its own, and of every 64 items an XCD gets eight consecutive ones.
// FIXED: a launch of the 8-bit kernel, which has neither channel items nor pairs.
template <bool ARGS, bool FIXED = false>
__device__ __forceinline__ bool decode(const FwdLaunch& a, const FrameDesc* __restrict__ table,
                                       const int32_t* __restrict__ prefix, const Counts& n, int i, Item* it) {
    const int L = n.split_log2;
    if ((i | 63) < n.nitems) i = (i & ~63) | (i & 7) << 3 | (i >> 3 & 7);
    const int sub = i & ((1 << (2 * L)) - 1);
    int k = i >> (2 * L), ch = -1;
    if (!FIXED && a.chan) {
        const int q = k / a.cmax;
        ch = k - q * a.cmax;
        k = q;
    }
    int f, rank;
    ranked_frame<ARGS>(a, prefix, n.nframes, k, &f, &rank);
    const auto describe = [&](const auto& d) {
        const FrameParams& fp = d.p;
        Place at;
        if constexpr (FIXED) {
            // Tiles of small radii cost much the same and are bound by memory: their order there.  (A run of eight
            // along a row of fragments stays on one XCD, and its tiles share lines.)  Per call, this order / the costliest first, 3 x
            // 1080 x 1920 planar, radii up to 3 22.0 / 27.2 us, 15 24.2 / 28.9, up to 48 over the whole frame 37.8 / 37.1, from the middle on 44.1 / 43.0;
            // interleaved 22.3 / 24.1, 24.3 / 25.6, 38.0 / 34.3, 43.5 / 39.6.  Frames that an XCD's cache of 4 MB holds gain less,
            // 480 x 640 x 3, up to 3 8.5 / 9.9, 15 9.1 / 10.0, and where a radius counts may lose, 16 with 20 px 12.1 / 10.9.
            if (a.r_cap <= 8 || (a.r_cap <= 16 && (int64_t)d.h * d.w * d.c >= 4 << 20)) at = row_place(fp.nbx, rank);
            else at = item_place(Grid{fp.nbx, d.nby, d.ahead_x, d.ahead_y, 0, 0, 0, 0}, rank, false);
        }
        else at = item_place(grid_of(d), rank, n.merge);
        Frag F = placed_at(d, f, at);
        const int bx = F.bx, by = F.by;
        const double sigma = uniform(fragment_sigma(fp, F.lb, bx, by));
        int r = __builtin_amdgcn_readfirstlane(radius_of(sigma));
        if (r > a.r_cap) r = a.r_cap;  // the host sized everything for r_cap; plans agree bit for bit
        // Vertical pairs at the cap (rows 2k and 2k+1, both sigma == cap, hence equal taps): one fragment's item covers
        // both (see item_place()).
        if (!FIXED && n.merge && r > 0 && sigma == fp.cap) {
            const int by2 = by ^ 1;
            if (by2 < d.nby && fragment_sigma(fp, F.lb + (by2 - by) * fp.nbx, bx, by2) == fp.cap) {
                if (at.box && ((__popc((by >> 1) ^ bx) ^ by) & 1)) return false;
                const Frag U = fragment_at(d, f, bx, by & ~1), V = fragment_at(d, f, bx, by | 1);
                F.ya = U.ya;
                F.bh = V.ya + V.bh - U.ya;
            }
        }
        if (!narrow_to_tile(F, d, L, sub)) return false;
        it->r = r;
        it->sigma = sigma;
        it->c_lo = max(ch, 0);
        it->c_hi = ch < 0 ? d.c : min(ch + 1, d.c);
        it->F = F;
        return it->c_lo < it->c_hi;
    };
    if constexpr (FIXED) return describe(geo_of<ARGS>(a, table, f));
    else return describe(frame_of<ARGS>(a, table, f));
}

// One workgroup per work item, in turn (PERSIST = false: handed out by the hardware dispatcher as workgroups
// retire; PERSIST = true: a grid sized to what the chip holds at once, workgroup b taking items b,
// b + grid, ...).
template <typename TIn, typename TOut, typename TS, typename TC, bool PERSIST, bool ARGS>
__global__ __launch_bounds__(kThreads) void fov_fwd_kernel(const FwdLaunch a, const FrameDesc* __restrict__ table,
                                                           const int32_t* __restrict__ prefix) {
    extern __shared__ __align__(16) unsigned char smem[];
    const Counts n = counts<ARGS>(a);
    for (int i = blockIdx.x; i < n.nitems; i += gridDim.x) {
        Item it;
        if (decode<ARGS>(a, table, prefix, n, i, &it)) {
            it.F.fd = &frame_of<ARGS>(a, table, it.F.f);
            process_fragment<TIn, TOut, TS, TC>(a.r_cap, a.strip_rows, it.r, it.sigma, it.F, it.c_lo, it.c_hi, smem);
        }
        if (!PERSIST) break;
        __syncthreads();  // this fragment's LDS reads are done before the next one is staged
    }
}

// ---- 8-bit main kernel ---------------------------------------------------------------------------
// 8-bit frames to 8-bit frames in launches of radius up to kFxRadius: one workgroup per work item, its
// tiles on the matrix cores (fixed.h); r = 0 is copied.
//
// The FP32 passes for a tile that the matrix cores leave.  A function of its own: it is rare, and inlined
// it would take registers from the common path.  Its arguments arrive in vector registers; they are made scalar again, as
// the passes need them: 1080 x 1920 x 3, radii up to 48, of a one-pixel checkerboard, all of whose tiles come here, 177 us a
// call with them as they arrive, 136 so (86 on the FP32 kernel alone; 32 for stripes, none of whose do).
__device__ __attribute__((noinline)) void fp32_tile(FrameDesc fd, double sigma, int r_cap, int strip_rows, int r,
                                                    int xa, int ya, int bw, int bh, int c_lo, int c_hi) {
    extern __shared__ __align__(16) unsigned char smem[];
    const auto scalar = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    struct Words {
        int32_t w[sizeof(FrameDesc) / 4];
    };
    Words words = __builtin_bit_cast(Words, fd);
#pragma unroll
    for (int32_t& w : words.w) w = scalar(w);
    const FrameDesc d = __builtin_bit_cast(FrameDesc, words);
    Frag P;
    P.fd = &d;
    P.f = P.lb = P.bx = P.by = 0;  // not used by the passes
    P.xa = scalar(xa);
    P.ya = scalar(ya);
    P.bw = scalar(bw);
    P.bh = scalar(bh);
    process_fragment<uint8_t, uint8_t, _Float16, float>(scalar(r_cap), scalar(strip_rows), scalar(r), uniform(sigma), P,
                                                        scalar(c_lo), scalar(c_hi), smem);
}

template <bool ARGS>
__global__ __launch_bounds__(kThreads, 3) void fov_fwd_u8_kernel(const FwdLaunch a, const FrameDesc* __restrict__ table,
                                                                 const int32_t* __restrict__ prefix) {
    extern __shared__ __align__(16) unsigned char smem[];
    const Counts n = counts<ARGS>(a);
    Item it;
    if ((int)blockIdx.x >= n.nitems || !decode<ARGS, true>(a, table, prefix, n, blockIdx.x, &it)) return;
    const FrameDesc& d = frame_of<ARGS>(a, table, it.F.f);
    it.F.fd = &d;
    if (it.r == 0) {
        copy_fragment<uint8_t, uint8_t>(it.F, it.c_lo, it.c_hi);
        return;
    }
    const int r = it.r, nk = fx_blocks(r);
    for (int c0 = it.c_lo; c0 < it.c_hi; c0 += kFxChan)
        for (int ty = 0; ty < it.F.bh; ty += kFxTile)
            for (int tx = 0; tx < it.F.bw; tx += kFxTile) {
                if (c0 > it.c_lo || (ty | tx)) __syncthreads();  // the previous tile's LDS is read
                const FxJob t{r, it.F.xa + tx, it.F.ya + ty, min(it.F.bw - tx, kFxTile), min(it.F.bh - ty, kFxTile), c0,
                              min(it.c_hi - c0, kFxChan)};
                bool left;
                if (nk == 2) left = fx_tile<2>(d, t, it.sigma, smem);
                else if (nk == 3) left = fx_tile<3>(d, t, it.sigma, smem);
                else left = fx_tile<4>(d, t, it.sigma, smem);
                if (left) {
                    __syncthreads();
                    fp32_tile(d, it.sigma, a.r_cap, a.strip_rows, r, t.xa, t.ya, t.bw, t.bh, c0, c0 + t.nc);
                }
            }
}

// Device plan for foveate_plan(): sigma and radius only.
__global__ void fov_plan_kernel(FrameParams fp, int n, double* sigma_out, int32_t* r_out) {
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= n) return;
    const int by = b / fp.nbx, bx = b - by * fp.nbx;
    double s = fp.sigma_map ? clip_map_sigma((double)fp.sigma_map[b], fp.cap) : fragment_sigma_ramp(fp, bx, by);
    if (sigma_out) sigma_out[b] = s;
    r_out[b] = radius_of(s);
}

template <typename TIn, typename TOut, typename TS, typename TC, bool PERSIST, bool ARGS>
fov_status launch_main(const FwdLaunch& a, size_t lds, hipStream_t stream,
                       size_t lds_limit, int cus, hipEvent_t ev_start, hipEvent_t ev_stop) {
    auto kern = fov_fwd_kernel<TIn, TOut, TS, TC, PERSIST, ARGS>;
    fov_status st = allow_dyn_lds((const void*)kern, lds_limit);
    if (st != FOV_OK) return st;
    int grid = a.nitems;
    if (PERSIST) grid = std::max(1, std::min(a.nitems, std::max(occupancy_of((const void*)kern, lds), 1) * cus));
    if (ev_start || ev_stop) {
        // The dispatch itself stamps the events: no separate event packets (each would leave a
        // gap of several microseconds between the kernels of the stream).
        hipExtLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), lds, stream, ev_start, ev_stop, 0, a,
                              (const FrameDesc*)a.table, (const int32_t*)a.prefix);
    } else {
        hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), lds, stream, a, (const FrameDesc*)a.table,
                           (const int32_t*)a.prefix);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_error(e, "forward kernel launch");
    return FOV_OK;
}

template <bool ARGS>
fov_status launch_u8(const FwdLaunch& a, size_t lds, hipStream_t stream, size_t lds_limit, hipEvent_t ev_start,
                     hipEvent_t ev_stop) {
    auto kern = fov_fwd_u8_kernel<ARGS>;
    fov_status st = allow_dyn_lds((const void*)kern, lds_limit);
    if (st != FOV_OK) return st;
    if (ev_start || ev_stop)
        hipExtLaunchKernelGGL(kern, dim3(a.nitems), dim3(kThreads), lds, stream, ev_start, ev_stop, 0, a,
                              (const FrameDesc*)a.table, (const int32_t*)a.prefix);
    else
        hipLaunchKernelGGL(kern, dim3(a.nitems), dim3(kThreads), lds, stream, a, (const FrameDesc*)a.table,
                           (const int32_t*)a.prefix);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_error(e, "forward kernel launch");
    return FOV_OK;
}

template <typename TIn, typename TOut, typename TS, typename TC>
fov_status launch_typed(const FwdLaunch& a, size_t lds, hipStream_t stream, size_t lds_limit, int cus, bool persist,
                        hipEvent_t ev_start, hipEvent_t ev_stop) {
    if constexpr (std::is_same<TOut, uint8_t>::value)
        if (!a.fp32 && forward_fixed(FOV_U8, FOV_U8, a.r_cap))
            return (a.from_args ? launch_u8<true> : launch_u8<false>)(a, lds, stream, lds_limit, ev_start, ev_stop);
    const auto main = a.from_args ? (persist ? launch_main<TIn, TOut, TS, TC, true, true> : launch_main<TIn, TOut, TS, TC, false, true>)
                                  : (persist ? launch_main<TIn, TOut, TS, TC, true, false> : launch_main<TIn, TOut, TS, TC, false, false>);
    return main(a, lds, stream, lds_limit, cus, ev_start, ev_stop);
}

int stage_size(int in_dtype) { return in_dtype == FOV_U8 ? 2 : (in_dtype == FOV_F32 ? 4 : 8); }
int compute_size(int in_dtype) { return in_dtype == FOV_F64 ? 8 : 4; }

}  // namespace

int forward_strip_max() { return kStripMax; }

int forward_tile_rows(int r, int tile_h) { return geom(r, 1, tile_h).TH; }

bool forward_fixed(int in_dtype, int out_dtype, int r_cap) {
    return in_dtype == FOV_U8 && out_dtype == FOV_U8 && r_cap >= 1 && r_cap <= kFxRadius;
}

bool forward_fixed_bytewise(const FrameDesc& d) { return d.w >= 4 && fx_mode(d) == kBytes; }

bool forward_fixed_reaches(const FrameDesc& d) { return fx_reaches(d); }

// Per call: 354 x 563 gray, 64 px fragments, 24.1 -> 9.8 us; 1080 x 1920 x 3, 64 px, 63 -> 46; 400 x 600 x 3, 48 px, 33 -> 11.5.
bool forward_tiled(int in_dtype, int out_dtype, int r_cap, int block) {
    return forward_fixed(in_dtype, out_dtype, r_cap) && block > kFxTile;
}

size_t forward_lds_bytes(int in_dtype, int out_dtype, int r_cap, int tile_w, int tile_h, int strip_rows, bool only_fp32) {
    const Geom g = geom(r_cap, tile_w, tile_h);
    int rows = strip_rows < g.TH ? strip_rows : g.TH;
    if (rows > kStripMax) rows = kStripMax;
    const int es = stage_size(in_dtype), ec = compute_size(in_dtype);
    // 8-bit input: (-r) mod 4 leading columns; 2r + ((-r) mod 4) never decreases with r, so r_cap sizes them
    const int TW = g.TW + (in_dtype == FOV_U8 ? ((-r_cap) & 3) : 0);
    const size_t fp32 = kTileLead + tap_lds_bytes(r_cap, ec) + align16((size_t)rows * tile_pitch(TW, es) * es) +
                        (size_t)g.G * kPH * inter_pitch(g.TH, ec) * ec + 64;
    if (only_fp32 || !forward_fixed(in_dtype, out_dtype, r_cap)) return fp32;
    // the matrix-core tiles and the FP32 passes take turns in one allocation
    return std::max(fp32, (size_t)fx_lds(fx_blocks(r_cap), kFxChan).total);
}

fov_status launch_forward(const FwdLaunch& a, int in_dtype, int out_dtype, size_t lds, hipStream_t stream,
                          size_t lds_limit, int cus, bool persist, hipEvent_t ev_start,
                          hipEvent_t ev_stop) {
    if (a.nfrag <= 0) return FOV_OK;
    if (in_dtype == FOV_U8 && out_dtype == FOV_U8)
        return launch_typed<uint8_t, uint8_t, _Float16, float>(a, lds, stream, lds_limit, cus, persist, ev_start, ev_stop);
    if (in_dtype == FOV_U8 && out_dtype == FOV_F32)
        return launch_typed<uint8_t, float, _Float16, float>(a, lds, stream, lds_limit, cus, persist, ev_start, ev_stop);
    if (in_dtype == FOV_F32 && out_dtype == FOV_F32)
        return launch_typed<float, float, float, float>(a, lds, stream, lds_limit, cus, persist, ev_start, ev_stop);
    if (in_dtype == FOV_F64 && out_dtype == FOV_F64)
        return launch_typed<double, double, double, double>(a, lds, stream, lds_limit, cus, persist, ev_start, ev_stop);
    return set_error(FOV_EDTYPE, "unsupported dtype pair");
}

int forward_occupancy(int in_dtype, int out_dtype, int r_cap, size_t lds, bool fp32) {
    const void* k = forward_main_kernel(in_dtype, out_dtype, r_cap, fp32);
    return k ? occupancy_of(k, lds) : 0;
}

const void* forward_main_kernel(int in_dtype, int out_dtype, int r_cap, bool fp32) {
    if (!fp32 && forward_fixed(in_dtype, out_dtype, r_cap)) return (const void*)fov_fwd_u8_kernel<false>;
    if (in_dtype == FOV_U8 && out_dtype == FOV_U8) return (const void*)fov_fwd_kernel<uint8_t, uint8_t, _Float16, float, false, false>;
    if (in_dtype == FOV_U8 && out_dtype == FOV_F32) return (const void*)fov_fwd_kernel<uint8_t, float, _Float16, float, false, false>;
    if (in_dtype == FOV_F32 && out_dtype == FOV_F32) return (const void*)fov_fwd_kernel<float, float, float, float, false, false>;
    if (in_dtype == FOV_F64 && out_dtype == FOV_F64) return (const void*)fov_fwd_kernel<double, double, double, double, false, false>;
    return nullptr;
}

fov_status launch_plan(const FrameParams& fp, int nblk, double* sigma_out, int32_t* r_out, hipStream_t stream) {
    if (nblk <= 0) return FOV_OK;
    hipLaunchKernelGGL(fov_plan_kernel, dim3((nblk + 255) / 256), dim3(256), 0, stream, fp, nblk, sigma_out, r_out);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_error(e, "plan kernel launch");
    return FOV_OK;
}

}  // namespace fov
