// 8-bit frames on the matrix cores, with the bytes of the FP32 kernel.
//
// Each output byte of an 8-bit frame is rint() of an FP32 sum whose order is
// fixed (hconv_sym, then vconv).  This path finds the same byte without
// running that sum for most pixels: it computes the exact value of the filter
// in fixed point on the integer matrix cores, with a proven bound on its own
// error and on the rounding error of the FP32 sum, and rounds.  Where the
// value lies so close to a half-integer that the bound does not decide the
// byte, the FP32 sum itself is run for that pixel, tap by tap in its order.  So
// the bytes are those of the FP32 kernel for every input.
//
// Numbers.  A sample x is the signed byte x - 128.  A tap w becomes the
// integer W = rint(w 2^F), F the largest with W < 2^23 - 0x8080, written in
// three signed base-256 digits W = W2 2^16 + W1 2^8 + W0.  The horizontal sums
// S_d = sum W_d (x - 128) are exact 32-bit integers from
// v_mfma_i32_32x32x32_i8; they combine to the intermediate value in units of
// 2^-Q, Q = min(16, F - 8), a 24-bit integer, again cut into three signed digits
// I2, I1, I0.  The vertical sums are L4 = sum W2 I2, L3 = sum (W2 I1 + W1 I2)
// and L2 = sum (W2 I0 + W1 I1 + W0 I2), exact as well; W1 I0 + W0 I1 + W0 I0
// are left out.  The value is
//   v = 2^-(F+Q) (2^32 L4 + 2^24 L3 + 2^16 L2) + 128 (sum W / 2^F)^2 + 2^-(Q+1).
//
// Bound.  Let V be the exact value for the FP32 taps, N = 2r + 1.
//  * |v - V| <= e1 =
//      1.01 * 255 * 2 sum |w - W 2^-F|  taps, in both passes
//    + 2^-(Q+1) + 2^-(F-8)            the intermediate is cut (not rounded) to 2^-Q; half of
//                                     that is added back in v
//    + 1.01 * N 2^(23-F-Q)            products left out, digits at most 128 in size
//    + 2^-15                          FP32 operations that put v together (|v| <= 256)
//  * The FP32 sum of V: every term is >= 0, so partial sums never exceed the
//    result, and an operation whose result is below 2^(m+1) errs by at most
//    u 2^m, u = 2^-24.  With 2^m <= v < 2^(m+1): the r + 1 operations of a
//    horizontal sum I err by at most u (r + 1) min(I, 128), weighted over the
//    rows u (r + 1) min(v, 128); the r + 1 operations of the vertical sum from
//    the centre tap on by u 2^m each; the r before the centre by u 2^m each or,
//    as their partial sums are at most 255 times the sum of the taps so far,
//    by 255 M in total, M = sum_{j > 0} j w_j (symmetric taps).  Together
//      e2 = 1.02 u ((r + 1) (min(v, 128) + 2^m) + min(128 r, 255 M)).
// |v - rint(v)| <= 1/2 - e1 - e2 then decides the byte.  For frames of random
// content about 2 (e1 + e2) of the pixels are left: 1.6 in a thousand at r = 48.
//
// Mapping.  One workgroup takes a tile of up to 32 x 32 pixels with up to three
// channels: its samples are staged in LDS as bytes, channel planes apart, and
// one wave computes one channel from start to end (the waves meet only at the
// staging barriers; the idle fourth wave rotates so that all SIMDs take
// turns).  Tap digits make one Toeplitz operand, T[k][j] = W[k - j], of which a
// wave holds 32 x 32 blocks in registers: both passes use the same registers, as
// the right operand of the horizontal product (samples x T) and as the left
// operand of the vertical one (T^T x intermediate).  The k index runs inside a
// 32-wide block in the order of the product's result registers (rows 8q + 4h + e
// in half-wave h), so the intermediate's digits go from the horizontal result
// straight into the vertical operand, lane by lane, with byte permutes only, and
// the samples are read from LDS in the same order.
//
// Measured per call (gratings with noise, 32 px fragments, radii up to 48, calls back to back from Python), in brackets as
// the FP32 kernel and the two kernels that it needed then took: 1080 x 1920 x 3 39.6 - 40.0 us (75.6), 480 x 640 gray 8.9 (17.7; now on the
// FP32 kernel by rule where radii are small or frames large), 2160 x 3840 x 3 158 - 163 (275), 64 mixed frames 3110 (5800).  The kernel alone, 1080 x
// 1920 x 3, other frames: 43 us in a trace.  A tile takes 31 thousand cycles (stamps of a 42 us launch): 4 to find the item, 3 to issue its loads, 8
// until the samples are in LDS, 1 for the tap digits, 7 for the products and 6 for the undecided
// pixels; vector units 50 % busy, matrix cores 11 %, waves wait 49 % of their time.  53 KB of LDS and 168 registers
// allow three workgroups a CU.
#pragma once

#include <hip/hip_runtime.h>

#include "conv.h"

namespace fov {
namespace {

constexpr int kFxRadius = 48;  // largest radius of this path (four 32-wide blocks per window)
constexpr int kFxTile = 32;    // output tile side
constexpr int kFxChan = 3;     // channels staged together
// Undecided pixels of one tile that are recomputed one by one; a tile with more
// of them (an image of many exact half-integer means, such as a one-pixel
// checkerboard) is handed to the FP32 passes as a whole.
constexpr int kFxCap = 32;
// Undecided pixels recomputed together: what the LDS beside the planes holds when three workgroups share a
// CU (four-block windows), else more than a tile usually has.
__host__ __device__ constexpr int fx_batch(int nk) { return nk == 4 ? 5 : 16; }

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

// 32-wide blocks of a window at radius r.
__host__ __device__ constexpr int fx_blocks(int r) { return 1 + (r + 15) / 16; }

// LDS row pitch of NK blocks of 32 bytes: an odd number of words, so that lanes on
// consecutive rows, and the two words of a lane pair, hit distinct banks.
__host__ __device__ constexpr int fx_pitch(int nk) { return nk * 32 + 4; }
__host__ __device__ constexpr int fx_plane(int nk) { return nk * 32 * fx_pitch(nk); }

// Bytes of one copy of a digit array: tap t of copy s at byte t + 32 + s.
__host__ __device__ constexpr int fx_digits(int nk) { return 32 * nk + 40; }
// Floats of one undecided pixel's column of horizontal sums.
__host__ __device__ constexpr int fx_col(int nk) { return 32 * (nk - 1) + 4; }

// What the tap wave tells the others, and the tile's undecided pixels: how many, and whether there are too
// many of them.
struct FxHead {
    int F, und, over;
    float bias, lim;  // added to every sum; 1/2 - e1 - the constant part of e2
};

// LDS layout: taps w[N] and 2^24 w_k (k = 1..r); the FxHead; the undecided
// pixels; the digit copies (later the columns of the recomputation); the
// channel planes.
struct FxLds {
    int ws, misc, list, digits, tile, total;
};
__host__ __device__ constexpr FxLds fx_lds(int nk, int nchan) {
    FxLds l{};
    l.ws = fx_col(nk) * 4;
    l.misc = l.ws + (16 * (nk - 1) + 4) * 4;
    l.list = l.misc + 32;
    l.digits = l.list + kFxCap * 2;
    const int dig = 12 * fx_digits(nk), cols = fx_batch(nk) * fx_col(nk) * 4;
    l.tile = l.digits + ((dig > cols ? dig : cols) + 15) / 16 * 16;
    l.total = l.tile + nchan * fx_plane(nk) + 32;  // the recomputation reads up to two words past a row
    return l;
}

__device__ __forceinline__ uint32_t perm(uint32_t hi, uint32_t lo, uint32_t sel) {
    return __builtin_amdgcn_perm(hi, lo, sel);
}

// Unaligned load of N words.
template <int N>
__device__ __forceinline__ void load_words(uint32_t* v, global_ptr<const uint8_t> p) {
    __builtin_memcpy(v, (const void*)p, 4 * N);
}

// Whether a tile's bytes lie within 32-bit offsets of its first one in the output.
__host__ __device__ inline bool fx_reaches(const FrameDesc& d) {
    const int64_t rows = (d.p.block < kFxTile ? d.p.block : kFxTile) - 1;
    return (d.h <= rows ? d.h - 1 : rows) * d.osh + (d.w <= rows ? d.w - 1 : rows) * d.osw < (int64_t)1 << 32;
}

// Staging of a tile's samples (rows y0.., columns x0.., clamped to the frame) in LDS, channel planes
// apart.  A lane takes 16 columns of a row at a time (8 lanes to a row, 4 where a window is two blocks
// wide): fewer and wider loads than one group of four columns per lane, whose 12-byte loads cost the
// L1 twice the accesses per row.
//   kRgb: interleaved three-channel rows, 48 bytes per lane, split into planes in registers;
//   kUnit: column stride 1, 16 bytes per lane and channel;
//   kBytes: any strides (and frames narrower than four columns), byte by byte, straight to LDS: slower than the
//   FP32 kernel (on_fp32()).
// A frame spans less than 2^31 bytes, so offsets are 32-bit.
enum { kRgb = 0, kUnit = 1, kBytes = 2 };
template <typename D>
__host__ __device__ inline int fx_mode(const D& d) {
    return d.w < 4 ? kBytes : (d.isw == 3 && d.isc == 1 && d.c == 3 ? kRgb : (d.isw == 1 ? kUnit : kBytes));
}

template <int NK>
struct FxStager {
    static constexpr int kLanes = NK == 2 ? 4 : 8;     // lanes per row
    static constexpr int kRows = 64 / kLanes;          // rows per wave and task
    static constexpr int kTasks = NK * 32 / (4 * kRows);
    uint32_t v[kTasks][12];  // kRgb: the row's words; kUnit: four words per channel
    int c0, nc, lrow, col;   // lrow: this lane's first row; its others are 4 kRows apart
    bool rgb, later;         // later: the samples are in v (else in LDS already)

    __device__ __forceinline__ void put(unsigned char* tile, int i, int ch, int g, uint32_t t) const {
        *reinterpret_cast<uint32_t*>(tile + (lrow + 4 * kRows * i) * fx_pitch(NK) + col + ch * fx_plane(NK) + 4 * g) = t;
    }
    // Three words of four interleaved pixels to their channels' words (frames of three channels, all staged together).
    __device__ __forceinline__ void put_rgb(unsigned char* tile, int i, int g, uint32_t a, uint32_t b, uint32_t c) const {
        const uint32_t r = perm(c, perm(b, a, 0x0c060300u), 0x05020100u);
        const uint32_t gr = perm(c, perm(b, a, 0x0c070401u), 0x06020100u);
        const uint32_t bl = perm(c, perm(b, a, 0x0c0c0502u), 0x07040100u);
        put(tile, i, 0, g, r);
        put(tile, i, 1, g, gr);
        put(tile, i, 2, g, bl);
    }

    // A tile of TH rows from column x0, row y0 of the frame: issues the loads (store() writes them to LDS).
    // A window that crosses the frame's left or right edge goes to LDS here: each group of four columns is
    // loaded from the nearest four columns inside and its bytes are moved; so do other strides, bytewise.
    __device__ __forceinline__ void load(unsigned char* tile, const FrameDesc& d, int x0, int y0, int c0_, int nc_, int TH,
                                         int wave, int lane) {
        c0 = c0_;
        nc = nc_;
        const int mode = fx_mode(d);
        rgb = mode == kRgb;
        lrow = kRows * wave + lane / kLanes;
        col = 16 * (lane & (kLanes - 1));
        later = mode != kBytes && x0 >= 0 && x0 + 32 * NK <= d.w;
        if (col >= 32 * NK) return;
        const global_ptr<const uint8_t> in = as_global(static_cast<const uint8_t*>(d.in));
        // Rows past the tile's last one are loaded from that one: no branches between the loads, so that
        // all of them are in flight together.
        const uint32_t ish = (uint32_t)d.ish, isc = (uint32_t)d.isc, coff = (uint32_t)c0 * isc;
        const int x = x0 + col, row_max = min(TH, 32 * NK) - 1;
        const auto row = [&](int i) {
            return (uint32_t)clampi(y0 + min(lrow + 4 * kRows * i, row_max), 0, d.h - 1) * ish;
        };
        if (later) {
            const uint32_t off = rgb ? (uint32_t)x * 3u : (uint32_t)x + coff;
            const uint32_t d1 = rgb ? 16u : isc, d2 = rgb ? 32u : (nc > 2 ? 2u * isc : d1);
            if (!rgb && nc == 1) {
#pragma unroll
                for (int i = 0; i < kTasks; ++i) load_words<4>(v[i], in + (row(i) + off));
            } else {
#pragma unroll
                for (int i = 0; i < kTasks; ++i) {
                    const uint32_t o = row(i) + off;
                    load_words<4>(v[i], in + o);
                    load_words<4>(v[i] + 4, in + (o + d1));
                    load_words<4>(v[i] + 8, in + (o + d2));
                }
            }
        } else if (mode == kRgb) {
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int base = clampi(x + 4 * g, 0, d.w - 4);
                uint32_t t[kTasks][3];
#pragma unroll
                for (int i = 0; i < kTasks; ++i) load_words<3>(t[i], in + (row(i) + (uint32_t)base * 3u));
                uint32_t sa[3] = {0, 0, 0}, sb[3] = {0, 0, 0};  // byte k: of column min(max(x + 4g + k / 3, 0), w - 1)
#pragma unroll
                for (int k = 0; k < 12; ++k) {
                    const uint32_t pos = 3 * (uint32_t)(clampi(x + 4 * g + k / 3, 0, d.w - 1) - base) + k % 3;
                    sa[k / 4] |= (pos < 8 ? pos : 0x0cu) << (8 * (k % 4));
                    sb[k / 4] |= (pos < 8 ? (uint32_t)(k % 4) : pos - 8 + 4) << (8 * (k % 4));
                }
#pragma unroll
                for (int i = 0; i < kTasks; ++i) {
                    uint32_t m[3];
#pragma unroll
                    for (int k = 0; k < 3; ++k) m[k] = perm(t[i][2], perm(t[i][1], t[i][0], sa[k]), sb[k]);
                    put_rgb(tile, i, g, m[0], m[1], m[2]);
                }
            }
        } else if (mode == kUnit) {
#pragma unroll 1
            for (int ch = 0; ch < nc; ++ch)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const int base = clampi(x + 4 * g, 0, d.w - 4);
                    uint32_t t[kTasks], sel = 0;
#pragma unroll
                    for (int i = 0; i < kTasks; ++i)
                        load_words<1>(&t[i], in + (row(i) + (uint32_t)base + coff + (uint32_t)ch * isc));
#pragma unroll
                    for (int k = 0; k < 4; ++k) sel |= (uint32_t)(clampi(x + 4 * g + k, 0, d.w - 1) - base) << (8 * k);
#pragma unroll
                    for (int i = 0; i < kTasks; ++i) put(tile, i, ch, g, perm(t[i], t[i], sel));
                }
        } else {
#pragma unroll 1
            for (int ch = 0; ch < nc; ++ch)
#pragma unroll 1
                for (int i = 0; i < kTasks; ++i)
#pragma unroll 1
                    for (int g = 0; g < 4; ++g) {
                        uint32_t t = 0;
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            t |= (uint32_t)in[row(i) + coff + (uint32_t)ch * isc +
                                              (uint32_t)clampi(x + 4 * g + k, 0, d.w - 1) * (uint32_t)d.isw]
                                 << (8 * k);
                        put(tile, i, ch, g, t);
                    }
        }
    }

    // Writes the samples that load() left in registers to the planes.
    __device__ __forceinline__ void store(unsigned char* tile) const {
        if (!later || col >= 32 * NK) return;
        if (rgb) {
#pragma unroll
            for (int i = 0; i < kTasks; ++i)
#pragma unroll
                for (int g = 0; g < 4; ++g) put_rgb(tile, i, g, v[i][3 * g], v[i][3 * g + 1], v[i][3 * g + 2]);
        } else {
#pragma unroll
            for (int i = 0; i < kTasks; ++i)
#pragma unroll
                for (int ch = 0; ch < 3; ++ch)
                    if (ch < nc) {
#pragma unroll
                        for (int g = 0; g < 4; ++g) put(tile, i, ch, g, v[i][4 * ch + g]);
                    }
        }
    }
};

// The FP32 horizontal sum (hconv_sym's terms in its order) at column cc of a staged row.
// ws[k-1] = 2^24 w_k, w0s = 2^24 w_0.
template <int NK>
__device__ __forceinline__ float fx_row_sum(const unsigned char* plane, int row, int cc, int r, float w0s,
                                            const float* __restrict__ ws) {
    // byte selectors: samples cc+1, cc+2 | cc+3, cc+4 and cc-1, cc-2 | cc-3, cc-4, each in 16 bits
    const uint32_t s = (uint32_t)cc & 3u, sr = (s + 1) & 3u, z = 0x0c000c00u;
    const uint32_t r12 = sr | (sr + 1) << 16 | z, r34 = r12 + 0x00020002u;
    const uint32_t l34 = (s + 1) | s << 16 | z, l12 = l34 + 0x00020002u;
    const uint32_t* line = reinterpret_cast<const uint32_t*>(plane + row * fx_pitch(NK));
    const uint32_t* left = line + (cc >> 2);         // words downwards, from the one of column cc
    const uint32_t* right = line + ((cc + 1) >> 2);  // words upwards, from the one of column cc + 1
    uint32_t Lh = left[0], Rl = right[0];
    float acc = fmaf(w0s, (float)as_h2((Lh >> (8 * s)) & 0xffu).x, 0.0f);
    const auto tap = [&](float w, float x) { acc = fmaf(w, x, acc); };
    int k = 0;
    for (; k + 8 <= r; k += 8, left -= 2, right += 2) {
        const uint32_t La = left[-1], Lb = left[-2], Ra = right[1], Rb = right[2];
        const h2v a = as_h2(perm(Ra, Rl, r12) + perm(Lh, La, l12));
        const h2v b = as_h2(perm(Ra, Rl, r34) + perm(Lh, La, l34));
        const h2v c = as_h2(perm(Rb, Ra, r12) + perm(La, Lb, l12));
        const h2v d = as_h2(perm(Rb, Ra, r34) + perm(La, Lb, l34));
        const float4 w = *reinterpret_cast<const float4*>(ws + k), y = *reinterpret_cast<const float4*>(ws + k + 4);
        tap(w.x, (float)a.x);
        tap(w.y, (float)a.y);
        tap(w.z, (float)b.x);
        tap(w.w, (float)b.y);
        tap(y.x, (float)c.x);
        tap(y.y, (float)c.y);
        tap(y.z, (float)d.x);
        tap(y.w, (float)d.y);
        Lh = Lb;
        Rl = Rb;
    }
    for (; k < r; k += 4, --left, ++right) {
        const uint32_t Ll = left[-1], Rh = right[1];
        const h2v a = as_h2(perm(Rh, Rl, r12) + perm(Lh, Ll, l12));
        const h2v b = as_h2(perm(Rh, Rl, r34) + perm(Lh, Ll, l34));
        const float4 w = *reinterpret_cast<const float4*>(ws + k);  // taps past r are not used
        tap(w.x, (float)a.x);
        if (k + 1 < r) tap(w.y, (float)a.y);
        if (k + 2 < r) tap(w.z, (float)b.x);
        if (k + 3 < r) tap(w.w, (float)b.y);
        Lh = Ll;
        Rl = Rh;
    }
    return acc;
}

// One channel of a tile by one wave: `plane` its staged samples, T the tap digit blocks.  Stores the
// bytes at o (rows osh, columns osw apart) and lists the undecided pixels; returns false if the
// list has no room for them.
template <int NK>
__device__ __forceinline__ bool fx_channel(const unsigned char* plane, const v4i (&T)[NK][3], FxHead& head,
                                           float e2, int bw, int bh, global_ptr<uint8_t> o, int64_t osh, int64_t osw,
                                           int ch, uint16_t* list, int lane) {
    const int l = lane & 31, h = lane >> 5;
    const unsigned char* lane_plane = plane + l * fx_pitch(NK) + 4 * h;
    v16i L4{}, L3{}, L2{};
    const int F = head.F, Q = min(16, F - 8), cut = F - 8 - Q;
    const float bias = head.bias, lim = head.lim;
#pragma unroll
    for (int b = 0; b < NK; ++b) {
        v4i P[NK];
#pragma unroll
        for (int j = 0; j < NK; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                P[j][q] = *reinterpret_cast<const int*>(lane_plane + 32 * b * fx_pitch(NK) + 32 * j + 8 * q) ^ (int)0x80808080;
        v16i A{}, C{};
#pragma unroll
        for (int j = 0; j < NK; ++j) A = __builtin_amdgcn_mfma_i32_32x32x32_i8(P[j], T[j][0], A, 0, 0, 0);
#pragma unroll
        for (int j = 0; j < NK; ++j) C = __builtin_amdgcn_mfma_i32_32x32x32_i8(P[j], T[j][2], C, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 16; ++i) A[i] >>= 8;
#pragma unroll
        for (int j = 0; j < NK; ++j) A = __builtin_amdgcn_mfma_i32_32x32x32_i8(P[j], T[j][1], A, 0, 0, 0);
        // intermediate digits, rows 4q .. 4q+3 of a register quad in the bytes of one operand register
        v4i I2, I1, I0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            uint32_t u[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) u[e] = (uint32_t)(((C[4 * q + e] * 256 + A[4 * q + e]) >> cut) + 0x8080);
            const uint32_t lo01 = perm(u[1], u[0], 0x05010400u), lo23 = perm(u[3], u[2], 0x05010400u);
            const uint32_t hi01 = perm(u[1], u[0], 0x0c0c0602u), hi23 = perm(u[3], u[2], 0x0c0c0602u);
            I0[q] = (int)(perm(lo23, lo01, 0x05040100u) ^ 0x80808080u);
            I1[q] = (int)(perm(lo23, lo01, 0x07060302u) ^ 0x80808080u);
            I2[q] = (int)perm(hi23, hi01, 0x05040100u);
        }
        L4 = __builtin_amdgcn_mfma_i32_32x32x32_i8(T[b][2], I2, L4, 0, 0, 0);
        L3 = __builtin_amdgcn_mfma_i32_32x32x32_i8(T[b][2], I1, L3, 0, 0, 0);
        L2 = __builtin_amdgcn_mfma_i32_32x32x32_i8(T[b][2], I0, L2, 0, 0, 0);
        L3 = __builtin_amdgcn_mfma_i32_32x32x32_i8(T[b][1], I2, L3, 0, 0, 0);
        L2 = __builtin_amdgcn_mfma_i32_32x32x32_i8(T[b][1], I1, L2, 0, 0, 0);
        L2 = __builtin_amdgcn_mfma_i32_32x32x32_i8(T[b][0], I2, L2, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);  // one block at a time: its registers are what three waves per SIMD leave
    }
    // Bytes: v + 1.5 2^23 holds rint(v) in its low bits.  The undecided are stored as well and
    // overwritten by the recomputation.
    const float s4 = ldexpf(1.0f, 32 - F - Q), s3 = ldexpf(1.0f, 16 - F - Q), kRound = 12582912.0f;
    const bool full = bw == kFxTile && bh == kFxTile;
    uint32_t und = 0;  // this lane's undecided pixels, the first in bit 15
    uint32_t off = (uint32_t)l * (uint32_t)osw + (uint32_t)(4 * h) * (uint32_t)osh;
    const auto byte = [&](int i) {
        const float v = fmaf((float)(L3[i] * 256 + L2[i]), s3, fmaf((float)L4[i], s4, bias));
        const float n = v + kRound;
        const float t = n - kRound, p2 = __uint_as_float(__float_as_uint(t) & 0x7f800000u);  // 2^m, or the next one
        const float off_by = fmaf(e2, p2, fmaf(e2, fminf(v, 128.0f), fabsf(v - t)));
        und = und + und + (off_by <= lim ? 0u : 1u);
        return (uint8_t)__float_as_uint(n);
    };
    if (full) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            o[off] = byte(i);
            off += (uint32_t)osh * ((i & 3) == 3 ? 5u : 1u);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const uint8_t v = byte(i);
            if (l < bw && 8 * (i >> 2) + 4 * h + (i & 3) < bh) o[off] = v;
            else und &= ~1u;
            off += (uint32_t)osh * ((i & 3) == 3 ? 5u : 1u);
        }
    }
    const int mine = __popc(und);
    if (__ballot(mine != 0) == 0) return true;
    int at = 0;
    if (mine) at = atomicAdd(&head.und, mine);
    const bool over = at + mine > kFxCap;
    if (__ballot(over)) return false;
    for (; und; und &= und - 1) {
        const int i = 15 - __builtin_ctz(und);
        list[at++] = (uint16_t)(ch << 10 | (8 * (i >> 2) + 4 * h + (i & 3)) << 5 | l);
    }
    return true;
}

// The undecided pixels: their horizontal sums by all threads, then one thread per vertical sum.
template <int NK>
__device__ __forceinline__ void fx_recompute(const FrameDesc& d, int r, int xa, int ya, int c0, const unsigned char* tile,
                                             const float* __restrict__ w, const float* __restrict__ ws, float* cols,
                                             const uint16_t* list, int count, int tid) {
    const int N = 2 * r + 1;
    const float w0s = w[r] * kSymScale;
    for (int p0 = 0; p0 < count; p0 += fx_batch(NK)) {
        const int np = min(fx_batch(NK), count - p0);
        const float rnp = 1.0f / (float)np;
        for (int t = tid; t < np * N; t += kThreads) {
            const int k = (int)(((float)t + 0.5f) * rnp), p = t - k * np;  // lanes of a row apart: fewer bank conflicts
            const int px = list[p0 + p];
            cols[p * fx_col(NK) + k] = fx_row_sum<NK>(tile + (px >> 10) * fx_plane(NK), ((px >> 5) & 31) + k,
                                                      (px & 31) + r, r, w0s, ws);
        }
        __syncthreads();
        const int p = (tid >> 6) + 4 * (tid & 63);  // spread over the waves
        if (p < np) {
            const int px = list[p0 + p];
            const float* col = cols + p * fx_col(NK);
            float acc = 0.0f;
            float4 c = *reinterpret_cast<const float4*>(col), t = *reinterpret_cast<const float4*>(w);
            int k = 0;
            for (; k + 4 <= N; k += 4) {
                const float4 cn = *reinterpret_cast<const float4*>(col + k + 4), tn = *reinterpret_cast<const float4*>(w + k + 4);
                acc = fmaf(t.x, c.x, acc);
                acc = fmaf(t.y, c.y, acc);
                acc = fmaf(t.z, c.z, acc);
                acc = fmaf(t.w, c.w, acc);
                c = cn;
                t = tn;
            }
            // N mod 4 is 1 or 3
            acc = fmaf(t.x, c.x, acc);
            if (k + 1 < N) {
                acc = fmaf(t.y, c.y, acc);
                acc = fmaf(t.z, c.z, acc);
            }
            as_global(static_cast<uint8_t*>(d.out))[(int64_t)(c0 + (px >> 10)) * d.osc + (int64_t)(ya + ((px >> 5) & 31)) * d.osh +
                                                    (int64_t)(xa + (px & 31)) * d.osw] =
                (uint8_t)__float_as_uint(acc + 12582912.0f);  // 0 <= acc < 255.5
        }
        if (p0 + fx_batch(NK) < count) __syncthreads();  // the columns are read
    }
}

// A tile: pixels (xa, ya) .. of up to kFxTile squared and channels c0 .. c0 + nc - 1 (nc <= kFxChan) of
// a fragment of radius r with 1 <= r <= kFxRadius.
struct FxJob {
    int r, xa, ya, bw, bh, c0, nc;
};

// Runs a tile with NK = fx_blocks(r).  Returns whether the tile is left to the FP32 passes (the same for every thread).  LDS is in use until every thread has returned.
template <int NK>
__device__ __forceinline__ bool fx_tile(const FrameDesc& d, const FxJob& t, double sigma, unsigned char* smem) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));  // lane addresses computed per tile, not held across tiles
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = t.r, N = 2 * r + 1, TH = t.bh + 2 * r;
    constexpr FxLds at = fx_lds(NK, kFxChan);
    float* w = reinterpret_cast<float*>(smem);
    float* ws = reinterpret_cast<float*>(smem + at.ws);
    FxHead* head = reinterpret_cast<FxHead*>(smem + at.misc);
    uint16_t* list = reinterpret_cast<uint16_t*>(smem + at.list);
    unsigned char* dig = smem + at.digits;
    unsigned char* tile = smem + at.tile;
    FxStager<NK> st;
    st.load(tile, d, t.xa - r, t.ya - r, t.c0, t.nc, TH, wave, lane);
    // The taps and their digits, four byte-shifted copies of each (so that a lane's four taps are one aligned
    // word), by the wave that has no channel to compute: it rotates over the workgroups of a CU.
    const int ch = (wave + (blockIdx.x >> 3)) & 3;
    constexpr int LEN = fx_digits(NK);
    for (int i = tid; i < 12 * LEN / 4; i += kThreads) reinterpret_cast<uint32_t*>(dig)[i] = 0;
    __syncthreads();
    // (Priorities: the others wait for the taps at the staging barrier, and a workgroup in its last phase frees its
    // place soonest.  1080 x 1920 x 3 42.3 -> 41.5 us, gray 27.8 -> 27.3; raised for the loads or the products too, 42.5
    // and 28.7.)
    if (ch == 3) {
        __builtin_amdgcn_s_setprio(3);
        asm volatile("" : "+s"(sigma));  // here, while the samples arrive, and not ahead of the tile loop
        const Taps tp(sigma, r, lane);
        const float w0 = (float)(1.0 / tp.sum);  // tap r
        int F = 22 - ilogbf(w0);
        if (ldexpf(w0, F) > 8355000.0f) --F;
        float off = 0.0f;  // |w 2^F - W|, summed over this lane's taps
        int W = 0, M = 0;  // this lane's taps in units of 2^-F; its part of M in units of 2^(8-F), rounded up
        const auto put_tap = [&](int i, double e) {
            const float t = (float)(e / tp.sum);
            w[i] = t;
            const float tf = ldexpf(t, F);
            const int v = (int)rintf(tf);
            off += fabsf(tf - (float)v);
            W += v;
            if (i > r) {
                ws[i - r - 1] = t * kSymScale;
                M += ((v >> 8) + 1) * (i - r);
            }
            const uint32_t u = (uint32_t)(v + 0x8080);
            const uint8_t b0 = (uint8_t)(u ^ 0x80u), b1 = (uint8_t)((u >> 8) ^ 0x80u), b2 = (uint8_t)(u >> 16);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                dig[(0 * 4 + s) * LEN + i + 32 + s] = b0;
                dig[(1 * 4 + s) * LEN + i + 32 + s] = b1;
                dig[(2 * 4 + s) * LEN + i + 32 + s] = b2;
            }
        };
        if (lane < N) put_tap(lane, tp.e0);
        if (lane + 64 < N) put_tap(lane + 64, tp.e1);
        const double both = wave_sum((double)W), m = wave_sum((double)M), offs = wave_sum((double)off);
        if (lane == 0) {
            const int Q = min(16, F - 8);
            const double sw = ldexp(both, -F);  // sum of the taps
            const float fN = (float)N, u = 1.02f * 5.9604645e-8f;
            const float e1 = 1.01f * 510.0f * ldexpf((float)offs, -F) + ldexpf(1.0f, -Q - 1) + ldexpf(1.0f, 8 - F) +
                             1.01f * ldexpf(fN, 23 - F - Q) + 3.0517578e-5f;
            const float eM = u * fminf(128.0f * (float)r, 255.0f * ldexpf((float)m, 8 - F));
            head->F = F;
            head->und = head->over = 0;
            head->bias = (float)(128.0 * sw * sw) + ldexpf(1.0f, -Q - 1);
            head->lim = 0.5f - e1 - eM;
        }
    }
    st.store(tile);
    __builtin_amdgcn_s_setprio(0);
    __syncthreads();
    v4i T[NK][3];
    {
        const int l = lane & 31, h = lane >> 5, s = l & 3;
#pragma unroll
        for (int j = 0; j < NK; ++j)
#pragma unroll
            for (int dg = 0; dg < 3; ++dg)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    T[j][dg][q] = *reinterpret_cast<const int*>(dig + (dg * 4 + s) * LEN + 32 * j + 8 * q + 4 * h - l + s + 32);
    }
    if (ch < t.nc) {
        global_ptr<uint8_t> o = as_global(static_cast<uint8_t*>(d.out)) + (int64_t)(t.c0 + ch) * d.osc +
                                (int64_t)t.ya * d.osh + (int64_t)t.xa * d.osw;
        const bool ok = fx_channel<NK>(tile + ch * fx_plane(NK), T, *head, 1.02f * 5.9604645e-8f * (float)(r + 1),
                                       t.bw, t.bh, o, d.osh, d.osw, ch, list, lane);
        if (!ok && lane == 0) head->over = 1;
    }
    __syncthreads();
    if (head->over) return true;
    const int und = head->und;
    __builtin_amdgcn_s_setprio(2);
    if (und) fx_recompute<NK>(d, r, t.xa, t.ya, t.c0, tile, w, ws, reinterpret_cast<float*>(dig), list, und, tid);
    return false;
}

}  // namespace
}  // namespace fov
