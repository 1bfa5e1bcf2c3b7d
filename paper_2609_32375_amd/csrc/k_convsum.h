// k_convsum.h -- the windowed sums of the background by convolution and the
// LDS they read: the workgroup shapes, the layouts and their bytes.
//
// Functions for the host and the device: the launches take their LDS bytes
// from here, and a test runs the sums on the host over buffers of those bytes.
#pragma once
#include "k_args.h"

namespace gpk {

constexpr int kCvT = 8;                     // taps are padded to a multiple of it
constexpr int kCvN = 16;                    // outputs per thread (register block), and taps per step
constexpr int kCvThreads = 128;             // threads per horizontal workgroup
constexpr int kCvSeg = kCvThreads * kCvN;   // outputs per horizontal workgroup
constexpr int kCvCols = 64;                 // columns per vertical workgroup
constexpr int kCvRows = 64;                 // output rows per vertical workgroup (4 wavefronts x 16)
static_assert(kCvSeg == kCvSegPx && kCvCols == kCvTilePx && kCvRows == kCvTilePx, "workgroup shapes");

// 64-bit words of validity bits per staged row in a tile: columns
// xc0 - hx + 0 .. 63 + padded taps + 7
constexpr int kCvBitWords = (kCvCols + kConvTapsPad + kCvT + 63) / 64;

__host__ __device__ __forceinline__ int cv_pad(int n) { return (n + kCvT - 1) / kCvT * kCvT; }
// A vertical workgroup's data: the band, or after A's sums the list of a few
// invalid pixels and the rows of their C; then the bits.
struct CvFew {
    double a;
    int32_t pos, pad;
};
// C is formed at a tile's invalid pixels alone, instead of over the tile, up to
// kCvFew of them whose windows hold up to kCvFewRows rows together: one thread
// sums a row, so that is four rounds of the workgroup, and both ways' rounds
// grow with the taps along x.  All 64 x 64 tiles of a masked 2048^2 frame, us a
// pass alone / over the tile, FP32: 65 x 65 taps 137 / 157 for 4 pixels, 158 /
// 164 for 16, 178 / 165 for 32; 129 x 129 264 / 307 for 4, 299 / 313 for 8, 359 /
// 316 for 16; 33 x 21 123 / 126 for 48, 127 / 127 for 64; 9 x 9 108 / 112 for 48;
// 5 x 129 (nearly no taps along x) 210 / 217 for 24, 225 / 219 for 48.  FP64:
// 65 x 65 212 / 213 for 16, 129 x 129 477 / 463 for 8, 33 x 21 161 / 164 for 48.
constexpr int kCvFew = 48, kCvFewRows = 1024;
__host__ __device__ __forceinline__ size_t conv_v_data_bytes(int ly, bool f64) {
    const size_t real = f64 ? 8 : 4;
    const size_t band = (size_t)(kCvRows + cv_pad(ly)) * kCvCols * real;
    const size_t few = (sizeof(CvFew) + ly * real) * kCvFew;
    return band > few ? band : few;
}

// A row of a horizontal pass in LDS: 16 bytes of padding after every 16
// values, so that the threads' blocks of 16, read 16 bytes at a time, fall on
// different banks (without it a pass took 426 us for 250).
template <typename V>
__host__ __device__ __forceinline__ constexpr int cv_hpos(int i) {
    return i + 16 / (int)sizeof(V) * (i / kCvN);
}

// acc[j] = sum_b k[b] w(j + b) over the taps in order for 16 outputs, w(i)
// the values from src on (ROW: of a row, at cv_hpos; else of a column of a
// 64-column band).  The window of 32 values is a ring whose halves steps of
// 16 taps refill in turn, so nothing in it moves: 16 LDS reads per 256 FMAs.
// The last (taps mod 16) go one by one with a window of their own: of a
// column its groups of four past the last output's window are read from the
// column's start instead, which leaves at most two values past that window for
// an odd number of taps, all within the kCvRows + cv_pad(taps) rows of a band
// (a row's stage holds every group).  No value outside an output's window
// meets its sum.
template <bool ROW, typename V>
__host__ __device__ __forceinline__ void cv_sum16(const V* src, const double* k, int taps, double (&acc)[kCvN]) {
    double lo[kCvN], hi[kCvN];
    // 16 values from index c (a multiple of 16) on
    auto load = [&](int c, double (&to)[kCvN]) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < kCvN; q += 4) {
            if constexpr (ROW && sizeof(V) == 8) {
                const double2* p = reinterpret_cast<const double2*>(src + cv_hpos<V>(c) + q);
                const double2 u = p[0], v = p[1];
                to[q] = u.x;
                to[q + 1] = u.y;
                to[q + 2] = v.x;
                to[q + 3] = v.y;
            } else if constexpr (ROW) {
                const float4 v = *reinterpret_cast<const float4*>(src + cv_hpos<V>(c) + q);
                to[q] = (double)v.x;
                to[q + 1] = (double)v.y;
                to[q + 2] = (double)v.z;
                to[q + 3] = (double)v.w;
            } else {
                const int g = c + q < taps + kCvN - 1 ? c + q : 0;
#pragma unroll
                for (int e = 0; e < 4; ++e) to[q + e] = (double)src[(g + e) * kCvCols];
            }
        }
    };
    // taps c .. c + nb - 1 over the window (x, y)
    auto step = [&](int c, int nb, const double (&x)[kCvN], const double (&y)[kCvN]) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < kCvN; ++b) {
            if (b < nb) {
                const double kb = k[c + b];
#pragma unroll
                for (int j = 0; j < kCvN; ++j) acc[j] = fma(kb, b + j < kCvN ? x[(b + j) % kCvN] : y[(b + j) % kCvN], acc[j]);
            }
        }
    };
#pragma unroll
    for (int j = 0; j < kCvN; ++j) acc[j] = 0.0;
    load(0, lo);
    int c = 0;
    for (; c + 2 * kCvN <= taps; c += 2 * kCvN) {
        load(c + kCvN, hi);
        step(c, kCvN, lo, hi);
        load(c + 2 * kCvN, lo);
        step(c + kCvN, kCvN, hi, lo);
    }
    // fewer than 32 taps are left
    while (c < taps) {
        load(c + kCvN, hi);
        step(c, taps - c, lo, hi);
#pragma unroll
        for (int q = 0; q < kCvN; ++q) lo[q] = hi[q];
        c += kCvN;
    }
}

// staged positions per thread, every load issued before the first store
constexpr int kHStage = (kCvSeg + kConvTapsPad + kCvThreads - 1) / kCvThreads;
template <typename V>
constexpr int kHRound = kCvThreads + 16 / (int)sizeof(V) * (kCvThreads / kCvN);   // a round of positions in LDS

template <typename Real>
inline size_t conv_h_lds() {
    return sizeof(Real) * (size_t)kHStage * kHRound<Real>;
}
inline size_t conv_v_lds(int ly, bool f64) {
    return conv_v_data_bytes(ly, f64) + (size_t)(kCvRows + cv_pad(ly)) * kCvBitWords * 8;
}

}  // namespace gpk
