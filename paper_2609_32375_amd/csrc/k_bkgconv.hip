// k_bkgconv.hip -- local background by convolution, with invalid pixels
// filled from their valid neighbours and a per-pixel noise map.
//
// B = K corr I' for a separable unit-sum kernel K = ky kx^T with half-sample
// reflected borders, where I' is the frame with every invalid pixel (mask
// set, or raw value >= sat) replaced by N = (K corr vI) / (K corr v), the
// kernel-weighted mean of the valid pixels around it (v = 1 valid, 0
// invalid).  Since I' = vI + (1 - v) N,
//   B = A + K corr ((1 - v) N),   A = K corr vI,
// so the path is two rounds of separable passes:
//   1. horizontal pass of vI -> hA; per row, one flag per 64-column band:
//      "an invalid pixel lies here"
//   2. vertical pass -> A; in the 64 x 64 tiles that hold an invalid pixel,
//      C = K corr v from the validity of the tile's neighbourhood (staged as
//      bits, both 1-D passes inside the tile) and the fill image
//      G = (1 - v) A / C -> A, G
//   3. horizontal pass of G -> hG, in the rows with an invalid pixel within
//      the kernel's reach only
//   4. vertical pass of hG, B = A + (K corr G), noise map R from B
// Everywhere else C is never read and K corr G is exactly +0 (a sum of zero
// products), so those sums are skipped: the results are those of the four
// full passes, bit for bit.
// Sums accumulate in FP64 from values stored in the working precision, with
// the unit-sum FP64 taps read as uniform kernel arguments.  Each pass stages
// its rows (or a column band) in LDS with the reflection applied on load, and
// every thread keeps 16 consecutive outputs in registers and slides a window
// over the staged data: one LDS read and conversion per 16 FMAs.  (A row of up
// to 128 outputs goes one output a thread.)
// Each output's sum runs over the taps in order.  Each pass is one
// launch over every frame of the call: a frame table in the workspace gives
// each frame's slices of the planes and flags and its first workgroup of
// each pass.  Noise map for a dark-subtracted frame in ADU:
//   R^2 = (g max(B, 0) + rn^2 + dark texp) / g^2.
#include "k_args.h"
#include "k_convsum.h"

namespace gpk {

// FP64 FMAs bound both passes at first sight (65 taps on 9600 x 6400: 110 us
// each; the vertical pass also moves 1 GB), the waits for the rows of the next
// workgroups and the traffic take the rest: horizontal 260 -> 222 us, vertical
// 445 -> 326 from blocks of 8 outputs whose window was moved by copies, with
// uniform row addresses, stores of 64 neighbours and C at a few invalid pixels
// alone.  (The first vertical pass spills at four wavefronts per SIMD: 40 bytes
// of scratch a lane in FP32, 80 in FP64, nearly all where a tile forms C.)

__device__ __forceinline__ FrameDesc cv_desc(const CvFrame& F) {
    FrameDesc d{};
    d.data = F.data;
    d.pitch = F.pitch;
    d.W = F.W;
    d.H = F.H;
    d.dtype = F.dtype;
    return d;
}

// The columns (or rows) that reads of [a, b] with half-sample reflection at
// the borders of [0, n) can touch lie in [lo, hi] (a superset; monotone in
// [a, b], so a sub-range never reaches beyond its range's reach).
__device__ __forceinline__ void cv_reach(int a, int b, int n, int& lo, int& hi) {
    if (a >= 0 && b < n) {
        lo = a;
        hi = b;
    } else if (a < 0 && b >= n) {
        lo = 0;
        hi = n - 1;
    } else if (a < 0) {
        lo = 0;
        hi = min(n - 1, max(b, -a - 1));
    } else {
        lo = max(0, min(a, 2 * n - 1 - b));
        hi = n - 1;
    }
}

// half-sample reflection into [0, n) for -n <= i < 2n (one reflection), as selects
__device__ __forceinline__ int reflect1(int i, int n) {
    i = i < 0 ? -i - 1 : i;
    return i >= n ? 2 * n - 1 - i : i;
}

// A row segment: its first column, the outputs in it and the staged values
// these read (position i of them: column x0 - hx + i, reflected).
struct CvSeg {
    int y, x0, nseg, n;
    __device__ CvSeg(int local, int W, int lx) {
        const int nsegs = (W + kCvSeg - 1) / kCvSeg;
        y = local / nsegs;
        x0 = (local - y * nsegs) * kCvSeg;
        nseg = min(kCvSeg, W - x0);
        n = nseg + lx - 1;
    }
};
// the columns of this thread's positions tid + 128 k (those past n repeat
// position n - 1), with a loop each for a segment inside the frame, for one
// reflection (the frame is at least half a kernel wide) and for any
template <typename Fn>
__device__ __forceinline__ void cv_columns(const CvSeg& S, int W, int hx, Fn&& fn) {
    const int tid = threadIdx.x, xl = S.x0 - hx;
    if (xl >= 0 && xl + S.n <= W) {
#pragma unroll
        for (int k = 0; k < kHStage; ++k)
            if (k * kCvThreads < S.n) fn(k, (uint32_t)(xl + min(tid + k * kCvThreads, S.n - 1)));
    } else if (W >= hx) {
#pragma unroll
        for (int k = 0; k < kHStage; ++k)
            if (k * kCvThreads < S.n) fn(k, (uint32_t)reflect1(xl + min(tid + k * kCvThreads, S.n - 1), W));
    } else {
#pragma unroll
        for (int k = 0; k < kHStage; ++k)
            if (k * kCvThreads < S.n) fn(k, (uint32_t)reflect_idx(xl + min(tid + k * kCvThreads, S.n - 1), W));
    }
}

// the sums of a staged segment, stored through LDS, so that a store
// instruction writes 64 neighbours.  A segment of at most one output a thread
// goes that way (16 each would leave all but 8 threads idle), with the same
// sums: 50 x 20000 pixels, 33 x 33 taps 81 us a pass, now 53; 128 wide, 129 taps
// 30 and 23.  Wider rows lose by it: 200 wide, two rounds, 129 taps 26.0 and
// 29.3, 300 wide, three, 23.7 and 30.7.
template <typename Real>
__device__ __forceinline__ void cv_hsum(const CvSeg& S, const CvArgs& a, unsigned char* dyn, Real* o0) {
    Real* so = reinterpret_cast<Real*>(dyn);
    if (S.nseg <= kCvThreads) {
        const int i = threadIdx.x;
        if (i >= S.nseg) return;
        double sum = 0.0;
#pragma unroll 8
        for (int b = 0; b < a.lx; ++b) sum = fma(a.kx[b], (double)so[cv_hpos<Real>(i + b)], sum);
        o0[i] = (Real)sum;
        return;
    }
    const int i0 = threadIdx.x * kCvN;
    double acc[kCvN];
    if (i0 < S.nseg) cv_sum16<true>(so + cv_hpos<Real>(i0), a.kx, a.lx, acc);
    __syncthreads();
    if (i0 < S.nseg) {
#pragma unroll
        for (int j = 0; j < kCvN; ++j) so[cv_hpos<Real>(i0) + j] = (Real)acc[j];
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kCvN; ++j) {
        const int i = threadIdx.x + j * kCvThreads;
        if (i < S.nseg) o0[i] = so[cv_hpos<Real>(threadIdx.x) + j * kHRound<Real>];
    }
}

// vI of a segment into LDS, and the flags of its bands
template <typename Real, typename T>
__device__ __forceinline__ void cv_stage_row(const CvFrame& F, const CvSeg& S, int hx, float sat, Real* s0, int* bfl) {
    typedef __attribute__((address_space(1))) const T gT;
    const int tid = threadIdx.x;
    gT* row = (gT*)F.data + (int64_t)S.y * F.pitch;
    T pv[kHStage];
    uint8_t mv[kHStage];
#pragma unroll
    for (int k = 0; k < kHStage; ++k) {
        pv[k] = (T)0;
        mv[k] = 0;
    }
    cv_columns(S, F.W, hx, [&](int k, uint32_t x) __attribute__((always_inline)) { pv[k] = row[x]; });
    if (F.mask) {
        const uint8_t* mrow = F.mask + (int64_t)S.y * F.pitch;
        cv_columns(S, F.W, hx, [&](int k, uint32_t x) __attribute__((always_inline)) { mv[k] = mrow[x]; });
    }
    uint32_t bad = 0u;   // bit k: position tid + 128 k is not valid
#pragma unroll
    for (int k = 0; k < kHStage; ++k) {
        const bool ok = mv[k] == 0 && (float)pv[k] < sat;
        if (!ok) bad |= 1u << k;
        s0[cv_hpos<Real>(tid) + k * kHRound<Real>] = ok ? (Real)pv[k] : (Real)0;
    }
    for (; bad != 0u; bad &= bad - 1u) {
        const int i = tid + __builtin_ctz(bad) * kCvThreads;
        if (i >= hx && i < hx + S.nseg) bfl[(i - hx) / kCvCols] = 1;
    }
}

// vI -> hA, and the flags of the bands
template <typename Real>
__global__ __launch_bounds__(kCvThreads) void k_conv_h(CvWork w, int nframes, int total, CvArgs a) {
    extern __shared__ __align__(16) unsigned char cv_dyn[];
    __shared__ int bfl[kCvSeg / kCvCols];
    const int item = xcd_item(blockIdx.x, (total + kXcds - 1) / kXcds);
    if (item >= total) return;
    const int f = frame_of_wave(nframes, item, [&](int i) { return w.hbase[i]; });
    const CvFrame F = w.tab[f];
    const CvSeg S(item - w.hbase[f], F.W, a.lx);
    const int tid = threadIdx.x, hx = a.lx >> 1, nb = (F.W + kCvCols - 1) / kCvCols;
    if (tid < kCvSeg / kCvCols) bfl[tid] = 0;
    __syncthreads();
    Real* s0 = reinterpret_cast<Real*>(cv_dyn);
    if (F.dtype == kDtypeU16) cv_stage_row<Real, uint16_t>(F, S, hx, a.sat, s0, bfl);
    else cv_stage_row<Real, float>(F, S, hx, a.sat, s0, bfl);
    __syncthreads();
    if (tid < kCvSeg / kCvCols) {
        // every band of every row is written once: no clearing between frames
        const int b = S.x0 / kCvCols + tid;
        if (b < nb) {
            w.flags[F.flags + (int64_t)S.y * nb + b] = (uint8_t)bfl[tid];
            if (bfl[tid]) atomicOr(w.fflag + f, 1);
        }
    }
    cv_hsum<Real>(S, a, cv_dyn, (Real*)w.hA + F.plane + (int64_t)S.y * F.W + S.x0);
}

// G -> hA in the rows whose reach holds an invalid pixel
template <typename Real>
__global__ __launch_bounds__(kCvThreads) void k_conv_h_fill(CvWork w, int nframes, int total, CvArgs a) {
    extern __shared__ __align__(16) unsigned char cv_dyn[];
    const int item = xcd_item(blockIdx.x, (total + kXcds - 1) / kXcds);
    if (item >= total) return;
    const int f = frame_of_wave(nframes, item, [&](int i) { return w.hbase[i]; });
    if (w.fflag[f] == 0) return;   // nothing to fill in this frame
    const CvFrame F = w.tab[f];
    const CvSeg S(item - w.hbase[f], F.W, a.lx);
    const int tid = threadIdx.x, hx = a.lx >> 1, nb = (F.W + kCvCols - 1) / kCvCols;
    const uint8_t* fr = w.flags + F.flags + (int64_t)S.y * nb;
    int lo, hi;
    cv_reach(S.x0 - hx, S.x0 + S.nseg - 1 + hx, F.W, lo, hi);
    bool any = false;
    for (int b = lo / kCvCols + tid; b <= hi / kCvCols; b += kCvThreads) any |= fr[b] != 0;
    if (!__syncthreads_or(any)) return;   // G is zero wherever this row segment reads it
    const Real* row = (const Real*)w.G + F.plane + (int64_t)S.y * F.W;
    Real* s0 = reinterpret_cast<Real*>(cv_dyn);
    Real pv[kHStage];
    uint8_t on[kHStage];
#pragma unroll
    for (int k = 0; k < kHStage; ++k) {
        pv[k] = (Real)0;
        on[k] = 0;
    }
    // G was written in the bands with an invalid pixel and is zero elsewhere
    cv_columns(S, F.W, hx, [&](int k, uint32_t x) __attribute__((always_inline)) {
        pv[k] = row[x];
        on[k] = fr[x / kCvCols];
    });
#pragma unroll
    for (int k = 0; k < kHStage; ++k) s0[cv_hpos<Real>(tid) + k * kHRound<Real>] = on[k] ? pv[k] : (Real)0;
    __syncthreads();
    cv_hsum<Real>(S, a, cv_dyn, (Real*)w.hA + F.plane + (int64_t)S.y * F.W + S.x0);
}

// rows y0 - hy + r, r < nrows, of a 64-column band (columns clamped to the
// frame; the values are only read for columns inside it); zero beyond nrows
// and, with act, in the rows act marks as zero.  Thread (c, g) stages column
// c of rows g, g + 4, ..., kVStage loads in flight before their stores.
constexpr int kVStage = 16;
template <typename Real>
__device__ __forceinline__ void cv_stage(const Real* __restrict__ src, const FrameDesc& d, int xc0, int y0, int hy,
                                         int nrows, int rows, const uint8_t* act, Real* band) {
    const int c = threadIdx.x & (kCvCols - 1), g = threadIdx.x / kCvCols;
    const Real* col = src + min(xc0 + c, d.W - 1);
    for (int r0 = g; r0 < rows; r0 += 4 * kVStage) {
        Real v[kVStage];
#pragma unroll
        for (int k = 0; k < kVStage; ++k) {
            const int r = r0 + 4 * k;
            v[k] = (Real)0;
            if (r < nrows && (!act || act[r])) v[k] = col[(int64_t)reflect_idx(y0 - hy + r, d.H) * d.W];
        }
#pragma unroll
        for (int k = 0; k < kVStage; ++k) {
            const int r = r0 + 4 * k;
            if (r < rows) band[r * kCvCols + c] = v[k];
        }
    }
}

// The same band of FP32 rows loaded straight into LDS (global_load_lds: no
// register round trip, every row's load in flight at once); rows past nrows
// repeat row nrows - 1, finite values that only the zero-padded taps and the
// discarded outputs below the tile read.  Each wavefront has to wait for its
// own loads before the barrier that publishes the band.
__device__ __forceinline__ void cv_stage_direct(const float* __restrict__ src, const FrameDesc& d, int xc0, int y0,
                                                int hy, int nrows, int rows, float* band) {
    // a wavefront takes whole rows: their addresses are uniform
    const int c = threadIdx.x & (kCvCols - 1), g = __builtin_amdgcn_readfirstlane(threadIdx.x / kCvCols);
    const int xc = min(xc0 + c, d.W - 1);
    for (int r = g; r < rows; r += kCvRows / kCvN) {
        const float* p = src + (int64_t)reflect_idx(y0 - hy + min(r, nrows - 1), d.H) * d.W + (uint32_t)xc;
        __builtin_amdgcn_global_load_lds((const void*)p, (void __attribute__((address_space(3)))*)&band[r * kCvCols],
                                         4, 0, 0);
    }
}

// Validity bits of a tile's neighbourhood: bit cc of row r for column xl + cc,
// row yl + r (reflected), cc < 64 + taps - 1; all set in the rows act does not
// mark.  A wavefront takes every fourth row, 8 of them in flight.
template <typename T>
__device__ __forceinline__ void cv_bits(const FrameDesc& d, const uint8_t* __restrict__ mask, float sat, int xl, int yl,
                                        int lx, int nrows, const uint8_t* act, uint64_t* bits) {
    typedef __attribute__((address_space(1))) const T gT;
    const int lane = threadIdx.x & 63, g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ncol = kCvCols + lx - 1;
    constexpr int B = 8;
    for (int c0 = 0; c0 < ncol; c0 += 64) {
        const uint32_t xs = (uint32_t)reflect_idx(xl + min(c0 + lane, ncol - 1), d.W);
        for (int r0 = g; r0 < nrows; r0 += 4 * B) {
            uint32_t on = 0u;   // rows to look at
#pragma unroll
            for (int u = 0; u < B; ++u)
                on |= (r0 + 4 * u < nrows && __builtin_amdgcn_readfirstlane(act[min(r0 + 4 * u, nrows - 1)]) ? 1u : 0u) << u;
            T pv[B];
            uint8_t mv[B];
#pragma unroll
            for (int u = 0; u < B; ++u) {
                pv[u] = (T)0;
                mv[u] = 0;
            }
            if (on != 0u) {
                int64_t row[B];
#pragma unroll
                for (int u = 0; u < B; ++u)
                    row[u] = (int64_t)reflect_idx(yl + min(r0 + 4 * u, nrows - 1), d.H) * d.pitch;
#pragma unroll
                for (int u = 0; u < B; ++u) pv[u] = ((gT*)d.data + row[u])[xs];
                if (mask)
#pragma unroll
                    for (int u = 0; u < B; ++u) mv[u] = (mask + row[u])[xs];
            }
#pragma unroll
            for (int u = 0; u < B; ++u) {
                const bool ok = !((on >> u) & 1u) || (mv[u] == 0 && (float)pv[u] < sat);
                const uint64_t m = __ballot(ok);
                if (lane == 0 && r0 + 4 * u < nrows) bits[(r0 + 4 * u) * kCvBitWords + c0 / 64] = m;
            }
        }
    }
}

// Horizontal pass of the validity v inside a tile: band[r][c] = sum_j kx[j]
// v(xc0 - hx + c + j, row r) for the staged rows, from bits[r] (bit cc of a
// row: column xc0 - hx + cc, reflected, is valid).  The same sums, in the
// same order and stored in the same precision, as a full horizontal pass of v.
template <typename Real>
__device__ __forceinline__ void cv_hbits(const uint64_t* bits, const double* k, int np, int rows, Real* band) {
    for (int it = threadIdx.x; it < rows * (kCvCols / kCvT); it += blockDim.x) {
        const int r = it / (kCvCols / kCvT), c0 = (it - r * (kCvCols / kCvT)) * kCvT;
        const uint8_t* by = reinterpret_cast<const uint8_t*>(bits + r * kCvBitWords);
        double acc[kCvT], w[2 * kCvT];
#pragma unroll
        for (int j = 0; j < kCvT; ++j) acc[j] = 0.0;
        unsigned b8 = by[c0 / 8];
#pragma unroll
        for (int q = 0; q < kCvT; ++q) w[q] = (b8 >> q) & 1u ? 1.0 : 0.0;
        for (int c = 0; c < np; c += kCvT) {
            b8 = by[(c0 + c) / 8 + 1];
#pragma unroll
            for (int q = 0; q < kCvT; ++q) w[kCvT + q] = (b8 >> q) & 1u ? 1.0 : 0.0;
#pragma unroll
            for (int b = 0; b < kCvT; ++b) {
                const double kb = k[c + b];
#pragma unroll
                for (int j = 0; j < kCvT; ++j) acc[j] = fma(kb, w[j + b], acc[j]);
            }
#pragma unroll
            for (int q = 0; q < kCvT; ++q) w[q] = w[kCvT + q];
        }
#pragma unroll
        for (int j = 0; j < kCvT; ++j) band[r * kCvCols + c0 + j] = (Real)acc[j];
    }
}

// The same sum at one column pc of the tile: a tap is added or an exact zero.
__device__ __forceinline__ double cv_hpixel(const uint64_t* bits, int pc, const double* k, int taps) {
    typedef const uint32_t __attribute__((may_alias)) word32_t;
    word32_t* words = reinterpret_cast<word32_t*>(bits);
    double acc = 0.0;
    for (int t0 = 0; t0 < taps; t0 += 32) {
        // 32 bits from bit pc + t0 on
        const int o = pc + t0;
        const uint64_t w = words[o >> 5] | (uint64_t)words[(o >> 5) + 1] << 32;
        const uint32_t v = (uint32_t)(w >> (o & 31));
        auto add = [&](int b) __attribute__((always_inline)) { acc += (v >> b) & 1u ? k[t0 + b] : 0.0; };
        if (taps - t0 >= 32) {
#pragma unroll
            for (int b = 0; b < 32; ++b) add(b);
        } else {
            for (int b = 0; b < taps - t0; ++b) add(b);
        }
    }
    return acc;
}

// noise map of a dark-subtracted frame in ADU from B.  FP64 maps: the
// formula as written, in FP64.  FP32 maps: R^2 = max(B, 0) / g + (rn^2 +
// dark t) / g^2 from the host's FP64 constants, rounded to FP32, and its
// correctly rounded FP32 square root (within 1.25 ulp of R).
template <typename Real>
__device__ __forceinline__ Real cv_noise(double b, const CvArgs& a) {
    const double sky = b > 0.0 ? b : 0.0;
    if (sizeof(Real) == 4) return (Real)sqrtf((float)fma(a.nm_c1, sky, a.nm_c0));
    const double var_e =
        fma((double)a.gain, sky, fma((double)a.read_noise, (double)a.read_noise, (double)a.dark * (double)a.exptime));
    return (Real)sqrt(var_e / ((double)a.gain * (double)a.gain));
}

// FIRST: A from hA; B and R where the fill round adds nothing; in tiles with
// an invalid pixel, C, the fill image G and the unfilled count.  Else, in the
// tiles the fill round reaches: B = A + (K corr G) and the noise map.
template <typename Real, bool FIRST>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_conv_v(CvWork w, int nframes, int total, CvArgs a) {
    extern __shared__ __align__(16) unsigned char cv_dyn[];
    __shared__ uint8_t act[kCvRows + kConvTapsPad];
    __shared__ int ninv;
    const int item = xcd_item(blockIdx.x, (total + kXcds - 1) / kXcds);
    if (item >= total) return;
    const int f = frame_of_wave(nframes, item, [&](int i) { return w.vbase[i]; });
    const int local = item - w.vbase[f];
    const CvFrame F = w.tab[f];
    uint8_t* late_tile = w.tiles + F.tiles;
    if (!FIRST && late_tile[local] == 0) return;   // B and R were written by the first vertical pass
    const FrameDesc d = cv_desc(F);
    const uint8_t* mask = F.mask;
    const float sat = a.sat;
    const Real* in0 = (const Real*)w.hA + F.plane;
    Real* outG = (Real*)w.G + F.plane;
    Real* back = (Real*)F.back;   // also A until the fill round adds to it
    Real* rms = (Real*)F.rms;
    const uint8_t* inval = w.flags + F.flags;
    int* flag = w.fflag + f;
    int64_t* unfilled = w.unfilled + f;
    // down the columns of tiles: the rows that neighbours share stay in the L2
    // (across: 340 us for 325 at 9600 x 6400)
    const int nty = (d.H + kCvRows - 1) / kCvRows, tx = local / nty, ty = local - tx * nty;
    const int np = cv_pad(a.ly), rows = kCvRows + np;
    Real* band = reinterpret_cast<Real*>(cv_dyn);
    const int xc0 = tx * kCvCols, y0 = ty * kCvRows, hy = a.ly >> 1, hx = a.lx >> 1;
    const int nr = min(kCvRows, d.H - y0), nrows = nr + a.ly - 1;
    const int nb = (d.W + kCvCols - 1) / kCvCols;
    const int c = threadIdx.x & (kCvCols - 1), g = __builtin_amdgcn_readfirstlane(threadIdx.x / kCvCols);
    const int x = xc0 + c, rb = g * kCvN;   // this thread's column and first row
    double s0[kCvN], s1[kCvN];
    uint32_t inv = 0u;   // FIRST, tiles with an invalid pixel: this thread's
    bool few = false;    // and their fill values are written (else C is in s1)
    // (the band's loads first: the flags are read while they are in flight)
    constexpr bool kDirect = FIRST && sizeof(Real) == 4;
    if constexpr (kDirect)
        cv_stage_direct(reinterpret_cast<const float*>(in0), d, xc0, y0, hy, nrows, rows,
                        reinterpret_cast<float*>(band));
    // late: K corr G may be non-zero in this tile (some staged row's reach
    // along x holds an invalid pixel; act marks those rows).  Known from the
    // flags of the first horizontal pass, so the first vertical pass already
    // finishes B and R where it is not.
    bool late = false;
    if (flag[0] != 0) {
        int lo, hi;
        cv_reach(xc0 - hx, min(xc0 + kCvCols, d.W) - 1 + hx, d.W, lo, hi);
        bool mine = false;
        for (int r = threadIdx.x; r < nrows; r += blockDim.x) {
            const uint8_t* fr = inval + (int64_t)reflect_idx(y0 - hy + r, d.H) * nb;
            bool on = false;
            for (int b = lo / kCvCols; b <= hi / kCvCols; ++b) on |= fr[b] != 0;
            act[r] = on;
            mine |= on;
        }
        late = __syncthreads_or(mine);
    }
    if (FIRST && threadIdx.x == 0) late_tile[local] = late;
    bool fill;   // FIRST: the tile holds an invalid pixel
    if (FIRST) {
        const bool mine = (int)threadIdx.x < nr && inval[(int64_t)(y0 + threadIdx.x) * nb + tx] != 0;
        fill = __syncthreads_or(mine);
    } else {
        fill = true;
    }
    if constexpr (!kDirect) cv_stage(in0, d, xc0, y0, hy, nrows, rows, FIRST ? nullptr : act, band);
    if constexpr (kDirect) __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (rb < nr) cv_sum16<false>(band + rb * kCvCols + c, a.ky, a.ly, s0);
    if (FIRST && fill) {
        // C: validity bits of the tile's neighbourhood (all set in the rows
        // whose reach holds no invalid pixel)
        uint64_t* bits = reinterpret_cast<uint64_t*>(cv_dyn + conv_v_data_bytes(a.ly, sizeof(Real) == 8));
        CvFew* list = reinterpret_cast<CvFew*>(cv_dyn);
        if (d.dtype == kDtypeU16) cv_bits<uint16_t>(d, mask, sat, xc0 - hx, y0 - hy, a.lx, nrows, act, bits);
        else cv_bits<float>(d, mask, sat, xc0 - hx, y0 - hy, a.lx, nrows, act, bits);
        if (threadIdx.x == 0) ninv = 0;
        __syncthreads();   // bits staged; every wave is done with the band of A
        // the thread's invalid pixels (bit q: row rb + q)
        {
            const int cb = c + hx;
            int n = 0;
#pragma unroll
            for (int q = 0; q < kCvN; ++q)
                if (rb + q < nr && x < d.W && !((bits[(rb + q + hy) * kCvBitWords + (cb >> 6)] >> (cb & 63)) & 1ull))
                    inv |= 1u << q;
            n = __popc(inv);
            const int at = n ? atomicAdd(&ninv, n) : 0;
            if (at + n <= kCvFew) {
                // few so far: their places and A into the list
                int o = at;
#pragma unroll
                for (int q = 0; q < kCvN; ++q)
                    if ((inv >> q) & 1u) list[o++] = CvFew{s0[q], (rb + q) * kCvCols + c, 0};
            }
        }
        __syncthreads();
        few = ninv <= kCvFew && ninv * a.ly <= kCvFewRows;
        if (few) {
            // C at the listed pixels: a thread per row of a pixel's window,
            // then a lane per pixel, with the sums in the order (and stored
            // in the precision) of the sums over the tile, so that a fill
            // value has the same bits whatever else the tile holds
            Real* hrow = reinterpret_cast<Real*>(list + kCvFew);
            for (int e = threadIdx.x; e < ninv * a.ly; e += blockDim.x) {
                const int i = e / a.ly, r = e - i * a.ly, pos = list[i].pos;
                const int pr = pos / kCvCols, pc = pos - pr * kCvCols;
                hrow[e] = (Real)cv_hpixel(bits + (pr + r) * kCvBitWords, pc, a.kx, a.lx);
            }
            __syncthreads();
            if (threadIdx.x < ninv) {
                const CvFew P = list[threadIdx.x];
                const Real* h = hrow + threadIdx.x * a.ly;
                double cs = 0.0;
#pragma unroll 8
                for (int r = 0; r < a.ly; ++r) cs = fma(a.ky[r], (double)h[r], cs);
                double gv = 0.0;
                if (cs != 0.0) gv = P.a / cs;
                else atomicAdd((unsigned long long*)unfilled, 1ull);
                const int pr = P.pos / kCvCols, pc = P.pos - pr * kCvCols;
                outG[(int64_t)(y0 + pr) * d.W + xc0 + pc] = (Real)gv;
            }
        } else {
            cv_hbits(bits, a.kx, cv_pad(a.lx), nrows, band);
            __syncthreads();
            if (rb < nr) cv_sum16<false>(band + rb * kCvCols + c, a.ky, a.ly, s1);
        }
    }
    if (x >= d.W) return;
    int64_t nun = 0;
    if (!FIRST) {
        // A of this thread's outputs, all loaded before back (its own plane) is written
        double av[kCvN];
#pragma unroll
        for (int q = 0; q < kCvN; ++q) av[q] = rb + q < nr ? (double)(back + (int64_t)(y0 + rb + q) * d.W)[(uint32_t)x] : 0.0;
#pragma unroll
        for (int q = 0; q < kCvN; ++q) s0[q] += av[q];
    }
    // four rows at a time, the rest moved up: a quarter of the code of 16
    // (a small frame's workgroups fetch it all for the first time)
#pragma unroll 1
    for (int q0 = 0; q0 < kCvN; q0 += 4) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = rb + q0 + q;
            if (r >= nr) break;
            const int64_t row = (int64_t)(y0 + r) * d.W;   // uniform
            Real *bo = back + row, *ro = rms + row;
            const bool bad = (inv >> (q0 + q)) & 1u;
            if (FIRST) {
                const Real ar = (Real)s0[q];
                if (late) {
                    bo[(uint32_t)x] = ar;   // finished by the fill round
                } else {
                    const double b = (double)ar + 0.0;   // B = A + (K corr G), the latter an exact +0 here
                    bo[(uint32_t)x] = (Real)b;
                    ro[(uint32_t)x] = cv_noise<Real>(b, a);
                }
                if (fill && !(few && bad)) {
                    double gv = 0.0;
                    if (bad) {
                        if (s1[q] != 0.0) gv = s0[q] / s1[q];
                        else ++nun;
                    }
                    (outG + row)[(uint32_t)x] = (Real)gv;
                }
            } else {
                bo[(uint32_t)x] = (Real)s0[q];
                ro[(uint32_t)x] = cv_noise<Real>(s0[q], a);
            }
        }
#pragma unroll
        for (int q = 0; q < kCvN - 4; ++q) {
            s0[q] = s0[q + 4];
            if (FIRST) s1[q] = s1[q + 4];
        }
    }
    if (FIRST && nun) atomicAdd((unsigned long long*)unfilled, (unsigned long long)nun);
}

// the frame records and workgroup bases of one chunk; the per-frame flags
// and unfilled counts start at zero
__global__ void k_conv_setup(CvChunk c, CvWork w) {
    const int i = threadIdx.x;
    if (i < c.count) {
        w.tab[c.first + i] = c.f[i];
        w.hbase[c.first + i] = c.hbase[i];
        w.vbase[c.first + i] = c.vbase[i];
        w.fflag[c.first + i] = 0;
        w.unfilled[c.first + i] = 0;
    }
}

template <typename Real>
static hipError_t conv_t(int nframes, int htotal, int vtotal, const CvArgs& a, const CvWork& w, hipStream_t s) {
    const size_t lh = conv_h_lds<Real>(), lv = conv_v_lds(a.ly, sizeof(Real) == 8);
    hipError_t e;
    const void* hk[2] = {(const void*)k_conv_h<Real>, (const void*)k_conv_h_fill<Real>};
    const void* vk[2] = {(const void*)k_conv_v<Real, true>, (const void*)k_conv_v<Real, false>};
    for (int i = 0; i < 2; ++i) {
        if ((e = hipFuncSetAttribute(hk[i], hipFuncAttributeMaxDynamicSharedMemorySize, (int)lh)) != hipSuccess)
            return e;
        if ((e = hipFuncSetAttribute(vk[i], hipFuncAttributeMaxDynamicSharedMemorySize, (int)lv)) != hipSuccess)
            return e;
    }
    // grids of whole XCD chunks over every frame's workgroups
    const unsigned gh = (unsigned)((htotal + kXcds - 1) / kXcds) * kXcds;
    const unsigned gv = (unsigned)((vtotal + kXcds - 1) / kXcds) * kXcds;
    // 1. horizontal: vI -> hA, invalid-pixel flags
    k_conv_h<Real><<<gh, kCvThreads, lh, s>>>(w, nframes, htotal, a);
    // 2. vertical: A -> back (B and R where step 4 adds nothing); C and the
    //    fill image G in flagged tiles
    k_conv_v<Real, true><<<gv, 256, lv, s>>>(w, nframes, vtotal, a);
    // 3. horizontal pass of G into hA, rows within reach of an invalid pixel
    k_conv_h_fill<Real><<<gh, kCvThreads, lh, s>>>(w, nframes, htotal, a);
    // 4. B = A + vertical pass of it and the noise map, in the tiles it reaches
    k_conv_v<Real, false><<<gv, 256, lv, s>>>(w, nframes, vtotal, a);
    return hipGetLastError();
}

hipError_t launch_conv(const CvChunk* chunks, int nchunks, int nframes, int htotal, int vtotal, const CvArgs& a,
                       const CvWork& w, bool f64, hipStream_t s) {
    for (int i = 0; i < nchunks; ++i) k_conv_setup<<<1, 64, 0, s>>>(chunks[i], w);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return f64 ? conv_t<double>(nframes, htotal, vtotal, a, w, s) : conv_t<float>(nframes, htotal, vtotal, a, w, s);
}

}  // namespace gpk
