// k_common.h -- device-side descriptors and helpers shared by the gfx950 kernels.
//
// Frames of a batch are described by FrameDesc records that live in the
// workspace; every stage kernel works on a flattened index space (meshes,
// tiles, objects) over all frames and finds its frame by a binary search over
// per-frame prefix offsets.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gpk {

constexpr int kTile = 64;          // detection tile edge; equals the wavefront width
constexpr int kMaxK = 15;          // largest filter edge
constexpr int kMaxR = kMaxK / 2;   // largest filter half-width
constexpr int kNixMax = 6;         // spline x-pieces a tile region (<= 78 columns) can touch (mesh >= 16)
constexpr int kRegion = kTile + 2 * kMaxR;  // 78: tile plus filter halo
constexpr int kLocalRecs = 160;    // components per tile accumulated in LDS
constexpr int kMaxRadii = 8;
constexpr int kDescChunk = 8;      // descriptors written per init launch
constexpr int kNumCounters = 64;   // detection counters (zeroed per call)
constexpr int kScanChunk = 512;    // rank bitmap: 1024-bit blocks per scan workgroup
constexpr int kMaxScanChunks = 4096;   // scan workgroups of one batch (2^31 pixels)

enum : int { kDtypeU16 = 1, kDtypeF32 = 2 };
enum : uint32_t { kFlagSat = 1u, kFlagEdge = 2u, kFlagNonpos = 4u, kFlagTrunc = 8u };

struct FrameDesc {
    const void* data;
    int64_t pitch;
    int32_t W, H, dtype, pad0;
    int32_t mw, mh, nx, ny;
    double* back_raw;     // [ny][nx]
    double* rms_raw;
    double* back;         // filtered
    double* rms;
    double* coef;         // [2][ny+1][nx+1][16]
    int32_t* iters;       // [ny][nx]
    double* ycoef;        // workspace: [2][ny+1][nx][4]
    double* scratch;      // workspace: Thomas sweeps of the y and x splines
    int32_t mesh_base;    // first flattened mesh of this frame
    int32_t tile_base;    // first flattened detection tile
    int32_t ntx, nty;     // detection tiles per row / column
    uint32_t* bitmap;     // first-pixel bitmap of this frame (1024-bit blocks)
    int32_t bm_block_base, nblocks;
    int32_t cat_base;     // first catalogue row of this frame
    int32_t pad1;
    int32_t* seg;         // nullable segmentation map (int32 [H][W])
};

struct DescChunk {
    int32_t first, count;
    FrameDesc d[kDescChunk];
};

// Per-component partial record (one per connected piece inside one tile).
// Sums are taken about the reference (x0, y0) = origin of the tile that
// produced the piece:
//   s[0..5]  = sum M, M dx, M dy, M dx^2, M dy^2, M dx dy
//   s[6..11] = the same with unit weights (n, dx, dy, ...)
// Every term added into s[] or acc[] is first rounded to a multiple of a power
// of two (quantum) chosen from exact integer bounds of the sum, so that every
// partial sum is an exact multiple of the quantum within the double range and
// the result does not depend on the order of the additions.  After the merge
// the component's root record holds in acc[] the sums of all its pieces about
// the root's tile origin, in cnpix its pixel count and in camax its max |M|.
struct CompRec {
    double s[12];
    double acc[12];
    int32_t xmin, xmax, ymin, ymax;  // frame coordinates (the component's, at the root)
    uint32_t pmin;                   // raster index of the first pixel in the frame
    uint32_t peak;                   // order-preserving bits of max M
    uint32_t flags;
    int32_t frame;
    int32_t x0, y0;
    uint32_t amax;                   // float bits of the piece's max |M|
    uint32_t camax;                  // float bits of the component's max |M| (root)
    int32_t cnpix;                   // pixels of the component (root)
    int32_t pad[3];
};

// Quantum of a sum bounded by `bound` (sum of |terms| <= bound): 2^e with
// bound < 2^(e + 51), so that the sum of the rounded terms stays an exact
// multiple of 2^e below 2^53 2^e.  Zero bound: every term is zero.
__device__ __forceinline__ int quantum_exp(double bound) {
    if (!(bound > 0.0)) return 0;
    int ex;
    (void)frexp(bound, &ex);   // bound < 2^ex
    return ex - 51;
}
__device__ __forceinline__ double quantize(double v, int e) { return ldexp(rint(ldexp(v, -e)), e); }

struct TileInfo {
    int32_t base;   // first record id (-1 when the tile holds no component)
    int32_t ncomp;
};

// Workspace pointers used by the detection kernels.
struct DetWork {
    FrameDesc* desc;
    int32_t nframes;
    int32_t total_tiles;
    uint32_t* counters;    // [0] records used, [1] overflow flag
    TileInfo* tiles;       // [total_tiles]
    int16_t* edges;        // [total_tiles][4][64]: top, bottom, left, right
    CompRec* recs;         // [rec_cap]
    int32_t* parent;       // [rec_cap]
    int32_t* root;         // [rec_cap]
    int32_t* label;        // [rec_cap]
    uint32_t* blockcnt;    // [total_blocks + 1] bitmap popcounts -> exclusive prefix
    uint32_t* chunksum;    // scan helper
    uint32_t* bitmap;      // all frames' first-pixel bitmaps
    int32_t rec_cap;
    int32_t total_blocks;
    int32_t ahead;         // tiles an XCD's resident workgroups span (the L2 warm-up distance)
    int32_t pad;
};

// ---------------------------------------------------------------------------
// order-preserving float bits (monotone uint32 image of IEEE float)
__device__ __forceinline__ uint32_t f2ord(float f) {
    uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float ord2f(uint32_t u) {
    return __uint_as_float((u & 0x80000000u) ? (u & 0x7fffffffu) : ~u);
}

// ---------------------------------------------------------------------------
// compensated FP32 arithmetic (Knuth two-sum)
struct F2 {
    float hi, lo;
};
__device__ __forceinline__ void two_sum(float a, float b, float& s, float& e) {
    s = a + b;
    float bb = s - a;
    e = (a - (s - bb)) + (b - bb);
}
// running compensated sum of single values
__device__ __forceinline__ void f2_acc(F2& a, float v) {
    float s, e;
    two_sum(a.hi, v, s, e);
    a.hi = s;
    a.lo += e;
}
// Workgroups are handed to the 8 XCDs (each with its own L2) in turn.  With a
// grid of 8 * chunk workgroups, item (blockIdx mod 8) * chunk + blockIdx / 8
// gives each XCD a contiguous run of items, so neighbours that share data
// (tile halos, overlapping apertures) meet in the same L2.  Items >= n: none.
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_item(int block, int chunk) { return (block % kXcds) * chunk + block / kXcds; }

// make one wavefront's LDS writes visible to its other lanes
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

__device__ __forceinline__ double f2_d(F2 a) { return (double)a.hi + (double)a.lo; }

// the value of lane l (uniform), and of the lane a DPP control selects
__device__ __forceinline__ double lane_d(double v, int l) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
    return __longlong_as_double((long long)((uint64_t)lo | ((uint64_t)hi << 32)));
}
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)((uint64_t)lo | ((uint64_t)hi << 32)));
}
__device__ __forceinline__ float lane_f(float v, int l) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// lanes exchanged between the halves of the wavefront (or, 16, of each half),
// added: the low half gets a's sum over the pair, the high half b's
__device__ __forceinline__ double swap_add32(double a, double b) {
    const uint64_t x = (uint64_t)__double_as_longlong(a), y = (uint64_t)__double_as_longlong(b);
    const auto l = __builtin_amdgcn_permlane32_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    return __longlong_as_double((long long)((uint64_t)l[0] | ((uint64_t)h[0] << 32))) +
           __longlong_as_double((long long)((uint64_t)l[1] | ((uint64_t)h[1] << 32)));
}
__device__ __forceinline__ double swap_add16(double a, double b) {
    const uint64_t x = (uint64_t)__double_as_longlong(a), y = (uint64_t)__double_as_longlong(b);
    const auto l = __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false);
    return __longlong_as_double((long long)((uint64_t)l[0] | ((uint64_t)h[0] << 32))) +
           __longlong_as_double((long long)((uint64_t)l[1] | ((uint64_t)h[1] << 32)));
}
// Sums of N (16 or 32) values over the wavefront's lanes, in a fixed order.
// The halves of the wavefront exchange halves of the list, then the 16-lane
// rows quarters of it, so that only N / 4 values are left for the four steps
// inside a row.  total(i) is value i's sum.
template <int N>
struct WaveTotals {
    double v[N / 4];
    __device__ __forceinline__ explicit WaveTotals(const double (&x)[N]) {
        double h[N / 2];
#pragma unroll
        for (int i = 0; i < N / 2; ++i) h[i] = swap_add32(x[i], x[i + N / 2]);   // lanes 32..: value i + N / 2
#pragma unroll
        for (int i = 0; i < N / 4; ++i) {
            double t = swap_add16(h[i], h[i + N / 4]);   // odd rows: value i + N / 4 of the half
            t += dpp_d<0xB1>(t);
            t += dpp_d<0x4E>(t);
            t += dpp_d<0x141>(t);
            t += dpp_d<0x140>(t);
            v[i] = t;
        }
    }
    __device__ __forceinline__ double total(int i) const {
        return lane_d(v[i % (N / 4)], 16 * (((i / (N / 4)) & 1) | (i / (N / 2)) << 1));
    }
};

// ---------------------------------------------------------------------------
// frame lookup by flattened index: the last frame whose base <= idx
template <typename Get>
__device__ __forceinline__ int frame_of(int nframes, int idx, Get base) {
    int lo = 0, hi = nframes - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (base(mid) <= idx) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// the same by a whole wavefront for one index: 64 bases per load (a chain of
// dependent loads otherwise), the bases <= idx being a prefix of them
template <typename Get>
__device__ __forceinline__ int frame_of_wave(int nframes, int idx, Get base) {
    if (nframes == 1) return 0;
    const int lane = threadIdx.x & 63;
    int f = -1;
    for (int i0 = 0; i0 < nframes; i0 += 64) {
        const int i = i0 + lane;
        const uint64_t m = __ballot(i < nframes && base(min(i, nframes - 1)) <= idx);
        f += __popcll(m);
        if (m != ~0ull) break;
    }
    return f;
}

// e / d by a multiplication, for e d < 2^32 and a divisor shared by the
// workgroup (an integer division is some 25 instructions)
struct Div {
    uint32_t d, m;
    __device__ __forceinline__ explicit Div(int n)
        : d((uint32_t)n), m((uint32_t)((((uint64_t)1 << 32) + (uint32_t)n - 1) / (uint32_t)n)) {}
    // (m of 1 does not fit 32 bits)
    __device__ __forceinline__ int operator()(int e) const { return d == 1u ? e : (int)__umulhi((uint32_t)e, m); }
};

// half-sample symmetric reflection into [0, n)
__device__ __forceinline__ int reflect_idx(int i, int n) {
    if (i >= 0 && i < n) return i;
    int p = 2 * n;
    int r = i % p;
    if (r < 0) r += p;
    return (r < n) ? r : (p - 1 - r);
}

// frames live in global memory: address them as such (global_load rather
// than the generic flat path)
typedef __attribute__((address_space(1))) const float gfloat_t;
typedef __attribute__((address_space(1))) const uint16_t gu16_t;
typedef __attribute__((address_space(1))) const double gdouble_t;
typedef __attribute__((address_space(1))) int32_t gi32_t;

__device__ __forceinline__ float load_px(const FrameDesc& d, int x, int y) {
    int64_t off = (int64_t)y * d.pitch + x;
    if (d.dtype == kDtypeU16) return (float)((gu16_t*)d.data)[off];
    return ((gfloat_t*)d.data)[off];
}

// mesh centre ("knot") along an axis and the spline piece holding a pixel:
// piece k spans [c_{k-1}, c_k); piece 0 and piece n extend to the frame edges
__device__ __forceinline__ double knot_at(int k, int n, int m) {
    int a = k * m;
    int b = min(a + m, n);
    return 0.5 * (double)(a + b - 1);
}
__device__ __forceinline__ int piece_of(int p, int n, int m) {
    int k0 = p / m;
    int a = k0 * m;
    int b = min(a + m, n);
    // c_{k0} = (a + b - 1) / 2 ; p >= c_{k0}  <=>  2p >= a + b - 1
    return k0 + ((2 * p >= a + b - 1) ? 1 : 0);
}
__device__ __forceinline__ double piece_ref(int piece, int n, int m) {
    return knot_at(piece > 0 ? piece - 1 : 0, n, m);
}

}  // namespace gpk
