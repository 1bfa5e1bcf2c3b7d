// k_background.hip -- mesh background for gfx950.
//
//  k_mesh_stats   one workgroup per mesh.  The values of a mesh are grouped by
//                 bins in LDS once; a clipping pass then takes the dropped ends
//                 off running sums and finds the median in its bin, all in one
//                 wavefront.  The sums are exact over terms that are whole
//                 numbers (floats: of two fixed units, one far below the
//                 other), so a mesh gives bit-identical results wherever it is
//                 scheduled.
//  k_spline_y_pcr, k_spline_x_pcr (and the *_blk variants)
//                 grids of at most 511 knots per axis: the f x f median over
//                 the mesh grid (truncated at the edges) and the natural cubic
//                 splines through the mesh centres, one wavefront per spline up
//                 to 63 knots on the solved axis, one workgroup with more
//                 threads than knots beyond, solved in FP64 by parallel cyclic
//                 reduction and turned into bicubic pieces per mesh cell.
//  k_grid_filter, k_spline_*
//                 the same for larger grids: one thread per mesh for the
//                 filter, one per spline for the FP64 Thomas solve.
//
// The statistics follow the SExtractor method the paper cites for local
// background estimation; the paper's background subsection fixes the output
// role: a per-pixel background and a per-pixel noise map (here the clipped
// rms, interpolated like the background).
#include "k_args.h"
#include "k_rowpoly.h"

namespace gpk {

// the value of lane ^ J, and the least and the greatest of the lanes' values,
// by DPP and permutes of registers: a shuffle through LDS waits some 100 cycles
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_xor(float v, int j, int lane) {
    if (j == 1) return dpp_f<0xB1>(v);
    if (j == 2) return dpp_f<0x4E>(v);
    if (j == 4) return dpp_f<0x1B>(dpp_f<0x141>(v));   // 7 - lane of each 8, then 3 - lane of each 4
    if (j == 8) return dpp_f<0x128>(v);
    const uint32_t u = __float_as_uint(v);
    if (j == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);   // rows 0 0 2 2 | 1 1 3 3
        return __uint_as_float((lane & 16) ? r[0] : r[1]);
    }
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);   // low low | high high
    return __uint_as_float((lane & 32) ? r[0] : r[1]);
}
__device__ __forceinline__ float wave_least(float v) {
    v = fminf(v, dpp_f<0xB1>(v));
    v = fminf(v, dpp_f<0x4E>(v));
    v = fminf(v, dpp_f<0x141>(v));
    v = fminf(v, dpp_f<0x140>(v));
    return fminf(fminf(lane_f(v, 0), lane_f(v, 16)), fminf(lane_f(v, 32), lane_f(v, 48)));
}
__device__ __forceinline__ float wave_greatest(float v) { return -wave_least(-v); }

// inclusive prefix sums over the lanes
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_from(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ uint32_t wave_prefix(uint32_t v) {
    v += dpp_from<0x111, 0xf>(v);   // 1, 2, 4, 8 lanes down inside a row
    v += dpp_from<0x112, 0xf>(v);
    v += dpp_from<0x114, 0xf>(v);
    v += dpp_from<0x118, 0xf>(v);
    v += dpp_from<0x142, 0xa>(v);   // a row's last lane to the next row (1 and 3)
    v += dpp_from<0x143, 0xc>(v);   // lane 31 to rows 2 and 3
    return v;
}

// Ascending bitonic sort of one value per lane of a wavefront.
__device__ __forceinline__ float wave_sort(float x, int lane) {
#pragma unroll
    for (int k = 2; k <= 64; k <<= 1) {
#pragma unroll
        for (int j = k >> 1; j > 0; j >>= 1) {
            const float o = lane_xor(x, j, lane);
            const bool up = (lane & k) == 0, lower = (lane & j) == 0;
            x = (lower == up) ? fminf(x, o) : fmaxf(x, o);
        }
    }
    return x;
}

// (read back as 16-bit halves)
typedef uint32_t __attribute__((may_alias)) word16_t;

// The mesh's values in LDS, grouped by bin, for a workgroup of NT threads with
// PPT pixels each.
//   val    the values, bin after bin (any order inside a bin)
//   start  first position of each bin (two 16-bit numbers per word: at most
//          16384 pixels), start[NB] = their number
//   w*     the wavefronts' sums, ranges and counts
template <typename T, int NT, int PPT>
struct MeshShared {
    static constexpr int NB = (NT * PPT <= 1024) ? 512 : (NT * PPT <= 8192) ? 2048 : 4096;
    static constexpr bool kInt = sizeof(T) == 2;
    T val[NT * PPT];
    word16_t start[NB / 2 + 1];
    double w1[NT / 64], wu[NT / 64], wh[NT / 64], wl[NT / 64];
    uint32_t wc[NT / 64];
    float wmin[NT / 64], wmax[NT / 64];
    float lo, scale, mid;
    uint32_t part[128];  // a large bin's parts (and an unused word per lane), or the values of one part
};

// Bins of a mesh: three quarters of them equal steps from lo on, the rest
// eight to the octave above (a star's wings and its saturated core spread
// over several).  A rising function of the value, whatever lo and scale are:
// these only decide how many values share a bin, never a result.
template <int NB>
__device__ __forceinline__ int mesh_bin(float x, float lo, float scale) {
#pragma clang fp contract(off)   // the same bin for a value wherever this is inlined
    constexpr int NC = NB - NB / 4;
    const float t = (x - lo) * scale;
    const int core = (int)fminf(fmaxf(t, 0.0f), (float)NC);
    const float u = fmaxf(t - (float)(NC - 1), 1.0f);
    const int tail = NC + ((__float_as_int(u) - 0x3f800000) >> 20);
    return t >= (float)NC ? min(tail, NB - 1) : core;
}

// sum over the wavefront's lanes (of values whose sums are exact: any order)
__device__ __forceinline__ double wave_total(double v) {
    v += dpp_d<0xB1>(v);    // lane ^ 1
    v += dpp_d<0x4E>(v);    // lane ^ 2
    v += dpp_d<0x141>(v);   // 7 - lane of each 8
    v += dpp_d<0x140>(v);   // 15 - lane of each 16
    return (lane_d(v, 0) + lane_d(v, 16)) + (lane_d(v, 32) + lane_d(v, 48));
}
// order-preserving integers of a pixel's values
template <typename T>
__device__ __forceinline__ uint32_t mesh_image(float x) { return sizeof(T) == 2 ? (uint32_t)x : f2ord(x); }
template <typename T>
__device__ __forceinline__ float mesh_value(uint32_t z) { return sizeof(T) == 2 ? (float)z : ord2f(z); }

// Of up to 64 values, one per lane (the lanes past m hold +inf): how many are
// smaller than the lane's, and the one with j smaller ones (or, among equals,
// fewer).
__device__ __forceinline__ int wave_rank(float x, int m) {
    int q = 0;
    for (int i = 0; i < m; i += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) q += lane_f(x, i + u) < x ? 1 : 0;
    }
    return q;
}
__device__ __forceinline__ float wave_kth(float x, int q, int m, int j) {
    const int lane = threadIdx.x & 63;
    uint64_t hit;
    while ((hit = __ballot(lane < m && q == j)) == 0ull) --j;
    return lane_f(x, __builtin_ctzll(hit));
}

// The values of rank j and j + 1 (+inf if there is none) of the m > 256 values
// of a bin, by one wavefront.  A value that many of them share (masked,
// clipped or saturated pixels) is tried first: a pass that counts it and the
// smaller ones.  Else their range is split into 64 equal parts of the
// order-preserving integers and the part that holds rank j counted out, until
// it has at most 64 values: a pass for the range, and one or two for the parts,
// where bisection takes 16 to 32.  The counts of the part that most of a few
// probes fall into stay in registers (an LDS atomic costs 4 cycles for each
// lane of the same address).  Called, not inlined: few meshes have such bins,
// and its registers would cost all of them wavefronts.  With the bins from a
// third of the sampled pixels, 2048^2 float in 128^2 meshes: 40% of the pixels
// zero 329 us by bisection, now 27; 40% saturated 319, now 27; half zero and
// the rest noise above zero (19 passes) 6867, now 224.
template <typename T>
using lds_t = __attribute__((address_space(3))) T;
template <typename T>
__device__ __attribute__((noinline)) float2 mesh_large_bin(const lds_t<T>* val, lds_t<uint32_t>* part, int m, int j) {
    const int lane = threadIdx.x & 63;
    // every value of the bin, four loads in flight
    auto each = [&](auto&& f) __attribute__((always_inline)) {
        int i = lane;
        for (; i - lane + 256 <= m; i += 256) {
            T x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = val[i + 64 * u];
#pragma unroll
            for (int u = 0; u < 4; ++u) f(mesh_image<T>((float)x[u]));
        }
        for (; i < m; i += 64) f(mesh_image<T>((float)val[i]));
    };
    // the most frequent of four probes among 64 of the values, if 9 or more share it
    const auto frequent = [&](uint32_t z, uint32_t none) __attribute__((always_inline)) {
        int most = 8;
        uint32_t best = none;
        for (int l = 0; l < 64; l += 16) {
            const uint32_t q = (uint32_t)__builtin_amdgcn_readlane((int)z, l);
            const int c = __popcll(__ballot(z == q));
            if (c > most) {
                best = q;
                most = c;
            }
        }
        return best;
    };
    const uint32_t first = mesh_image<T>((float)val[lane]);
    uint32_t a0 = 0u, a1 = ~0u;
    int mm = m, before = 0;   // values in [a0, a1], of which the one of rank j is sought
    const uint32_t shared = frequent(first, ~0u);
    if (shared != ~0u) {
        uint32_t n = 0u;   // smaller ones, equal ones << 16
        each([&](uint32_t z) __attribute__((always_inline)) { n += z < shared ? 1u : z == shared ? 0x10000u : 0u; });
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) n += (uint32_t)__shfl_xor((int)n, d);
        const int lt = __builtin_amdgcn_readfirstlane((int)(n & 0xffffu)), eq = __builtin_amdgcn_readfirstlane((int)(n >> 16));
        if (j >= lt && j < lt + eq) {
            a0 = a1 = shared;
            j -= lt;
            mm = eq;
        }
    }
    while (a0 != a1) {
        if (4 * mm > before) {
            // (at first, and where the last parts hardly split the values: one
            // value many times, or a range with few values at its ends)
            uint32_t z0 = ~0u, z1 = 0u;
            each([&](uint32_t z) __attribute__((always_inline)) {
                z0 = min(z0, z >= a0 ? z : ~0u);
                z1 = max(z1, z <= a1 ? z : 0u);
            });
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1) {
                z0 = min(z0, (uint32_t)__shfl_xor((int)z0, o));
                z1 = max(z1, (uint32_t)__shfl_xor((int)z1, o));
            }
            a0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)z0);
            a1 = (uint32_t)__builtin_amdgcn_readfirstlane((int)z1);
        }
        if (a0 == a1 || mm <= 64) break;
        before = mm;
        const int sft = max(0, 26 - __clz((int)(a1 - a0)));
        const uint32_t probe = (first - a0) >> sft;   // (past the range: above 63)
        const uint32_t hot = frequent(min(probe, 64u), 64u);
        part[lane] = 0u;
        wave_sync();
        int mine = 0;
        each([&](uint32_t z) __attribute__((always_inline)) {
            const uint32_t q = (z - a0) >> sft;
            const bool in = z >= a0 && z <= a1;
            atomicAdd((uint32_t*)&part[in && q != hot ? q : 64u + lane], 1u);
            mine += in && q == hot ? 1 : 0;
        });
        wave_sync();
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) mine += __shfl_xor(mine, d);
        const int c = (int)part[lane] + ((uint32_t)lane == hot ? mine : 0);
        const int incl = (int)wave_prefix((uint32_t)c);
        const int q = __builtin_ctzll(__ballot(incl > j));
        mm = __builtin_amdgcn_readlane(c, q);
        j -= __builtin_amdgcn_readlane(incl, q) - mm;
        a0 += (uint32_t)q << sft;
        a1 = min(a1, a0 + ((1u << sft) - 1u));
        wave_sync();
    }
    float x1 = mesh_value<T>(a0), x2 = x1;
    if (a0 != a1) {
        part[64] = 0u;   // the number found so far
        wave_sync();
        each([&](uint32_t z) __attribute__((always_inline)) {
            if (z >= a0 && z <= a1) part[atomicAdd((uint32_t*)&part[64], 1u)] = z;
        });
        wave_sync();
        const float x = lane < mm ? mesh_value<T>(part[lane]) : INFINITY;
        wave_sync();
        const int q = wave_rank(x, mm);
        x1 = wave_kth(x, q, mm, j);
        if (j + 1 < mm) x2 = wave_kth(x, q, mm, j + 1);
    }
    if (j + 1 >= mm) {
        // the next value lies above the part
        x2 = INFINITY;
        each([&](uint32_t z) __attribute__((always_inline)) { x2 = z > a1 ? fminf(x2, mesh_value<T>(z)) : x2; });
        x2 = wave_least(x2);
    }
    return make_float2(x1, x2);
}

// One workgroup per mesh.  Whatever was clipped before, the surviving values
// are always those of one interval [L, H).  The workgroup groups the values by
// bin in LDS once (a histogram whose returned counts are the places inside a
// bin, a prefix sum, one store per value); then one wavefront runs the whole
// clipping loop.  A pass reads only the bins between the old and the new ends
// of the interval, to take the values it drops off the sums, and the bin that
// holds the median: no barrier and no pass over the pixels per iteration, and
// the other wavefronts have left.
//
// The places inside a bin follow the order of the LDS atomics, so every sum
// is made exact, hence independent of that order: uint16 values give integer
// sums below 2^53; a float's (v - c) and its square are each taken as a
// multiple of 2^-38 and the rest as a multiple of 2^-76 of the range (of its
// square), whose sums all stay below 2^53 units (16384 pixels).  A value so
// loses less than in FP64 sums of plain products; where sigma has fallen
// 2^20 times below that range (a no-data value among the pixels was clipped),
// or the mean lies 2^10 sigmas from c, the survivors are summed anew about
// their median, in units of their own range.  A mesh gives bit-identical
// results wherever it runs.
//
// Bound by latency: loads, the histogram's LDS atomics, scan and stores, then
// a chain of 3-14 clipping passes in one wavefront.  What hides it is meshes
// per CU: 7 of 64^2, two of 128^2 (74 KB of LDS).
// A pass over all pixels in registers per iteration, with a sorted window for
// the median (float) or prefix sums of a histogram (uint16), took: 12300^2
// crowded float in 128^2 meshes 2222 us, now 1067; 6144^2 260, now 143;
// 2048^2 in 64^2 meshes 40, now 24; 371 MP of uint16 1122, now 645.  (Floats
// with one part of 2^-38 and no second: 981, 131 and 22.)
//
// ONE: a one-frame call, whose descriptor comes with the launch (d1);
// workgroup 0 stores it in the table for the launches that follow.
// (Registers for seven wavefronts per SIMD up to 8192 pixels; nothing spilled to
// memory.)
template <typename T, int NT, int PPT, bool ONE>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(NT * PPT > 8192 ? 4 : 7))) void k_mesh_stats(FrameDesc* __restrict__ desc, FrameDesc d1, int nframes,
                                                   BkgArgs a) {
    using SH = MeshShared<T, NT, PPT>;
    constexpr bool kInt = SH::kInt;
    constexpr int NB = SH::NB, NW = NT / 64;
    __shared__ SH sh;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int gm = blockIdx.x;
    if (ONE && gm == 0 && tid == 0) desc[0] = d1;
    const int f = ONE ? 0 : frame_of_wave(nframes, gm, [&](int i) { return desc[i].mesh_base; });
    const FrameDesc d = ONE ? d1 : desc[f];
    if ((d.dtype == kDtypeU16) != kInt) return;   // the other kernel's mesh of a mixed batch
    const int lm = gm - d.mesh_base;
    const int mi = lm % d.nx, mj = lm / d.nx;
    const int x0 = mi * d.mw, y0 = mj * d.mh;
    const int w = min(d.mw, d.W - x0), h = min(d.mh, d.H - y0);
    const int n = w * h;
    const int out_idx = mj * d.nx + mi;

    // 1. pixel k * NT + tid of the mesh in registers.  A full mesh whose width
    //    divides NT puts every thread's k-th pixel dy = NT / w rows below its
    //    previous one: buffer loads with the row step as a scalar offset.
    //    Other meshes step by NT without divisions.
    float v[PPT];
    {
        typedef __attribute__((address_space(1))) const T gpx_t;
        const int dy = NT / w, dx = NT - dy * w;
        int yy = tid / w, xx = tid - yy * w;
        // (byte offsets within the mesh must fit the 32-bit buffer offsets)
        if (n == NT * PPT && dx == 0 && (int64_t)h * d.pitch * (int)sizeof(T) < ((int64_t)1 << 31)) {
            const int64_t o0 = ((int64_t)y0 * d.pitch + x0) * (int)sizeof(T);
            const __amdgpu_buffer_rsrc_t rs =
                __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)d.data + o0), (short)0, 0x7fffffff, 0x00020000);
            const int vo = (yy * (int)d.pitch + xx) * (int)sizeof(T);
            const int so = dy * (int)d.pitch * (int)sizeof(T);
#pragma unroll
            for (int k = 0; k < PPT; ++k)
                v[k] = kInt ? (float)__builtin_amdgcn_raw_buffer_load_b16(rs, vo, k * so, 0)
                            : __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs, vo, k * so, 0));
        } else {
            const gpx_t* src = (const gpx_t*)d.data;
#pragma unroll
            for (int k = 0; k < PPT; ++k) {
                v[k] = NAN;   // padding (pixel values are finite)
                if (k * NT + tid < n) v[k] = (float)src[(int64_t)(y0 + yy) * d.pitch + x0 + xx];
                xx += dx;
                yy += dy;
                if (xx >= w) {
                    xx -= w;
                    ++yy;
                }
            }
        }
    }
    // 2. the mesh's range, and the bins from 64 of its pixels (one per lane of
    //    the first wavefront, at different heights): the shortest interval with
    //    a third of them gives the sky's level and width even where stars, or
    //    masked or saturated pixels of one value, cover half the mesh
    float mn = INFINITY, mx = -INFINITY;
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        mn = fminf(mn, v[k]);   // (NaN is passed over)
        mx = fmaxf(mx, v[k]);
    }
    mn = wave_least(mn);
    mx = wave_greatest(mx);
    for (int b = tid; b < NB / 2; b += NT) sh.start[b] = 0u;
    if (lane == 0) {
        sh.wmin[wv] = mn;
        sh.wmax[wv] = mx;
    }
    if (wv == 0) {
        // (spread over the pixels the lane has: all of the 64 in a narrow mesh too)
        const int at = (lane * ((n - min(lane, n - 1) + NT - 1) / NT)) >> 6;
        float s = v[0];
#pragma unroll
        for (int k = 1; k < PPT; ++k)
            if (at == k) s = v[k];
        const uint64_t have = __ballot(s == s);   // (lane 0 always has its first pixel)
        s = wave_sort(s == s ? s : INFINITY, lane);
        const int m = __popcll(have);
        constexpr float NC = (float)(NB - NB / 4);
        const int third = (m - 1) / 3;
        const float up = __shfl(s, min(lane + third, 63)), mid = __shfl(s, min(lane + third / 2, 63));
        // (not one that reaches from pixels of one value to a few others)
        const float wide = lane + third < m && up > mid && mid > s ? up - s : INFINITY;
        const float least = wave_least(wide);
        float q50 = lane_f(s, (m - 1) / 2);
        float wd = 0.0f;
        if (least < INFINITY) {
            // (the shortest of 64 normal values: 0.4 to 0.9 sigma)
            wd = 1.5f * least;
            q50 = lane_f(s, __builtin_ctzll(__ballot(wide == least)) + third / 2);
        }
        if (lane == 0) sh.mid = q50;
        if (kInt) {
            // steps of one unit where the sky's range leaves room for them:
            // such a bin holds one value
            wd = fmaxf(wd, 1.0f);
            if (lane == 0) {
                sh.lo = floorf(q50 - 6.0f * wd);
                sh.scale = fminf(1.0f, NC / (14.0f * wd));
            }
        } else if (lane == 0) {
            if (!(wd > 0.0f)) wd = fmaxf(fabsf(q50) * 0x1p-10f, 0x1p-100f);
            sh.lo = q50 - 6.0f * wd;
            sh.scale = NC / (14.0f * wd);
        }
    }
    __syncthreads();
    // (what all lanes share goes to scalar registers here and below)
    const float blo = lane_f(sh.lo, 0), bscale = lane_f(sh.scale, 0);
    mn = sh.wmin[0];
    mx = sh.wmax[0];
#pragma unroll
    for (int i = 1; i < NW; ++i) {
        mn = fminf(mn, sh.wmin[i]);
        mx = fmaxf(mx, sh.wmax[i]);
    }
    mn = lane_f(mn, 0);
    mx = lane_f(mx, 0);
    if (mn == mx) {
        if (tid == 0) {
            d.back_raw[out_idx] = (double)mn;
            d.rms_raw[out_idx] = 0.0;
            d.iters[out_idx] = 0;
        }
        return;
    }
    // 3. group by bin: (bin, place inside it) of every pixel, the sums of all
    //    pixels, bin starts, store.  cs: a value of the mesh near the sky
    //    level; mg, mq and ng, nq, 2^-38 of each: adding and taking off 1.5 *
    //    2^52 units rounds to a whole number of units (all in scalar registers).
    double cs = lane_d((double)sh.mid, 0), mg, mq, ng, nq;
    auto units = [&](double range) __attribute__((always_inline)) {
        int ex;
        (void)frexp(range, &ex);
        ex = __builtin_amdgcn_readfirstlane(ex);
        mg = lane_d(ldexp(1.5, ex - 38 + 52), 0);
        mq = lane_d(ldexp(1.5, 2 * ex - 38 + 52), 0);
        ng = lane_d(ldexp(1.5, ex - 76 + 52), 0);
        nq = lane_d(ldexp(1.5, 2 * ex - 76 + 52), 0);
        return ex;
    };
    const int ex0 = units(fmax((double)mx - cs, cs - (double)mn));
    auto accum = [&](double e, double& s1, double& su, double& sq, double& sl) __attribute__((always_inline)) {
        if (kInt) {
            s1 += e;
            sq = fma(e, e, sq);
        } else {
            const double h1 = (e + mg) - mg, hq = fma(e, e, mq) - mq;
            s1 += h1;
            su += ((e - h1) + ng) - ng;
            sq += hq;
            sl += (fma(e, e, -hq) + nq) - nq;
        }
    };
    double t1 = 0.0, tu = 0.0, th = 0.0, tl = 0.0;
    // Positive floats that lie within 2^14 of each other's size (a sky with its
    // level and its stars): each (v - c) is itself a multiple of 2^-38 of the
    // range, so its sum needs no parts, and the rest of its square no rounding;
    // the same sums by 7 FP64 operations a pixel for 15.
    int en;
    (void)frexp(mn, &en);
    const bool plain = !kInt && mn > 0.0f && mx < INFINITY && ex0 - __builtin_amdgcn_readfirstlane(en) <= 14;
    // (four pixels of a thread at a time: a small mesh has no others)
    auto sums = [&](auto&& add) __attribute__((always_inline)) {
#pragma unroll
        for (int k0 = 0; k0 < PPT; k0 += 4) {
            if (k0 * NT >= n) break;
#pragma unroll
            for (int k = k0; k < k0 + 4; ++k) add(v[k] == v[k] ? (double)v[k] - cs : 0.0);
        }
    };
    if (plain) {
        sums([&](double e) __attribute__((always_inline)) {
            const double hq = fma(e, e, mq) - mq;
            t1 += e;
            th += hq;
            tl += fma(e, e, -hq);
        });
    } else if (!kInt) {
        sums([&](double e) __attribute__((always_inline)) { accum(e, t1, tu, th, tl); });
    }
    uint32_t pk[PPT];
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        pk[k] = 0u;
        if (v[k] == v[k]) {
            const uint32_t b = (uint32_t)mesh_bin<NB>(v[k], blo, bscale);
            const uint32_t sft = (b & 1u) * 16u;
            const uint32_t old = atomicAdd((uint32_t*)&sh.start[b >> 1], 1u << sft);
            pk[k] = (b << 16) | ((old >> sft) & 0xffffu);
            if (kInt) accum((double)v[k] - cs, t1, tu, th, tl);
        }
    }
    t1 = wave_total(t1);
    th = wave_total(th);
    if (!kInt) {
        tu = wave_total(tu);
        tl = wave_total(tl);
    }
    if (lane == 0) {
        sh.w1[wv] = t1;
        sh.wu[wv] = tu;
        sh.wh[wv] = th;
        sh.wl[wv] = tl;
    }
    __syncthreads();
    {
        constexpr int PER = (NB / 2 + NT - 1) / NT;   // words of two bins per thread
        uint32_t c[PER], tot = 0u;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int i = tid * PER + q;
            c[q] = (i < NB / 2) ? sh.start[i] : 0u;
            tot += (c[q] & 0xffffu) + (c[q] >> 16);
        }
        const uint32_t incl = wave_prefix(tot);
        if (lane == 63) sh.wc[wv] = incl;
        __syncthreads();
        uint32_t run = incl - tot;
#pragma unroll
        for (int i = 0; i < NW - 1; ++i) run += (i < wv) ? sh.wc[i] : 0u;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int i = tid * PER + q;
            const uint32_t s1 = run + (c[q] & 0xffffu);
            if (i < NB / 2) sh.start[i] = run | (s1 << 16);
            run = s1 + (c[q] >> 16);
        }
        if (tid == 0) sh.start[NB / 2] = (uint32_t)n;
    }
    __syncthreads();
    const uint16_t* start = reinterpret_cast<const uint16_t*>(sh.start);
#pragma unroll
    for (int k = 0; k < PPT; ++k)
        if (v[k] == v[k]) sh.val[start[pk[k] >> 16] + (pk[k] & 0xffffu)] = (T)v[k];
    __syncthreads();
    if (wv != 0) return;
    if (!kInt) {
        // a pixel that is not a number lies in no bin: no statistics
        uint32_t binned = 0u;
#pragma unroll
        for (int i = 0; i < NW; ++i) binned += sh.wc[i];
        if (binned != (uint32_t)n) {
            if (lane == 0) {
                d.back_raw[out_idx] = (double)NAN;
                d.rms_raw[out_idx] = 0.0;
                d.iters[out_idx] = 0;
            }
            return;
        }
    }
    __builtin_amdgcn_s_setprio(3);   // one wavefront's chain of latencies from here on
    t1 = sh.w1[0];
    tu = sh.wu[0];
    th = sh.wh[0];
    tl = sh.wl[0];
#pragma unroll
    for (int i = 1; i < NW; ++i) {
        t1 += sh.w1[i];
        tu += sh.wu[i];
        th += sh.wh[i];
        tl += sh.wl[i];
    }
    t1 = lane_d(t1, 0);
    tu = lane_d(tu, 0);
    th = lane_d(th, 0);
    tl = lane_d(tl, 0);
    // 4. the clipping loop (one wavefront; every branch below is uniform)
    const int half = lane >> 5, hl = lane & 31;
    int ncur = n, rank0 = 0;              // surviving values, and how many lie below them
    // survivors: L <= v < H (at first the whole range, so that an end that
    // stays beyond it reads no bin)
    float L = mn, H = kInt ? mx + 1.0f : mx < INFINITY ? ord2f(f2ord(mx + 0.0f) + 1u) : INFINITY;   // (past +0 for -0)
    int pL = 0, pH = n;                   // positions of the bins that hold them
    constexpr int G = NB / 64;
    const int top = start[lane * G];      // every G-th bin start
    float med_h = 0.0f, med_l = 0.0f;     // median (an unevaluated pair: exact)
    double mean = 0.0, sig = 0.0, sig0 = 0.0;
    int iters = 0;
    for (;; ++iters) {
        // mean and standard deviation
        const double nd = (double)ncur;
        if (kInt) {
            // n^2 var = n S2 - S1^2 in 64-bit integers (< 2^61); the mean
            // from the sum about the minimum
            const int64_t i1 = (int64_t)t1;
            const int64_t num = (int64_t)ncur * (int64_t)th - i1 * i1;
            sig = sqrt((double)num / (nd * nd));
            mean = (double)mn + (t1 + nd * (cs - (double)mn)) / nd;
        } else {
            double q1 = (t1 + tu) / nd, vv = (th + tl) / nd - q1 * q1;
            bool flat = false;
            // sigma below 2^-20 of the sums' range (mq: 1.5 * 2^14 of its
            // square) or 2^-10 of the mean's distance from cs, or one value only
            if (vv <= fmax(mq * (0x1p-54 / 1.5), 0x1p-20 * (q1 * q1))) {
                float lmn = INFINITY, lmx = -INFINITY;
                for (int i = pL + lane; i < pH; i += 64) {
                    const float x = (float)sh.val[i];
                    if (x >= L && x < H) {
                        lmn = fminf(lmn, x);
                        lmx = fmaxf(lmx, x);
                    }
                }
                lmn = wave_least(lmn);
                lmx = wave_greatest(lmx);
                flat = lmn == lmx;
                cs = lane_d((double)fminf(fmaxf(iters > 0 ? med_h : (float)(cs + q1), lmn), lmx), 0);
                t1 = tu = th = tl = 0.0;
                if (!flat) {
                    units(fmax((double)lmx - cs, cs - (double)lmn));
                    for (int i = pL + lane; i < pH; i += 64) {
                        const float x = (float)sh.val[i];
                        if (x >= L && x < H) accum((double)x - cs, t1, tu, th, tl);
                    }
                    t1 = lane_d(wave_total(t1), 0);
                    tu = lane_d(wave_total(tu), 0);
                    th = lane_d(wave_total(th), 0);
                    tl = lane_d(wave_total(tl), 0);
                }
                q1 = (t1 + tu) / nd;
                vv = (th + tl) / nd - q1 * q1;
            }
            mean = cs + q1;
            sig = vv > 0.0 && !flat ? sqrt(vv) : 0.0;
        }
        mean = lane_d(mean, 0);
        sig = lane_d(sig, 0);
        if (iters == 0) sig0 = sig;
        // the median: the bin of its rank (bins start at rising positions),
        // then the order statistic inside the bin
        {
            const int r2 = rank0 + ncur / 2, r1 = (ncur & 1) ? r2 : r2 - 1;
            float o0 = 0.0f, o1 = 0.0f;   // (no array: an index at run time puts it in scratch memory)
            int have = 0;
#pragma unroll 1
            while (have < 2) {
                const int r = have ? r2 : r1;
                const int g = __popcll(__ballot(top <= r)) - 1;
                const int in = start[g * G + 1 + (G == 64 ? lane : min(lane, G - 1))];   // ends of its bins
                const int k = __popcll(__ballot(lane < G && in <= r));
                const int b = g * G + k;
                const int e = __builtin_amdgcn_readlane(in, k);
                const int s = __builtin_amdgcn_readlane(k > 0 ? in : top, k > 0 ? k - 1 : g);
                const int m = e - s, j = r - s;
                const bool both = r2 < e;   // the upper middle value lies here too
                float x1, x2;               // the values of rank r and, if it lies here, r2
                if (kInt && bscale == 1.0f && b > 0 && b < NB - NB / 4) {
                    x1 = x2 = blo + (float)b;   // a bin of one value
                } else if (m <= 64) {
                    // the value with j smaller ones (or, among equals, fewer)
                    const float x = (lane < m) ? (float)sh.val[s + lane] : INFINITY;
                    const int q = wave_rank(x, m);
                    x1 = x2 = wave_kth(x, q, m, j);
                    if (both && r2 != r) x2 = wave_kth(x, q, m, j + 1);
                } else if (m <= 256) {
                    // the smallest value with more than j at or below it, by
                    // bisection, and the next one up
                    float y[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) y[u] = (lane + 64 * u < m) ? (float)sh.val[s + lane + 64 * u] : INFINITY;
                    auto upto = [&](float x) {
                        int c = 0;
#pragma unroll
                        for (int u = 0; u < 4; ++u) c += __popcll(__ballot(y[u] <= x));
                        return c;
                    };
                    uint32_t a0 = mesh_image<T>(mn), a1 = mesh_image<T>(mx);
                    while (a0 < a1) {
                        const uint32_t mid = a0 + ((a1 - a0) >> 1);
                        if (upto(mesh_value<T>(mid)) > j) a1 = mid;
                        else a0 = mid + 1;
                    }
                    x1 = x2 = mesh_value<T>(a0);
                    if (both && r2 != r && upto(x1) == j + 1) {
                        x2 = INFINITY;
#pragma unroll
                        for (int u = 0; u < 4; ++u) x2 = y[u] > x1 ? fminf(x2, y[u]) : x2;
                        x2 = wave_least(x2);
                    }
                } else {
                    const float2 x = mesh_large_bin<T>((const lds_t<T>*)&sh.val[s], (lds_t<uint32_t>*)sh.part, m, j);
                    x1 = x.x;
                    x2 = (r2 == r) ? x.x : x.y;
                }
                if (!have) o0 = x1;
                o1 = have ? x1 : x2;
                have = both ? 2 : have + 1;
            }
            if (r1 == r2) {
                med_h = o0;
                med_l = 0.0f;
            } else {
                float s, e;
                two_sum(o0, o1, s, e);
                med_h = 0.5f * s;
                med_l = 0.5f * e;
            }
        }
        if (iters >= a.max_iter) break;
        // the new ends of the interval
        float Ln, Hn;
        if (kInt) {
            // the integers with |v - med| <= lim (the differences are exact;
            // the bounds from FP64 are nudged to the exact decision)
            const double med = (double)med_h + (double)med_l, lim = (double)a.clip * sig;
            double cl = fmax(ceil(med - lim), (double)mn), ch = fmin(floor(med + lim), (double)mx);
            while (cl - 1.0 >= (double)mn && med - (cl - 1.0) <= lim) cl -= 1.0;
            while (cl <= (double)mx && med - cl > lim) cl += 1.0;
            while (ch + 1.0 <= (double)mx && (ch + 1.0) - med <= lim) ch += 1.0;
            while (ch >= (double)mn && ch - med > lim) ch -= 1.0;
            Ln = (float)cl;
            Hn = (float)(ch + 1.0);
        } else {
            // a value is kept when |(v - med_h) - med_l| <= thr in FP32; the
            // difference rises with v, so the first value kept and the first
            // dropped above are found among 32 neighbours of med -+ thr (one
            // end per half of the wavefront), else by bisection
            const float thr = (float)((double)a.clip * sig);
            auto on = [&](float x) {
                const float dx = (x - med_h) - med_l;
                return half ? dx > thr : dx >= -thr;
            };
            const double md = (double)med_h + (double)med_l;
            const float g = (float)(half ? md + (double)thr : md - (double)thr);
            const uint32_t k0 = f2ord(g) - 16u;
            const uint64_t bm = __ballot(fabsf(g) < 1e38f && on(ord2f(k0 + (uint32_t)hl)));
            const int pc0 = __popcll(bm & 0xffffffffull), pc1 = __popcll(bm >> 32);
            float t;
            if (pc0 > 0 && pc0 < 32 && pc1 > 0 && pc1 < 32) {
                t = ord2f(k0 + 32u - (uint32_t)(half ? pc1 : pc0));
            } else {
                uint32_t z0 = f2ord(-3.402823466e38f), z1 = f2ord(INFINITY);
                for (int s = 0; s < 32; ++s) {
                    const uint32_t mid = z0 + ((z1 - z0) >> 1);
                    const bool yes = z0 < z1 && on(ord2f(mid));
                    if (yes) z1 = mid;
                    else if (z0 < z1) z0 = mid + 1;
                }
                t = ord2f(z0);
            }
            Ln = lane_f(t, 0);
            Hn = lane_f(t, 32);
        }
        Ln = lane_f(fmaxf(L, Ln), 0);
        Hn = lane_f(fminf(H, Hn), 0);
        if (!(Ln < Hn)) {   // nothing left
            ++iters;
            break;
        }
        // what leaves, [L, Ln) and [Hn, H): the positions of the bins from
        // one end of each range to the other, taken as one run
        const int bL = mesh_bin<NB>(Ln, blo, bscale), bH = mesh_bin<NB>(Hn, blo, bscale);
        const int sL = start[bL], sH = start[bH], eH = start[bH + 1];
        // (an end that has not moved drops nothing: its bin may be a large one)
        const int nl = Ln > L ? (int)start[bL + 1] - pL : 0, run = nl + (Hn < H ? pH - sH : 0);
        double s1 = 0.0, su = 0.0, sq = 0.0, sl = 0.0;
        int low = 0, gone = 0;
        // (a value that stays adds an exact zero: no branch for a chain of FP64
        // additions to wait at)
        auto drop = [&](float x, int i) __attribute__((always_inline)) {
            const bool lo = i < nl && x >= L && x < Ln;
            const bool hi = i >= nl && i < run && x >= Hn && x < H;
            const uint64_t bl = __ballot(lo), bh = __ballot(hi);
            low += __popcll(bl);
            gone += __popcll(bl | bh);
            accum(lo || hi ? (double)x - cs : 0.0, s1, su, sq, sl);
        };
        int i0 = 0;
        for (; i0 + 256 <= run; i0 += 256) {
            float x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = i0 + 64 * u + lane;
                x[u] = (float)sh.val[i < nl ? pL + i : sH + (i - nl)];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) drop(x[u], i0 + 64 * u + lane);
        }
        for (; i0 < run; i0 += 64) {
            const int i = min(i0 + lane, run - 1);
            drop((float)sh.val[i < nl ? pL + i : sH + (i - nl)], i0 + lane);
        }
        if (gone == 0 || gone == ncur) {
            ++iters;
            break;
        }
        t1 = lane_d(t1 - wave_total(s1), 0);
        th = lane_d(th - wave_total(sq), 0);
        if (!kInt) {
            tu = lane_d(tu - wave_total(su), 0);
            tl = lane_d(tl - wave_total(sl), 0);
        }
        ncur -= gone;
        rank0 += low;
        L = Ln;
        H = Hn;
        pL = sL;
        pH = eH;
    }
    if (lane == 0) {
        const double med = (double)med_h + (double)med_l;
        const double dsig = fabs(sig - sig0);
        const double back = (dsig < (double)a.crowd * sig0) ? mean
                                                             : ((double)a.mode_a * med - (double)a.mode_b * mean);
        d.back_raw[out_idx] = back;
        d.rms_raw[out_idx] = sig;
        d.iters[out_idx] = iters;
    }
}

// ---------------------------------------------------------------------------
// f x f median over the mesh grid, back and rms separately
// median of w[0], w[S], ..., w[(n-1) S] (insertion sort in place)
__device__ double median_small(double* w, int n, int S) {
    for (int i = 1; i < n; ++i) {
        const double x = w[i * S];
        int j = i - 1;
        while (j >= 0 && w[j * S] > x) {
            w[(j + 1) * S] = w[j * S];
            --j;
        }
        w[(j + 1) * S] = x;
    }
    return (n & 1) ? w[(n / 2) * S] : 0.5 * (w[(n / 2 - 1) * S] + w[(n / 2) * S]);
}

// median of the first n of w[0, N) (the rest +inf) by rank counting: the value
// of rank k has k smaller values (equal ones ranked by position)
template <int N>
__device__ __forceinline__ double median_regs(const double (&w)[N], int n) {
    const int k1 = (n - 1) / 2, k2 = n / 2;
    double a = 0.0, b = 0.0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        int r = 0;
#pragma unroll
        for (int j = 0; j < N; ++j) r += (w[j] < w[i] || (w[j] == w[i] && j < i)) ? 1 : 0;
        a = (r == k1) ? w[i] : a;
        b = (r == k2) ? w[i] : b;
    }
    return (n & 1) ? a : 0.5 * (a + b);
}

// one thread per mesh.  F > 0: the F x F window in registers (all loads in
// flight); F == 0: any size, the window in the thread's own LDS column
constexpr int kGridThreads = 64;
template <int F>
__global__ __launch_bounds__(kGridThreads) void k_grid_filter(const FrameDesc* __restrict__ desc, int nframes,
                                                              int total, int fsize) {
    __shared__ double w[(F > 0) ? 1 : 49 * kGridThreads];
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= total) return;
    const int f = frame_of(nframes, g, [&](int i) { return desc[i].mesh_base; });
    const FrameDesc& d = desc[f];
    const int lm = g - d.mesh_base;
    const int i = lm % d.nx, j = lm / d.nx;
    const int hh = (F > 0) ? F / 2 : fsize / 2;
    if constexpr (F > 0) {
        double wb[F * F], wr[F * F];
        int n = 0;
#pragma unroll
        for (int e = 0; e < F * F; ++e) {
            const int b = j - hh + e / F, c = i - hh + e % F;
            const bool in = b >= 0 && b < d.ny && c >= 0 && c < d.nx;
            wb[e] = in ? d.back_raw[b * d.nx + c] : INFINITY;
            wr[e] = in ? d.rms_raw[b * d.nx + c] : INFINITY;
            n += in ? 1 : 0;
        }
        d.back[lm] = median_regs(wb, n);
        d.rms[lm] = median_regs(wr, n);
    } else {
        double* wt = w + threadIdx.x;
        for (int q = 0; q < 2; ++q) {
            const double* src = q ? d.rms_raw : d.back_raw;
            double* dst = q ? d.rms : d.back;
            int n = 0;
            for (int b = j - hh; b <= j + hh; ++b)
                for (int c = i - hh; c <= i + hh; ++c)
                    if (b >= 0 && b < d.ny && c >= 0 && c < d.nx) wt[(n++) * kGridThreads] = src[b * d.nx + c];
            dst[lm] = median_small(wt, n, kGridThreads);
        }
    }
}

// ---------------------------------------------------------------------------
// Natural spline second derivatives through (t_k, f_k), k < n, by Thomas
// elimination.  The elimination factors depend on the knots only, so a block
// computes them once into LDS (spline_factor) and every column then runs a
// single dependent chain (spline_solve), its right-hand sides loaded ahead.
__device__ void spline_factor(int n, const double* t, double* c, double* den) {
    double cp = 0.0;
    for (int k = 1; k <= n - 2; ++k) {
        const double h0 = t[k] - t[k - 1], h1 = t[k + 1] - t[k];
        const double b = 2.0 * (h0 + h1);
        const double dk = (k == 1) ? b : b - h0 * cp;
        den[k] = dk;
        cp = h1 / dk;
        c[k] = cp;
    }
}

// f at stride fs; r (work) and m (result) at stride ms
__device__ void spline_solve(int n, const double* t, const double* c, const double* den,
                             const double* __restrict__ f, int fs, double* __restrict__ r,
                             double* __restrict__ m, int ms) {
    m[0] = 0.0;
    if (n > 1) m[(n - 1) * ms] = 0.0;
    if (n < 3) return;
    double rp = 0.0;
    double f0 = f[0], f1 = f[fs];
    for (int k = 1; k <= n - 2; ++k) {
        const double f2 = f[(k + 1) * fs];
        const double h0 = t[k] - t[k - 1], h1 = t[k + 1] - t[k];
        const double rhs = 6.0 * ((f2 - f1) / h1 - (f1 - f0) / h0);
        rp = (k == 1) ? rhs / den[k] : (rhs - h0 * rp) / den[k];
        r[k * ms] = rp;
        f0 = f1;
        f1 = f2;
    }
    double mk = rp;
    m[(n - 2) * ms] = mk;
    for (int k = n - 3; k >= 1; --k) {
        mk = r[k * ms] - c[k] * mk;
        m[k * ms] = mk;
    }
}

// cubic of one spline piece in local coordinate s = t - ref:
// piece 0 (t < t_0) and piece n (t >= t_{n-1}) are the end tangents,
// piece j in [1, n-1] spans [t_{j-1}, t_j)
__device__ void piece_poly(int n, const double* t, const double* f, int fs, const double* m, int ms,
                           int piece, double out[4]) {
    out[0] = out[1] = out[2] = out[3] = 0.0;
    if (n == 1) {
        out[0] = f[0];
        return;
    }
    if (piece == 0) {
        double h = t[1] - t[0];
        out[0] = f[0];
        out[1] = (f[fs] - f[0]) / h - h * (2.0 * m[0] + m[ms]) / 6.0;
        return;
    }
    if (piece == n) {
        double h = t[n - 1] - t[n - 2];
        out[0] = f[(n - 1) * fs];
        out[1] = (f[(n - 1) * fs] - f[(n - 2) * fs]) / h + h * (m[(n - 2) * ms] + 2.0 * m[(n - 1) * ms]) / 6.0;
        return;
    }
    int j = piece - 1;
    double h = t[j + 1] - t[j];
    double mj = m[j * ms], mj1 = m[(j + 1) * ms];
    out[0] = f[j * fs];
    out[1] = (f[(j + 1) * fs] - f[j * fs]) / h - h * (2.0 * mj + mj1) / 6.0;
    out[2] = 0.5 * mj;
    out[3] = (mj1 - mj) / (6.0 * h);
}

constexpr int kSplThreads = 256;
constexpr int kSplCols = 64;       // small grids: columns per workgroup (one wavefront)
constexpr int kSplSmallN = 100;    // small grids: knots per axis held in LDS

// The same elimination with reciprocals: ih[k] = 1 / (t_{k+1} - t_k) (every
// thread computes its share before the call), c[k] and iden[k] = 1 / den[k]
// (one thread), so the column solves are chains of FMAs.
__device__ __forceinline__ void spline_factor_inv(int n, const double* t, double* c, double* iden) {
    double cp = 0.0;
    for (int k = 1; k <= n - 2; ++k) {
        const double h0 = t[k] - t[k - 1], h1 = t[k + 1] - t[k];
        const double b = 2.0 * (h0 + h1);
        const double id = 1.0 / ((k == 1) ? b : b - h0 * cp);
        iden[k] = id;
        cp = h1 * id;
        c[k] = cp;
    }
}

// second derivatives m (stride ms) of the column f (stride fs); m holds the
// forward sweep's values until the back sweep overwrites them in place
__device__ __forceinline__ void spline_solve_inv(int n, const double* t, const double* c, const double* iden,
                                                 const double* ih, const double* f, int fs, double* m, int ms) {
    m[0] = 0.0;
    if (n > 1) m[(n - 1) * ms] = 0.0;
    if (n < 3) return;
    double rp = 0.0;
    double f0 = f[0], f1 = f[fs];
    for (int k = 1; k <= n - 2; ++k) {
        const double f2 = f[(k + 1) * fs];
        const double rhs = 6.0 * ((f2 - f1) * ih[k] - (f1 - f0) * ih[k - 1]);
        rp = (rhs - (t[k] - t[k - 1]) * rp) * iden[k];
        m[k * ms] = rp;
        f0 = f1;
        f1 = f2;
    }
    double mk = rp;
    for (int k = n - 3; k >= 1; --k) {
        mk = m[k * ms] - c[k] * mk;
        m[k * ms] = mk;
    }
}

// piece_poly with the reciprocal spacings
__device__ __forceinline__ void piece_poly_inv(int n, const double* t, const double* ih, const double* f, int fs,
                                               const double* m, int ms, int piece, double out[4]) {
    constexpr double kSixth = 1.0 / 6.0;
    out[0] = out[1] = out[2] = out[3] = 0.0;
    if (n == 1) {
        out[0] = f[0];
        return;
    }
    if (piece == 0) {
        const double h = t[1] - t[0];
        out[0] = f[0];
        out[1] = (f[fs] - f[0]) * ih[0] - h * (2.0 * m[0] + m[ms]) * kSixth;
        return;
    }
    if (piece == n) {
        const double h = t[n - 1] - t[n - 2];
        out[0] = f[(n - 1) * fs];
        out[1] = (f[(n - 1) * fs] - f[(n - 2) * fs]) * ih[n - 2] + h * (m[(n - 2) * ms] + 2.0 * m[(n - 1) * ms]) * kSixth;
        return;
    }
    const int j = piece - 1;
    const double h = t[j + 1] - t[j];
    const double mj = m[j * ms], mj1 = m[(j + 1) * ms];
    out[0] = f[j * fs];
    out[1] = (f[(j + 1) * fs] - f[j * fs]) * ih[j] - h * (2.0 * mj + mj1) * kSixth;
    out[2] = 0.5 * mj;
    out[3] = (mj1 - mj) * ih[j] * kSixth;
}

// A column of n values (stride s) into the LDS column `lane` of fl.  The
// first kSplPre loads are issued by prefetch_column and waited for only in
// store_column, so the knot factorisation runs while they are in flight; the
// rest follow 16 at a time.  Indices are clamped to the column, so no load
// needs a branch.
constexpr int kSplPre = 64;

__device__ __forceinline__ void prefetch_column(double (&x)[kSplPre], const double* v, int s, int n) {
    const gdouble_t* g = (const gdouble_t*)v;   // global loads: they do not hold up LDS waits
#pragma unroll
    for (int j = 0; j < kSplPre; ++j) x[j] = g[(size_t)min(j, n - 1) * s];
}

__device__ __forceinline__ void store_column(double* fl, int lane, const double (&x)[kSplPre], const double* v,
                                             int s, int n) {
#pragma unroll
    for (int j = 0; j < kSplPre; ++j)
        if (j < n) fl[j * kSplCols + lane] = x[j];
    const gdouble_t* g = (const gdouble_t*)v;
    for (int k0 = kSplPre; k0 < n; k0 += 16) {
        double y[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) y[j] = g[(size_t)min(k0 + j, n - 1) * s];
#pragma unroll
        for (int j = 0; j < 16; ++j)
            if (k0 + j < n) fl[(k0 + j) * kSplCols + lane] = y[j];
    }
}

// Small grids (at most kSplSmallN knots on the solved axis): a wavefront takes
// 64 columns; their values are loaded into LDS at once (all loads in flight),
// solved and cut into pieces there, and only the pieces go to global memory.
// blockIdx.y = frame.  Y: one column per (quantity, mesh column).
__global__ __launch_bounds__(kSplCols) void k_spline_y_small(const FrameDesc* __restrict__ desc) {
    __shared__ double tk[kSplSmallN], cf[kSplSmallN], idn[kSplSmallN], ih[kSplSmallN];
    __shared__ double fl[kSplSmallN * kSplCols], ml[kSplSmallN * kSplCols];
    const FrameDesc& d = desc[blockIdx.y];
    const int ny = d.ny, nx = d.nx, lane = threadIdx.x;
    if ((int)blockIdx.x * kSplCols >= 2 * nx) return;
    const int g = blockIdx.x * kSplCols + lane;
    const bool on = g < 2 * nx;
    const int q = on ? g / nx : 0, i = on ? g - q * nx : 0;
    const double* col = (q ? d.rms : d.back) + i;
    for (int k = lane; k < ny; k += kSplCols) tk[k] = knot_at(k, d.H, d.mh);
    __syncthreads();
    double x[kSplPre];
    prefetch_column(x, col, nx, ny);
    for (int k = lane; k + 1 < ny; k += kSplCols) ih[k] = 1.0 / (tk[k + 1] - tk[k]);
    if (lane == 0) spline_factor_inv(ny, tk, cf, idn);
    store_column(fl, lane, x, col, nx, ny);
    __syncthreads();
    if (!on) return;
    spline_solve_inv(ny, tk, cf, idn, ih, fl + lane, kSplCols, ml + lane, kSplCols);
    for (int jy = 0; jy <= ny; ++jy) {
        double c[4];
        piece_poly_inv(ny, tk, ih, fl + lane, kSplCols, ml + lane, kSplCols, jy, c);
        double* o = d.ycoef + (((size_t)q * (ny + 1) + jy) * nx + i) * 4;
        o[0] = c[0];
        o[1] = c[1];
        o[2] = c[2];
        o[3] = c[3];
    }
}

// X: one column per (quantity, y piece, power of u), as k_spline_x
__global__ __launch_bounds__(kSplCols) void k_spline_x_small(const FrameDesc* __restrict__ desc) {
    __shared__ double tk[kSplSmallN], cf[kSplSmallN], idn[kSplSmallN], ih[kSplSmallN];
    __shared__ double fl[kSplSmallN * kSplCols], ml[kSplSmallN * kSplCols];
    const FrameDesc& d = desc[blockIdx.y];
    const int nx = d.nx, ny = d.ny, lane = threadIdx.x;
    const int G = 8 * (ny + 1);
    if ((int)blockIdx.x * kSplCols >= G) return;
    const int g = blockIdx.x * kSplCols + lane;
    const bool on = g < G;
    const int r = g & 3;
    const int jy = on ? (g >> 2) % (ny + 1) : 0;
    const int q = on ? (g >> 2) / (ny + 1) : 0;
    const double* vals = d.ycoef + (((size_t)q * (ny + 1) + jy) * nx) * 4 + r;  // stride 4
    for (int k = lane; k < nx; k += kSplCols) tk[k] = knot_at(k, d.W, d.mw);
    __syncthreads();
    double x[kSplPre];
    prefetch_column(x, vals, 4, nx);
    for (int k = lane; k + 1 < nx; k += kSplCols) ih[k] = 1.0 / (tk[k + 1] - tk[k]);
    if (lane == 0) spline_factor_inv(nx, tk, cf, idn);
    store_column(fl, lane, x, vals, 4, nx);
    __syncthreads();
    if (!on) return;
    spline_solve_inv(nx, tk, cf, idn, ih, fl + lane, kSplCols, ml + lane, kSplCols);
    for (int ix = 0; ix <= nx; ++ix) {
        double c[4];
        piece_poly_inv(nx, tk, ih, fl + lane, kSplCols, ml + lane, kSplCols, ix, c);
        double* o = d.coef + (((size_t)q * (ny + 1) + jy) * (nx + 1) + ix) * 16;
        for (int p = 0; p < 4; ++p) o[p * 4 + r] = c[p];
    }
}

// ---------------------------------------------------------------------------
// Grids of at most kPcrMax knots on the solved axis: one wavefront per spline, lane k =
// knot k.  The tridiagonal system of the natural spline's second derivatives
// (interior rows h_{k-1} m_{k-1} + 2 (h_{k-1} + h_k) m_k + h_k m_{k+1} =
// 6 (f_{k+1} - f_k) / h_k - 6 (f_k - f_{k-1}) / h_{k-1}, m_0 = m_{n-1} = 0)
// is solved by parallel cyclic reduction: six rounds, each eliminating the
// couplings to the rows at distance 1, 2, ..., 32 (fetched by lane shuffles;
// rows outside the spline are identity rows).  The matrix is strictly
// diagonally dominant, so the reduction is stable.  Lane p then forms piece p
// from the values of lanes clamp(p - 1, 0, n - 2) and the next one.  The
// y splines also apply the mesh filter (lane k takes mesh (k, i)).
constexpr int kPcrMax = 63;   // knots: the n + 1 pieces fit one wavefront

// second derivatives at the knots; t0 = t_{k-1}, t1 = t_k, t2 = t_{k+1}
__device__ __forceinline__ double pcr_second_derivs(int n, int lane, double t0, double t1, double t2, double fm,
                                                    double f, double fp) {
    const bool row = lane >= 1 && lane <= n - 2;
    const double h0 = t1 - t0, h1 = t2 - t1;
    double a = row ? h0 : 0.0, b = row ? 2.0 * (h0 + h1) : 1.0, c = row ? h1 : 0.0;
    double d = row ? 6.0 * ((fp - f) / h1 - (f - fm) / h0) : 0.0;
#pragma unroll
    for (int st = 1; st < 64; st <<= 1) {
        const double rb = 1.0 / b;
        const bool okl = lane >= st, okh = lane + st < 64;
        const int sl = okl ? lane - st : lane, sh = okh ? lane + st : lane;
        const double al = __shfl(a, sl), cl = __shfl(c, sl), dl = __shfl(d, sl), rl = __shfl(rb, sl);
        const double ah = __shfl(a, sh), ch = __shfl(c, sh), dh = __shfl(d, sh), rh = __shfl(rb, sh);
        const double al_ = okl ? al : 0.0, cl_ = okl ? cl : 0.0, dl_ = okl ? dl : 0.0, rl_ = okl ? rl : 1.0;
        const double ah_ = okh ? ah : 0.0, ch_ = okh ? ch : 0.0, dh_ = okh ? dh : 0.0, rh_ = okh ? rh : 1.0;
        const double alpha = -a * rl_, gamma = -c * rh_;
        b = b + alpha * cl_ + gamma * ah_;
        d = d + alpha * dl_ + gamma * dh_;
        a = alpha * al_;
        c = gamma * ch_;
    }
    return d / b;
}

// piece p of the spline through n knots from the values at knots A =
// clamp(p - 1, 0, n - 2) and A + 1 and their spacing hA; out[r] = coefficient
// of u^r, u = position - reference knot
__device__ __forceinline__ void spline_piece(int n, int p, double fA, double fB, double mA, double mB, double hA,
                                             double out[4]) {
    constexpr double kSixth = 1.0 / 6.0;
    const double ih = 1.0 / hA;
    out[0] = out[1] = out[2] = out[3] = 0.0;
    if (n == 1) {
        out[0] = fA;
    } else if (p == 0) {
        out[0] = fA;
        out[1] = (fB - fA) * ih - hA * (2.0 * mA + mB) * kSixth;
    } else if (p == n) {
        out[0] = fB;
        out[1] = (fB - fA) * ih + hA * (mA + 2.0 * mB) * kSixth;
    } else {
        out[0] = fA;
        out[1] = (fB - fA) * ih - hA * (2.0 * mA + mB) * kSixth;
        out[2] = 0.5 * mA;
        out[3] = (mB - mA) * ih * kSixth;
    }
}

// piece p = lane, the values of knots A and A + 1 fetched by lane shuffles
__device__ __forceinline__ void pcr_piece(int n, int lane, double f, double m, double h, double out[4]) {
    const int A = min(max(lane - 1, 0), max(n - 2, 0));
    const double fA = __shfl(f, A), fB = __shfl(f, A + 1), mA = __shfl(m, A), mB = __shfl(m, A + 1);
    const double hA = __shfl(h, A);
    spline_piece(n, lane, fA, fB, mA, mB, hA, out);
}

// Grids of 64 to kPcrBlkMax knots on the solved axis: the same reduction over
// a workgroup of NT = 128, 256 or 512 threads (thread = knot), seven to nine
// rounds, the rows exchanged through LDS (s*: NT doubles each).  More knots go
// to the serial solve: its columns fill few lanes and each is one chain of
// divisions (16 frames of up to 150 x 100 knots: 219 us with the filter, 52 us here).
constexpr int kPcrBlkMax = 511;

template <int NT>
__device__ double pcr_second_derivs_blk(int n, int k, double t0, double t1, double t2, double fm, double f,
                                        double fp, double* sa, double* sc, double* sd, double* sr) {
    const bool row = k >= 1 && k <= n - 2;
    const double h0 = t1 - t0, h1 = t2 - t1;
    double a = row ? h0 : 0.0, b = row ? 2.0 * (h0 + h1) : 1.0, c = row ? h1 : 0.0;
    double d = row ? 6.0 * ((fp - f) / h1 - (f - fm) / h0) : 0.0;
    for (int st = 1; st < NT; st <<= 1) {
        sa[k] = a;
        sc[k] = c;
        sd[k] = d;
        sr[k] = 1.0 / b;
        __syncthreads();
        const bool okl = k >= st, okh = k + st < NT;
        const double al = okl ? sa[k - st] : 0.0, cl = okl ? sc[k - st] : 0.0, dl = okl ? sd[k - st] : 0.0;
        const double rl = okl ? sr[k - st] : 1.0;
        const double ah = okh ? sa[k + st] : 0.0, ch = okh ? sc[k + st] : 0.0, dh = okh ? sd[k + st] : 0.0;
        const double rh = okh ? sr[k + st] : 1.0;
        __syncthreads();
        const double alpha = -a * rl, gamma = -c * rh;
        b = b + alpha * cl + gamma * ah;
        d = d + alpha * dl + gamma * dh;
        a = alpha * al;
        c = gamma * ch;
    }
    return d / b;
}

// y splines (and the mesh filter when F > 0), one workgroup per (quantity,
// mesh column); blockIdx.y = frame
template <int F, int NT>
__global__ __launch_bounds__(NT) void k_spline_y_pcr_blk(const FrameDesc* __restrict__ desc) {
    __shared__ double sa[NT], sc[NT], sd[NT], sr[NT];
    const FrameDesc& d = desc[blockIdx.y];
    const int nx = d.nx, ny = d.ny, t = threadIdx.x;
    const int g = blockIdx.x;
    if (g >= 2 * nx) return;
    const int q = g / nx, i = g - q * nx;
    const int k = min(t, ny - 1);
    double f;
    if constexpr (F > 0) {
        constexpr int hh = F / 2;
        const gdouble_t* raw = (const gdouble_t*)(q ? d.rms_raw : d.back_raw);
        double w[F * F];
        int cnt = 0;
#pragma unroll
        for (int e = 0; e < F * F; ++e) {
            const int b = k - hh + e / F, c = i - hh + e % F;
            const bool in = b >= 0 && b < ny && c >= 0 && c < nx;
            w[e] = in ? raw[b * nx + c] : INFINITY;
            cnt += in ? 1 : 0;
        }
        f = median_regs(w, cnt);
        if (t < ny) (q ? d.rms : d.back)[k * nx + i] = f;
    } else {
        f = ((const gdouble_t*)(q ? d.rms : d.back))[k * nx + i];
    }
    const double t0 = knot_at(max(k - 1, 0), d.H, d.mh), t1 = knot_at(k, d.H, d.mh);
    const double t2 = knot_at(min(k + 1, ny - 1), d.H, d.mh);
    sd[t] = f;
    __syncthreads();
    const double fm = sd[max(t - 1, 0)], fp = sd[min(t + 1, NT - 1)];
    __syncthreads();
    const double m = pcr_second_derivs_blk<NT>(ny, t, t0, t1, t2, fm, f, fp, sa, sc, sd, sr);
    sa[t] = f;
    sc[t] = m;
    sd[t] = t2 - t1;
    __syncthreads();
    if (t <= ny) {
        const int A = min(max(t - 1, 0), max(ny - 2, 0));
        double cf[4];
        spline_piece(ny, t, sa[A], sa[A + 1], sc[A], sc[A + 1], sd[A], cf);
        double* o = d.ycoef + (((size_t)q * (ny + 1) + t) * nx + i) * 4;
        o[0] = cf[0];
        o[1] = cf[1];
        o[2] = cf[2];
        o[3] = cf[3];
    }
}

// x splines, one workgroup per (quantity, y piece, power of u); blockIdx.y = frame
template <int NT>
__global__ __launch_bounds__(NT) void k_spline_x_pcr_blk(const FrameDesc* __restrict__ desc) {
    __shared__ double sa[NT], sc[NT], sd[NT], sr[NT];
    const FrameDesc& d = desc[blockIdx.y];
    const int nx = d.nx, ny = d.ny, t = threadIdx.x;
    const int g = blockIdx.x;
    if (g >= 8 * (ny + 1)) return;
    const int b = g >> 2, r = g & 3;   // b = q (ny + 1) + jy
    const int k = min(t, nx - 1);
    const double f = ((const gdouble_t*)d.ycoef)[((size_t)b * nx + k) * 4 + r];
    const double t0 = knot_at(max(k - 1, 0), d.W, d.mw), t1 = knot_at(k, d.W, d.mw);
    const double t2 = knot_at(min(k + 1, nx - 1), d.W, d.mw);
    sd[t] = f;
    __syncthreads();
    const double fm = sd[max(t - 1, 0)], fp = sd[min(t + 1, NT - 1)];
    __syncthreads();
    const double m = pcr_second_derivs_blk<NT>(nx, t, t0, t1, t2, fm, f, fp, sa, sc, sd, sr);
    sa[t] = f;
    sc[t] = m;
    sd[t] = t2 - t1;
    __syncthreads();
    if (t <= nx) {
        const int A = min(max(t - 1, 0), max(nx - 2, 0));
        double cf[4];
        spline_piece(nx, t, sa[A], sa[A + 1], sc[A], sc[A + 1], sd[A], cf);
        double* o = d.coef + ((size_t)b * (nx + 1) + t) * 16;
        for (int pp = 0; pp < 4; ++pp) o[pp * 4 + r] = cf[pp];
    }
}

// y splines (and the mesh filter when F > 0): blockIdx.y = frame, one
// wavefront per (quantity, mesh column), four per workgroup
template <int F>
__global__ __launch_bounds__(256) void k_spline_y_pcr(const FrameDesc* __restrict__ desc) {
    const FrameDesc& d = desc[blockIdx.y];
    const int nx = d.nx, ny = d.ny, lane = threadIdx.x & 63;
    const int g = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (g >= 2 * nx) return;
    const int q = g / nx, i = g - q * nx;
    const int k = min(lane, ny - 1);
    double f;
    if constexpr (F > 0) {
        constexpr int hh = F / 2;
        const gdouble_t* raw = (const gdouble_t*)(q ? d.rms_raw : d.back_raw);
        double w[F * F];
        int cnt = 0;
#pragma unroll
        for (int e = 0; e < F * F; ++e) {
            const int b = k - hh + e / F, c = i - hh + e % F;
            const bool in = b >= 0 && b < ny && c >= 0 && c < nx;
            w[e] = in ? raw[b * nx + c] : INFINITY;
            cnt += in ? 1 : 0;
        }
        f = median_regs(w, cnt);
        if (lane < ny) (q ? d.rms : d.back)[k * nx + i] = f;
    } else {
        f = ((const gdouble_t*)(q ? d.rms : d.back))[k * nx + i];
    }
    const double t0 = knot_at(max(k - 1, 0), d.H, d.mh), t1 = knot_at(k, d.H, d.mh);
    const double t2 = knot_at(min(k + 1, ny - 1), d.H, d.mh);
    const double fm = __shfl(f, max(lane - 1, 0)), fp = __shfl(f, min(lane + 1, 63));
    const double m = pcr_second_derivs(ny, lane, t0, t1, t2, fm, f, fp);
    double c[4];
    pcr_piece(ny, lane, f, m, t2 - t1, c);
    if (lane <= ny) {
        double* o = d.ycoef + (((size_t)q * (ny + 1) + lane) * nx + i) * 4;
        o[0] = c[0];
        o[1] = c[1];
        o[2] = c[2];
        o[3] = c[3];
    }
}

// x splines: blockIdx.y = frame; workgroup = (quantity, y piece), its four
// wavefronts the four powers of u
__global__ __launch_bounds__(256) void k_spline_x_pcr(const FrameDesc* __restrict__ desc) {
    const FrameDesc& d = desc[blockIdx.y];
    const int nx = d.nx, ny = d.ny, lane = threadIdx.x & 63, r = threadIdx.x >> 6;
    const int b = blockIdx.x;
    if (b >= 2 * (ny + 1)) return;
    const int k = min(lane, nx - 1);
    const double f = ((const gdouble_t*)d.ycoef)[((size_t)b * nx + k) * 4 + r];   // b = q (ny + 1) + jy
    const double t0 = knot_at(max(k - 1, 0), d.W, d.mw), t1 = knot_at(k, d.W, d.mw);
    const double t2 = knot_at(min(k + 1, nx - 1), d.W, d.mw);
    const double fm = __shfl(f, max(lane - 1, 0)), fp = __shfl(f, min(lane + 1, 63));
    const double m = pcr_second_derivs(nx, lane, t0, t1, t2, fm, f, fp);
    double c[4];
    pcr_piece(nx, lane, f, m, t2 - t1, c);
    if (lane <= nx) {
        double* o = d.coef + ((size_t)b * (nx + 1) + lane) * 16;
        for (int p = 0; p < 4; ++p) o[p * 4 + r] = c[p];
    }
}

// Larger grids: y-splines, blockIdx.y = frame; one thread per (quantity, mesh column)
__global__ __launch_bounds__(kSplThreads) void k_spline_y(const FrameDesc* __restrict__ desc) {
    __shared__ double tk[kSplineMaxKnots], cf[kSplineMaxKnots], dn[kSplineMaxKnots];
    const FrameDesc& d = desc[blockIdx.y];
    const int ny = d.ny, nx = d.nx;
    if ((int)blockIdx.x * kSplThreads >= 2 * nx) return;
    for (int k = threadIdx.x; k < ny; k += kSplThreads) tk[k] = knot_at(k, d.H, d.mh);
    __syncthreads();
    if (threadIdx.x == 0) spline_factor(ny, tk, cf, dn);
    __syncthreads();
    const int g = blockIdx.x * kSplThreads + threadIdx.x;
    if (g >= 2 * nx) return;
    const int q = g / nx, i = g - q * nx;
    const double* col = (q ? d.rms : d.back) + i;
    // scratch [k][g]: work then second derivatives, 2 nx columns each
    double* r = d.scratch + g;
    double* mm = d.scratch + (size_t)2 * nx * ny + g;
    spline_solve(ny, tk, cf, dn, col, nx, r, mm, 2 * nx);
    for (int jy = 0; jy <= ny; ++jy) {
        double c[4];
        piece_poly(ny, tk, col, nx, mm, 2 * nx, jy, c);
        double* o = d.ycoef + (((size_t)q * (ny + 1) + jy) * nx + i) * 4;
        o[0] = c[0];
        o[1] = c[1];
        o[2] = c[2];
        o[3] = c[3];
    }
}

// x-splines: the tensor spline's row cubic on y piece jy is a cubic in u whose
// four coefficients are linear in the column values, so the x spline of each
// coefficient vector (one natural spline per (quantity, jy, power of u)) gives
// the bicubic pieces directly: coef[q][jy][ix][p*4+r] = x-piece p coefficient
// of the spline through (ycoef[q][jy][k][r])_k.  Exact on constant grids.
// blockIdx.y = frame; one thread per (quantity, jy, power).
__global__ __launch_bounds__(kSplThreads) void k_spline_x(const FrameDesc* __restrict__ desc) {
    __shared__ double tk[kSplineMaxKnots], cf[kSplineMaxKnots], dn[kSplineMaxKnots];
    const FrameDesc& d = desc[blockIdx.y];
    const int nx = d.nx, ny = d.ny;
    const int G = 8 * (ny + 1);
    if ((int)blockIdx.x * kSplThreads >= G) return;
    for (int k = threadIdx.x; k < nx; k += kSplThreads) tk[k] = knot_at(k, d.W, d.mw);
    __syncthreads();
    if (threadIdx.x == 0) spline_factor(nx, tk, cf, dn);
    __syncthreads();
    const int g = blockIdx.x * kSplThreads + threadIdx.x;
    if (g >= G) return;
    const int r = g & 3;
    const int jy = (g >> 2) % (ny + 1);
    const int q = (g >> 2) / (ny + 1);
    double* base = d.scratch + (size_t)8 * nx * ny;   // after the y-spline scratch
    double* w = base + g;                               // [k][g], G columns
    double* mm = base + (size_t)G * nx + g;
    const double* vals = d.ycoef + (((size_t)q * (ny + 1) + jy) * nx) * 4 + r;  // stride 4
    spline_solve(nx, tk, cf, dn, vals, 4, w, mm, G);
    for (int ix = 0; ix <= nx; ++ix) {
        double c[4];
        piece_poly(nx, tk, vals, 4, mm, G, ix, c);
        double* o = d.coef + (((size_t)q * (ny + 1) + jy) * (nx + 1) + ix) * 16;
        for (int p = 0; p < 4; ++p) o[p * 4 + r] = c[p];
    }
}

// ---------------------------------------------------------------------------
// launchers
// cfg: 0 = automatic, 1 = 256 x 16, 2 = 512 x 16, 3 = 512 x 32, 4 = 1024 x 16,
// 5 = 64 x 16 (threads x pixels per thread; the product must cover the
// largest mesh).  The automatic choice is the smallest that covers it: 32 x 32
// meshes in 256-thread workgroups leave three wavefronts of four idle (4.3 MP
// of them: 216 us in the 256 x 16 shape of the register passes, 34 us in 64 x
// 16).
template <typename T, int NT, int PPT>
static void launch_mesh_nt(FrameDesc* desc, const FrameDesc* one, int nframes, int total_meshes, BkgArgs a,
                           hipStream_t s) {
    if (one) k_mesh_stats<T, NT, PPT, true><<<total_meshes, NT, 0, s>>>(desc, *one, nframes, a);
    else k_mesh_stats<T, NT, PPT, false><<<total_meshes, NT, 0, s>>>(desc, FrameDesc{}, nframes, a);
}

template <typename T>
static void launch_mesh_t(FrameDesc* desc, const FrameDesc* one, int nframes, int total_meshes, int max_area,
                          BkgArgs a, int cfg, hipStream_t s) {
    const bool fits = cfg == 1 ? max_area <= 4096 : cfg == 2 ? max_area <= 8192 : cfg == 5 ? max_area <= 1024 : true;
    if (cfg == 0 || !fits) cfg = max_area <= 1024 ? 5 : max_area <= 4096 ? 1 : max_area <= 8192 ? 2 : 3;
    switch (cfg) {
        case 1: launch_mesh_nt<T, 256, 16>(desc, one, nframes, total_meshes, a, s); break;
        case 2: launch_mesh_nt<T, 512, 16>(desc, one, nframes, total_meshes, a, s); break;
        case 4: launch_mesh_nt<T, 1024, 16>(desc, one, nframes, total_meshes, a, s); break;
        case 5: launch_mesh_nt<T, 64, 16>(desc, one, nframes, total_meshes, a, s); break;
        default: launch_mesh_nt<T, 512, 32>(desc, one, nframes, total_meshes, a, s); break;
    }
}

// uint16 meshes
void launch_mesh_stats_u16(FrameDesc* desc, const FrameDesc* one, int nframes, int total_meshes, int max_area,
                           BkgArgs a, int cfg, hipStream_t s) {
    launch_mesh_t<uint16_t>(desc, one, nframes, total_meshes, max_area, a, cfg, s);
}

// float32 meshes
void launch_mesh_stats(FrameDesc* desc, const FrameDesc* one, int nframes, int total_meshes, int max_area, BkgArgs a,
                       int cfg, hipStream_t s) {
    launch_mesh_t<float>(desc, one, nframes, total_meshes, max_area, a, cfg, s);
}

void launch_grid_filter(const FrameDesc* desc, int nframes, int total_meshes, int fsize, hipStream_t s) {
    const int blocks = (total_meshes + kGridThreads - 1) / kGridThreads;
    switch (fsize) {
        case 1: k_grid_filter<1><<<blocks, kGridThreads, 0, s>>>(desc, nframes, total_meshes, fsize); break;
        case 3: k_grid_filter<3><<<blocks, kGridThreads, 0, s>>>(desc, nframes, total_meshes, fsize); break;
        case 5: k_grid_filter<5><<<blocks, kGridThreads, 0, s>>>(desc, nframes, total_meshes, fsize); break;
        default: k_grid_filter<0><<<blocks, kGridThreads, 0, s>>>(desc, nframes, total_meshes, fsize); break;
    }
}

// mesh filter of size fsize (0: none, the grids are given) and the splines
// in two launches, for grids of at most kPcrBlkMax knots per axis and filters of
// at most 5 x 5 (filter_spline_fits)
bool filter_spline_fits(int max_nx, int max_ny, int fsize) {
    return max_nx <= kPcrBlkMax && max_ny <= kPcrBlkMax && fsize <= 5;
}

template <int NT>
static void launch_y_blk(const FrameDesc* desc, int nframes, int max_nx, int fsize, hipStream_t s) {
    const dim3 gy(2 * max_nx, nframes);
    switch (fsize) {
        case 0: k_spline_y_pcr_blk<0, NT><<<gy, NT, 0, s>>>(desc); break;
        case 1: k_spline_y_pcr_blk<1, NT><<<gy, NT, 0, s>>>(desc); break;
        case 3: k_spline_y_pcr_blk<3, NT><<<gy, NT, 0, s>>>(desc); break;
        default: k_spline_y_pcr_blk<5, NT><<<gy, NT, 0, s>>>(desc); break;
    }
}

// each axis by its own knot count: up to kPcrMax one wavefront per spline,
// up to kPcrBlkMax the smallest workgroup with more threads than knots
void launch_filter_spline(const FrameDesc* desc, int nframes, int max_nx, int max_ny, int fsize, hipStream_t s) {
    if (max_ny <= kPcrMax) {
        const dim3 gy((2 * max_nx + 3) / 4, nframes);
        switch (fsize) {
            case 0: k_spline_y_pcr<0><<<gy, 256, 0, s>>>(desc); break;
            case 1: k_spline_y_pcr<1><<<gy, 256, 0, s>>>(desc); break;
            case 3: k_spline_y_pcr<3><<<gy, 256, 0, s>>>(desc); break;
            default: k_spline_y_pcr<5><<<gy, 256, 0, s>>>(desc); break;
        }
    } else if (max_ny < 128) {
        launch_y_blk<128>(desc, nframes, max_nx, fsize, s);
    } else if (max_ny < 256) {
        launch_y_blk<256>(desc, nframes, max_nx, fsize, s);
    } else {
        launch_y_blk<512>(desc, nframes, max_nx, fsize, s);
    }
    const dim3 gx(8 * (max_ny + 1), nframes);
    if (max_nx <= kPcrMax) k_spline_x_pcr<<<dim3(2 * (max_ny + 1), nframes), 256, 0, s>>>(desc);
    else if (max_nx < 128) k_spline_x_pcr_blk<128><<<gx, 128, 0, s>>>(desc);
    else if (max_nx < 256) k_spline_x_pcr_blk<256><<<gx, 256, 0, s>>>(desc);
    else k_spline_x_pcr_blk<512><<<gx, 512, 0, s>>>(desc);
}

void launch_spline(const FrameDesc* desc, int nframes, int max_nx, int max_ny, hipStream_t s) {
    if (max_ny <= kSplSmallN)
        k_spline_y_small<<<dim3((2 * max_nx + kSplCols - 1) / kSplCols, nframes), kSplCols, 0, s>>>(desc);
    else
        k_spline_y<<<dim3((2 * max_nx + kSplThreads - 1) / kSplThreads, nframes), kSplThreads, 0, s>>>(desc);
    if (max_nx <= kSplSmallN)
        k_spline_x_small<<<dim3((8 * (max_ny + 1) + kSplCols - 1) / kSplCols, nframes), kSplCols, 0, s>>>(desc);
    else
        k_spline_x<<<dim3((8 * (max_ny + 1) + kSplThreads - 1) / kSplThreads, nframes), kSplThreads, 0, s>>>(desc);
}

// ---------------------------------------------------------------------------
// full-resolution background and noise maps of one frame (diagnostic output;
// the same per-row cubic and per-pixel evaluation as the detection kernel)
template <typename Real>
__global__ __launch_bounds__(256) void k_bkg_map(FrameDesc d, double* bmap, double* rmap) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= d.W) return;
    for (int y = blockIdx.y; y < d.H; y += gridDim.y) {
    const int jy = piece_of(y, d.H, d.mh);
    const double u = (double)y - piece_ref(jy, d.H, d.mh);
    const int ix = piece_of(x, d.W, d.mw);
    const RowT<Real> t = make_row<Real>(d.coef, d.nx, d.ny, ix, jy, u);
    const Real s = (Real)((double)x - piece_ref(ix, d.W, d.mw));
    const size_t o = (size_t)y * d.W + x;
    if (bmap) bmap[o] = eval_B(t, s);
    if (rmap) rmap[o] = (double)eval_R(t, s);
    }
}

void launch_bkg_map(const FrameDesc& d, double* bmap, double* rmap, bool f64, hipStream_t s) {
    dim3 grid((d.W + 255) / 256, d.H < 32768 ? d.H : 32768);
    if (f64) k_bkg_map<double><<<grid, 256, 0, s>>>(d, bmap, rmap);
    else k_bkg_map<float><<<grid, 256, 0, s>>>(d, bmap, rmap);
}

}  // namespace gpk
