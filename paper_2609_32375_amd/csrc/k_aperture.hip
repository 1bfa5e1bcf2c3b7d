// k_aperture.hip -- circular aperture photometry with exact pixel/disk overlap.
//
// One wavefront per catalogued object.  The rows of the object's box are taken
// in bands whose background and noise-map cubics fit a fixed share of LDS (FP64
// -> working precision; one band for the usual radii), the pixels the outer
// circle can touch are numbered run by run and spread over the lanes, and each
// lane forms M = I - B for its pixels and classifies them against every circle
// (the aperture radii, r_in and r_out).  Pixels wholly inside or outside a
// circle take weight 1 or 0; the rest get the exact area of the circle inside
// the pixel from a cancellation-free formula: clipped rectangle + trapezoid
// under the chord + circular segment (theta - sin theta by series for small
// angles).
//
// The paper measures fluxes in circular apertures of several radii with the
// variance propagated through the same weights and float64 accumulation; the
// annulus background is this path's addition.
#include "k_args.h"
#include "k_overlap.h"
#include "k_rowpoly.h"

namespace gpk {

constexpr int kApWaves = 4;
constexpr int kApCubics = 80;  // row cubics (rows x spline pieces) of a band
constexpr int kApList = 256;   // queued (pixel, circle) cuts per wavefront
// wavefronts per SIMD the registers are held to (FP32): more circles keep more
// sums.  At four, 128 registers: batches spill 16 bytes a lane for five
// circles, one-frame calls 32 for four and 48 for five, nothing from six on
// (151 registers at three)
constexpr int ap_occ(int nc) { return nc <= 5 ? 4 : nc <= 7 ? 3 : 2; }
static_assert(kApCubics <= 2 * 64, "two row cubics per lane");

// a queued cut: M, the pixel variance, and box column | box row << 8 | circle << 16
template <typename Real>
struct ApEntry {
    Real m, var;
    uint32_t code;
};

// Per-wavefront LDS layout (dynamic shared memory; the host sizes it).
//   col   local spline coordinate and piece of each box column
//   row   of each row of the band: element offset and column of its first
//         pixel, less the pixel's number in the band
//   mark  one bit per pixel number: a row starts at the next number
template <typename Real>
struct ApCol {
    Real sx;
    int32_t piece;
};
struct ApRow {
    int32_t off, x0;
};
template <typename Real, int NC>
struct ApLayout {
    int o_col, o_row, o_mark, o_tab, o_list, o_rad, marks, bytes;
    __host__ __device__ ApLayout(int side) {
        int o = 0;
        auto take = [&](int n, int al) {
            o = (o + al - 1) / al * al;
            const int r = o;
            o += n;
            return r;
        };
        marks = 2 * (min(64, side) * side / 64 + 2);   // 32-bit words
        o_col = take(side * (int)sizeof(ApCol<Real>), 16);
        o_row = take(min(64, side) * (int)sizeof(ApRow), 16);
        o_mark = take(marks * 4, 16);
        o_tab = take(kApCubics * (int)sizeof(RowT<Real>), 16);
        o_list = take(kApList * (int)sizeof(ApEntry<Real>), 16);
        o_rad = take(NC * (int)sizeof(Real), 16);
        bytes = (o + 15) / 16 * 16;
    }
};
// object-count prefix over the frames (whole workgroup), before the wavefronts' parts
__host__ __device__ __forceinline__ int ap_prefix_bytes(int nframes) { return (4 * (nframes + 1) + 15) / 16 * 16; }

// Circles: the aperture radii, r_in and r_out, sorted by radius on the host
// (a.crad / a.crole).  Circles are nested, so a pixel lies wholly inside every
// circle from some index kin on, wholly outside those before kout, and only
// the circles in [kout, kin) cut it (usually none or one).  A pixel adds
// (M, 1, var) to the sums of every circle that holds it.  A cut pixel is
// queued and, in a compacted lane-parallel pass, adds its exact weight w as
// (w M, w, w^2 var) to its circle.
//
// Only the pixels the outer circle can touch are visited: each row of the box
// contributes the run of columns within half a pixel plus the chord of the
// outer circle; the runs of a band are numbered consecutively and spread over
// the lanes, and a pixel's row is the number of row starts marked below it.
// Sums are kept per lane in registers (FP64: flux, area, variance) and
// reduced in a fixed order, so an object's result does not depend on what
// else runs.
//
// (No test whether a circle holds any of the 64 pixels before its sums: ten
// such branches in a row cost more than ten pairs of additions.  500 objects
// with eight radii up to 40 and r_out 64: 365 us with them, now 278; 20000 with
// two and r_out 15: 173, now 164.)
//
// Bound by VALU issue and the latency between an object's LDS tables, its
// pixels and its queue, at four wavefronts per SIMD (r_out 15: 6.7 KB of LDS each).
// Keeping the sums of every lane in LDS bins, finding a pixel's row by 17
// compares, two bands per box, pieces of straddling pixels one after another
// and the object's descriptor in vector registers took: 106,344 objects of
// 371 MP uint16 (r_out 15, two apertures) 1605 us, now 860; 60,243 of a
// crowded 12300^2 frame (r_out 18, three) 1255, now 636; 13,233 of 6144^2 289,
// now 137; FP64, 1092 objects, 73, now 33.
// ONE: a one-frame call, whose descriptor comes with the launch (d1) instead
// of from the workspace table
template <typename Real, int NC, bool ONE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(Real) == 4 ? ap_occ(NC) : 1))) void
k_aperture(const FrameDesc* __restrict__ desc, FrameDesc d1, ApArgs a, ApCat cat, int nixmax) {
    extern __shared__ __align__(16) unsigned char ap_dyn[];
    // (the wavefront's number, and with it everything about its object, in scalar registers)
    const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int R = (int)ceilf(a.rmax) + 1;
    const int side = 2 * R + 2;
    const ApLayout<Real, NC> L(side);
    int32_t* fpre = reinterpret_cast<int32_t*>(ap_dyn);
    unsigned char* base = ap_dyn + ap_prefix_bytes(a.nframes) + (size_t)wv * L.bytes;
    ApCol<Real>* cols = (ApCol<Real>*)(base + L.o_col);
    ApRow* rows = (ApRow*)(base + L.o_row);
    uint32_t* mark = (uint32_t*)(base + L.o_mark);
    RowT<Real>* tab = (RowT<Real>*)(base + L.o_tab);
    ApEntry<Real>* list = (ApEntry<Real>*)(base + L.o_list);
    Real* rad = (Real*)(base + L.o_rad);
    const uint64_t below = (lane == 0) ? 0ull : ((~0ull) >> (64 - lane));

    Real cr2[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) cr2[j] = (Real)a.crad[j] * (Real)a.crad[j];
    const Real rmax = (Real)a.crad[NC - 1], rmax2 = cr2[NC - 1];
    const Real inv_gain = (a.gain > 0.f) ? (Real)1 / (Real)a.gain : (Real)0;
    // radius by circle index for the cut-pixel pass (a lane-varying index)
#pragma unroll
    for (int j = 0; j < NC; ++j)
        if (lane == j) rad[j] = (Real)a.crad[j];

    // The catalogued objects of all frames, numbered consecutively (frame by
    // frame, rows < n_obj only), are split into 8 contiguous ranges, one per
    // XCD: neighbouring objects, whose boxes overlap, share that XCD's L2.
    const int nf = a.nframes;
    if (wv == 0) {
        // prefix of min(n_obj, capacity) over the frames (one wavefront)
        int run = 0;
        for (int f0 = 0; f0 < nf; f0 += 64) {
            const int fr = f0 + lane;
            const int c = fr < nf ? min(cat.n_obj[fr], a.capacity) : 0;
            int incl = c;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(incl, o);
                if (lane >= o) incl += y;
            }
            if (fr < nf) fpre[fr] = run + incl - c;
            run += __shfl(incl, 63);
        }
        if (lane == 0) fpre[nf] = run;
    }
    __syncthreads();
    const int total = __builtin_amdgcn_readfirstlane(fpre[nf]);
    const int chunk = (total + kXcds - 1) / kXcds;
    const int xcd = blockIdx.x % kXcds, per_xcd = gridDim.x / kXcds;
    const int o_end = min(total, (xcd + 1) * chunk);
    for (int o = xcd * chunk + (blockIdx.x / kXcds) * nw + wv; o < o_end; o += per_xcd * nw) {
        // frame of object o: last frame whose prefix is <= o
        int lo = 0, hi = nf - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (__builtin_amdgcn_readfirstlane(fpre[mid]) <= o) lo = mid;
            else hi = mid - 1;
        }
        const int f = lo, k = o - __builtin_amdgcn_readfirstlane(fpre[f]);
        const int row = f * a.capacity + k;
        const FrameDesc& d = ONE ? d1 : desc[f];
        // (a centre far off the frame, infinite or not a number: one whose
        // integers are in range, and that no circle reaches the frame from)
        const double xc = lane_d(fmin(fmax(cat.x[row], -1000.0), (double)d.W + 1000.0), 0);
        const double yc = lane_d(fmin(fmax(cat.y[row], -1000.0), (double)d.H + 1000.0), 0);
        const int cxi = (int)floor(xc), cyi = (int)floor(yc);
        const Real fx = (Real)(xc - (double)cxi), fy = (Real)(yc - (double)cyi);
        const int bx0 = cxi - R, by0 = cyi - R;
        const int cx_lo = max(bx0, 0), cx_hi = min(bx0 + side - 1, d.W - 1);
        const int ixlo = (cx_lo <= cx_hi) ? piece_of(cx_lo, d.W, d.mw) : 0;
        const int nix = (cx_lo <= cx_hi) ? min(piece_of(cx_hi, d.W, d.mw) - ixlo + 1, nixmax) : 1;
        wave_sync();
        for (int c = lane; c < side; c += 64) {
            const int px = bx0 + c;
            if (px >= 0 && px < d.W) {
                const int ix = piece_of(px, d.W, d.mw);
                cols[c] = ApCol<Real>{(Real)((double)px - piece_ref(ix, d.W, d.mw)), min(ix - ixlo, nixmax - 1)};
            }
        }
        double S[NC], V[NC], A[NC];   // sums of the pixels a circle holds or cuts
        int notin[NC], used = 0;      // visited pixels a circle does not hold, visited pixels
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            S[j] = V[j] = A[j] = 0.0;
            notin[j] = 0;
        }
        // queued cuts: pixels within one quadrant from the bottom of the list
        // (listn entries), pixels that straddle an axis through the centre
        // from the top (nstr entries), whose pieces on the two sides are
        // evaluated by two lanes
        int listn = 0, nstr = 0;
        auto add_w = [&](const ApEntry<Real>& E, bool on, Real w) __attribute__((always_inline)) {
            const double ws = (double)w * (double)E.m;
            const Real wvv = w * w * E.var;
            const int jj = on ? (int)(E.code >> 16) : -1;
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                S[j] += jj == j ? ws : 0.0;
                A[j] += (double)(jj == j ? w : (Real)0);
                V[j] += (double)(jj == j ? wvv : (Real)0);
            }
        };
        // exact weights of the queued cut pixels
        auto flush = [&]() __attribute__((always_inline)) {
            wave_sync();
            for (int e0 = 0; e0 < listn; e0 += 64) {
                const ApEntry<Real> E = list[min(e0 + lane, listn - 1)];
                const Real rj = rad[E.code >> 16];
                const Real ax = fabs((Real)((int)(E.code & 255u) - R) - fx);
                const Real ay = fabs((Real)((int)((E.code >> 8) & 255u) - R) - fy);
                const Real w = quad_area<Real, false>(ax - (Real)0.5, ax + (Real)0.5, ay - (Real)0.5, ay + (Real)0.5,
                                                      rj, rj * rj);
                add_w(E, e0 + lane < listn, w);
            }
            for (int e0 = 0; e0 < nstr; e0 += 32) {
                // lane pair: the two sides of the axis x = xc (or of y = yc);
                // a pixel on both axes has two pieces per lane
                const int e = e0 + (lane >> 1);
                const ApEntry<Real> E = list[kApList - 1 - min(e, nstr - 1)];
                const Real rj = rad[E.code >> 16];
                const Real ax = fabs((Real)((int)(E.code & 255u) - R) - fx);
                const Real ay = fabs((Real)((int)((E.code >> 8) & 255u) - R) - fy);
                const Real xl = ax - (Real)0.5, xh = ax + (Real)0.5, yl = ay - (Real)0.5, yh = ay + (Real)0.5;
                const bool sx = xl < (Real)0, sy = yl < (Real)0, second = (lane & 1) != 0;
                const Real px0 = sx ? (Real)0 : xl, px1 = sx && !second ? -xl : xh;
                Real py0 = yl, py1 = yh;
                if (sy) {
                    py0 = (Real)0;
                    py1 = sx || !second ? -yl : yh;
                }
                const Real a1 = quad_area<Real, true>(px0, px1, py0, py1, rj, rj * rj);
                Real a2 = (Real)0;
                if (__ballot(sx && sy) != 0ull && sx && sy) a2 = quad_area<Real, true>(px0, px1, (Real)0, yh, rj, rj * rj);
                const Real o1 = __shfl_xor(a1, 1), o2 = __shfl_xor(a2, 1);
                add_w(E, e < nstr && !second, ((a1 + a2) + o1) + o2);
            }
            listn = 0;
            nstr = 0;
            wave_sync();
        };
        const int ry0 = max(by0, 0), ry1 = min(by0 + side - 1, d.H - 1);
        const int band = min(64, kApCubics / nix);
        for (int band0 = ry0; band0 <= ry1; band0 += band) {
            const int nb = min(band, ry1 - band0 + 1);
            wave_sync();
            // the band's row runs: columns within half a pixel of the outer
            // circle's chord (one pixel of margin each side), clipped to the box
            int cnt = 0, xl = 0;
            if (lane < nb) {
                const int py = band0 + lane;
                const Real dy = (Real)(py - cyi) - fy;
                const Real nyd = fmax(fabs(dy) - (Real)0.5, (Real)0);
                if (nyd < rmax) {
                    const double hw = 0.5 + sqrt(fmax((double)rmax2 - (double)nyd * (double)nyd, 0.0));
                    xl = max(cx_lo, (int)floor(xc - hw) - 1);
                    const int xr = min(cx_hi, (int)ceil(xc + hw) + 1);
                    cnt = max(xr - xl + 1, 0);
                }
            }
            int incl = cnt;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(incl, o);
                if (lane >= o) incl += y;
            }
            const int total = __builtin_amdgcn_readlane(incl, nb - 1);
            // (the rows with pixels are consecutive: a chord grows towards the centre)
            int r0 = total > 0 ? __builtin_ctzll(__ballot(cnt > 0)) : 0;   // row of the numbers reached so far
            for (int i = lane; i < (total + 63) / 64 * 2; i += 64) mark[i] = 0u;
            wave_sync();
            if (lane < nb) {
                const int start = incl - cnt;
                rows[lane] = ApRow{(band0 + lane) * (int)d.pitch + xl - start, xl - start};
                if (start > 0) atomicOr(&mark[(start - 1) >> 5], 1u << ((start - 1) & 31));
            }
            for (int i = lane; i < 2 * nb * nix; i += 64) {
                const int e = i >> 1, rr = e / nix, pi = e - rr * nix;
                const int py = band0 + rr;
                const int jy = piece_of(py, d.H, d.mh);
                const double u = (double)py - piece_ref(jy, d.H, d.mh);
                make_half_row(d.coef, d.nx, d.ny, i & 1, ixlo + pi, jy, u, tab[e]);
            }
            wave_sync();
            // row, column and value of pixel number b + lane (row -1: past the band)
            auto fetch = [&](int b, int& r, int& px, float& v) __attribute__((always_inline)) {
                r = -1;
                px = bx0;
                v = 0.0f;
                if (b >= total) return;
                const uint32_t m0 = mark[b >> 5], m1 = mark[(b >> 5) + 1];
                const int rr = r0 + (int)__builtin_amdgcn_mbcnt_hi(m1, __builtin_amdgcn_mbcnt_lo(m0, 0u));
                r0 += __popc(m0) + __popc(m1);
                if (b + lane < total) {
                    const ApRow W = rows[rr];
                    const int off = W.off + b + lane;
                    r = rr;
                    px = W.x0 + b + lane;
                    v = d.dtype == kDtypeU16 ? (float)((gu16_t*)d.data)[off] : ((gfloat_t*)d.data)[off];
                }
            };
            int r_, px;
            float iv;
            fetch(0, r_, px, iv);
            int b0 = 0;
            do {
                int rn, pxn;
                float ivn;
                fetch(b0 + 64, rn, pxn, ivn);   // (the next round's loads under this one's work)
                const int c = px - bx0, cy = band0 + max(r_, 0) - by0;
                const Real dx = (Real)(c - R) - fx;
                const Real dy = (Real)(cy - R) - fy;
                const Real ax = fabs(dx), ay = fabs(dy);
                const Real nxd = fmax(ax - (Real)0.5, (Real)0), nyd = fmax(ay - (Real)0.5, (Real)0);
                const Real fxd = ax + (Real)0.5, fyd = ay + (Real)0.5;
                const Real dmin2 = nxd * nxd + nyd * nyd, dmax2 = fxd * fxd + fyd * fyd;
                const bool use = r_ >= 0 && dmin2 < rmax2;
                int kin = 0, kout = 0;
                Real m = 0, var = 0;
                if (use) {
                    const ApCol<Real> C = cols[c];
                    const RowT<Real> T = tab[r_ * nix + C.piece];
                    m = eval_M(T, C.sx, (Real)iv);
                    if (a.want_err) {
                        const Real rv = eval_R(T, C.sx);
                        var = rv * rv + ((m > (Real)0) ? m * inv_gain : (Real)0);
                    }
                    ++used;
                }
#pragma unroll
                for (int j = 0; j < NC; ++j) {
                    const bool cut = use && cr2[j] < dmax2, in = use && !cut;
                    kin += cut ? 1 : 0;
                    kout += use && cr2[j] <= dmin2 ? 1 : 0;
                    notin[j] += cut ? 1 : 0;
                    S[j] += (double)(in ? m : (Real)0);
                    V[j] += (double)(in ? var : (Real)0);
                }
                // circles that cut the pixel: queue (pixel, circle) pairs; the
                // queue is worked off when full and at the object's last round
                const int ncut = kin - kout;
                const bool str = ax < (Real)0.5 || ay < (Real)0.5;
                const uint32_t code = (uint32_t)c | ((uint32_t)cy << 8);
                const bool last = band0 + band > ry1 && b0 + 64 >= total;
                for (int q = 0;; ++q) {
                    const bool has = q < ncut;
                    const uint64_t bm = __ballot(has && !str), bs = __ballot(has && str);
                    const bool none = (bm | bs) == 0ull;
                    if (has) {
                        const int pos = str ? kApList - 1 - (nstr + __popcll(bs & below))
                                            : listn + __popcll(bm & below);
                        list[pos] = ApEntry<Real>{m, var, code | ((uint32_t)(kout + q) << 16)};
                    }
                    listn += __popcll(bm);
                    nstr += __popcll(bs);
                    if (listn + nstr > kApList - 64 || (none && last)) flush();
                    if (none) break;
                }
                r_ = rn;
                px = pxn;
                iv = ivn;
            } while ((b0 += 64) < total);
        }
        constexpr int N = (3 * NC <= 16) ? 16 : 32;
        double x[N];
#pragma unroll
        for (int j = 0; j < N; ++j) x[j] = 0.0;
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            x[j] = S[j];
            x[NC + j] = A[j] + (double)(used - notin[j]);
            x[2 * NC + j] = V[j];
        }
        const WaveTotals<N> T(x);
        double Sin = 0, Ain = 0, Sout = 0, Aout = 0;
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            S[j] = T.total(j);
            A[j] = T.total(NC + j);
            V[j] = T.total(2 * NC + j);
            const int role = a.crole[j];
            if (role == kMaxRadii) {
                Sin = S[j];
                Ain = A[j];
            } else if (role == kMaxRadii + 1) {
                Sout = S[j];
                Aout = A[j];
            }
        }
        const double Aa = Aout - Ain, Sa = Sout - Sin;
        const double bk = (Aa > 0.0) ? Sa / Aa : 0.0;
        if (lane == 0) {
            const int nr = a.nr;
#pragma unroll
            for (int j = 0; j < NC; ++j) {
                const int q = a.crole[j];
                if (q < nr) {
                    cat.area[(size_t)row * nr + q] = A[j];
                    cat.flux[(size_t)row * nr + q] = S[j] - bk * A[j];
                    if (a.want_err && cat.fluxerr) cat.fluxerr[(size_t)row * nr + q] = sqrt(fmax(V[j], 0.0));
                }
            }
            cat.bkg[row] = bk;
            const double rm = (double)a.rmax;
            if (xc - rm < -0.5 || xc + rm > (double)d.W - 0.5 || yc - rm < -0.5 || yc + rm > (double)d.H - 0.5)
                cat.flags[row] |= kFlagTrunc;
        }
    }
}

template <typename Real, int NC>
static void launch_ap_nc(const FrameDesc* desc, const FrameDesc* one, const ApArgs& a, const ApCat& cat, int blocks,
                         int side, int nixmax, hipStream_t s) {
    const ApLayout<Real, NC> L(side);
    // waves per workgroup: as many (up to kApWaves) as keep the workgroup's
    // LDS within 64 KB; the grid keeps the same number of wavefronts
    const size_t pre = (size_t)ap_prefix_bytes(a.nframes);
    int nw = kApWaves;
    while (nw > 1 && pre + (size_t)L.bytes * nw > 64 * 1024) nw >>= 1;
    const size_t lds = pre + (size_t)L.bytes * nw;
    const int wg = blocks * (kApWaves / nw);
    const int g = kXcds * std::max(1, (wg + kXcds - 1) / kXcds);
    if (one) k_aperture<Real, NC, true><<<g, 64 * nw, lds, s>>>(desc, *one, a, cat, nixmax);
    else k_aperture<Real, NC, false><<<g, 64 * nw, lds, s>>>(desc, FrameDesc{}, a, cat, nixmax);
}

template <typename Real>
static void launch_ap_t(const FrameDesc* desc, const FrameDesc* one, const ApArgs& a, const ApCat& cat, int blocks,
                        int side, int nixmax, hipStream_t s) {
    switch (a.nr + 2) {
        case 3: launch_ap_nc<Real, 3>(desc, one, a, cat, blocks, side, nixmax, s); break;
        case 4: launch_ap_nc<Real, 4>(desc, one, a, cat, blocks, side, nixmax, s); break;
        case 5: launch_ap_nc<Real, 5>(desc, one, a, cat, blocks, side, nixmax, s); break;
        case 6: launch_ap_nc<Real, 6>(desc, one, a, cat, blocks, side, nixmax, s); break;
        case 7: launch_ap_nc<Real, 7>(desc, one, a, cat, blocks, side, nixmax, s); break;
        case 8: launch_ap_nc<Real, 8>(desc, one, a, cat, blocks, side, nixmax, s); break;
        case 9: launch_ap_nc<Real, 9>(desc, one, a, cat, blocks, side, nixmax, s); break;
        default: launch_ap_nc<Real, 10>(desc, one, a, cat, blocks, side, nixmax, s); break;
    }
}

// Pieces a box of `side` columns can touch: knots are one mesh apart except
// the last, which is at least half a mesh from its neighbour, so at most
// (side - 1) / mesh + 2 knots fall inside and the box spans one more piece.
static int ap_nixmax(int side, int mesh, int nmesh) {
    return std::max(1, std::min(nmesh + 1, (side - 1) / std::max(mesh, 1) + 3));
}

void launch_aperture(const FrameDesc* desc, const FrameDesc* one, const ApArgs& a, const ApCat& cat, int total_rows,
                     int blocks, int mesh_w, int max_nx, bool f64, hipStream_t s) {
    if (total_rows <= 0) return;
    const int R = (int)ceilf(a.rmax) + 1;
    const int side = 2 * R + 2;
    const int nixmax = ap_nixmax(side, mesh_w, max_nx);
    if (f64) launch_ap_t<double>(desc, one, a, cat, blocks, side, nixmax, s);
    else launch_ap_t<float>(desc, one, a, cat, blocks, side, nixmax, s);
}

}  // namespace gpk
