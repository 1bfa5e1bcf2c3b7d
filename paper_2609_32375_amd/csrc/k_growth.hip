// k_growth.hip -- growth curves on top-hat kernels.
//
// For each integer radius r_k the aperture sum of a source is the correlation
// of M = I - B with the top-hat kernel of radius r_k, read at the pixel that
// holds the source's centroid; the noise-map variance R^2 goes through the
// same taps, and every sum is FP64 (Adaptive Aperture Photometry subsection).
// A tap is the exact area of the disk of radius r_k about the kernel's middle
// pixel centre inside the tap's pixel.  The paper evaluates each radius as one
// full-frame correlation (FFT) and keeps its values at the sources; those are
// the values computed here, directly at the sources.
//
// The kernels are nested, so a pixel offset either lies wholly inside the disk
// from some radius on (it joins the running sums there with weight 1: the
// "full" list of that radius) or is cut by one or two circles (each takes it
// with its exact area: the "cut" lists).  sum_k = sum of the full lists j <= k
// plus the cut list k.  k_growth_table builds the lists once per call (FP64
// areas, raster order within each list); k_growth copies them to LDS.
//
// One wavefront per source: it evaluates M (and R^2) over the (2R+1)^2 window
// once into LDS from per-row background cubics, then walks the lists, lane e
// mod 64 taking entry e, and reduces the radii over the lanes in a fixed
// order, so a source's result does not depend on what else runs.  Bound by
// the latency of its LDS reads at the few wavefronts its windows leave room
// for: with 12 of them per compute unit for 8, the full lists read without a
// gap at each radius and one reduction per four radii for twelve butterflies,
// 20000 sources with 13 radii up to 15 took 151 us for 281.
#include "k_args.h"
#include "k_overlap.h"
#include "k_rowpoly.h"

namespace gpk {

constexpr int kGrMaxFrames = kMaxFramesPerCall;
constexpr int kGrPrefixBytes = (int)((sizeof(int32_t) * (kGrMaxFrames + 1) + 15) / 16 * 16);

// pixel offset classes of the nested top-hat kernels (exact in FP64: the
// squared distances are multiples of 1/4)
__device__ __forceinline__ void gr_class(int dx, int dy, double& dmin2, double& dmax2) {
    const double ax = fabs((double)dx), ay = fabs((double)dy);
    const double nx = fmax(ax - 0.5, 0.0), ny = fmax(ay - 0.5, 0.0);
    dmin2 = nx * nx + ny * ny;
    dmax2 = (ax + 0.5) * (ax + 0.5) + (ay + 0.5) * (ay + 0.5);
}

// One workgroup per list, list L < nr the full list of radius L, L >= nr the
// cut list of radius L - nr.  Its wavefronts scan consecutive quarters of the
// window in raster order twice, to count and then to place with ballots, so
// the order inside a list is the raster order; the exact areas then take one
// thread per cut pixel.  Bound by latency: one workgroup for all lists, with
// the areas inside its scan, took 44 us for 13 radii up to 15, now 6.
constexpr int kGrTabThreads = 256;
constexpr int kGrCutMax = 512;   // pixels a circle of radius <= 32 can cut (about 8 r)
__global__ __launch_bounds__(kGrTabThreads) void k_growth_table(GrowArgs a, GrowTab t) {
    __shared__ int32_t code[kGrCutMax];
    __shared__ int32_t cnt[kGrTabThreads / 64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    constexpr int nw = kGrTabThreads / 64;
    const uint64_t below = (lane == 0) ? 0ull : ((~0ull) >> (64 - lane));
    const int side = a.side, R = a.R, n2 = side * side;
    const int L = blockIdx.x;
    const bool full = L < a.nr;
    const int k = full ? L : L - a.nr;
    const double r = (double)a.radii[k], r2 = r * r;
    const double rp2 = (k > 0) ? (double)a.radii[k - 1] * (double)a.radii[k - 1] : -1.0;
    const int beg = full ? a.full_off[k] : a.cut_off[k];
    const int n = (full ? a.full_off[k + 1] : a.cut_off[k + 1]) - beg;
    const int per = (n2 + 64 * nw - 1) / (64 * nw) * 64;   // pixels per wavefront
    auto scan = [&](auto&& place) {
        int run = 0;
        for (int b = wv * per; b < min(n2, (wv + 1) * per); b += 64) {
            const int i = b + lane;
            bool take = false;
            int wy = 0, wx = 0;
            if (i < n2) {
                double dmin2, dmax2;
                wy = (int)(((uint32_t)i * (uint32_t)a.div_magic) >> 20);
                wx = i - wy * side;
                gr_class(wx - R, wy - R, dmin2, dmax2);
                take = full ? (dmax2 <= r2 && dmax2 > rp2) : (dmin2 < r2 && r2 < dmax2);
            }
            const uint64_t bm = __ballot(take);
            if (take) place(run + __popcll(bm & below), (wy << 16) | wx);
            run += __popcll(bm);
        }
        return run;
    };
    const int mine = scan([](int, int) {});
    if (lane == 0) cnt[wv] = mine;
    __syncthreads();
    int first = 0;
    for (int i = 0; i < wv; ++i) first += cnt[i];
    scan([&](int pos, int c) {
        const int q = first + pos;
        if (q >= n) return;
        if (full) {
            t.full[beg + q] = c;
        } else {
            t.cut[beg + q] = c;
            if (q < kGrCutMax) code[q] = c;
        }
    });
    if (full) return;
    __syncthreads();
    for (int q = threadIdx.x; q < min(n, kGrCutMax); q += kGrTabThreads)
        t.cutw[beg + q] = pixel_area<double>((double)((code[q] & 0xffff) - R), (double)((code[q] >> 16) - R), r, r2);
}

template <typename Real>
struct GrLayout {
    int o_full, o_cut, o_cutw, shared;   // table (whole workgroup), after the frame prefix
    int o_m, o_v, o_tab, o_colp, o_cols, wave;   // per wavefront
    __host__ __device__ GrLayout(int nfull, int ncut, int side, int nixmax, int want_var) {
        int o = kGrPrefixBytes;
        auto take = [&](int n, int al) {
            o = (o + al - 1) / al * al;
            const int r = o;
            o += n;
            return r;
        };
        o_full = take(4 * nfull, 16);
        o_cut = take(4 * ncut, 16);
        o_cutw = take(8 * ncut, 16);
        shared = (o + 15) / 16 * 16;
        o = 0;
        o_m = take(side * side * (int)sizeof(Real), 16);
        o_v = take(want_var ? side * side * (int)sizeof(Real) : 0, 16);
        o_tab = take(side * nixmax * (int)sizeof(RowT<Real>), 16);
        o_colp = take(side * 4, 16);
        o_cols = take(side * (int)sizeof(Real), 16);
        wave = (o + 15) / 16 * 16;
    }
};

constexpr int kGrUnroll = 4;   // window pixels per lane in flight

template <typename Real, bool ONE>
__global__ __launch_bounds__(64 * kGrowMaxWaves) void k_growth(const FrameDesc* __restrict__ desc, FrameDesc d1, GrowArgs a,
                                                GrowTab t, GrowOut g) {
    extern __shared__ __align__(16) unsigned char gr_dyn[];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int side = a.side, R = a.R, n2 = side * side, nixmax = a.nixmax, nr = a.nr;
    const GrLayout<Real> L(a.nfull, a.ncut, side, nixmax, a.want_var);
    int32_t* fpre = reinterpret_cast<int32_t*>(gr_dyn);
    int32_t* fl = (int32_t*)(gr_dyn + L.o_full);
    int32_t* cl = (int32_t*)(gr_dyn + L.o_cut);
    double* cw = (double*)(gr_dyn + L.o_cutw);
    unsigned char* base = gr_dyn + L.shared + (size_t)wv * L.wave;
    Real* Mw = (Real*)(base + L.o_m);
    Real* Vw = (Real*)(base + L.o_v);
    RowT<Real>* tab = (RowT<Real>*)(base + L.o_tab);
    int32_t* colp = (int32_t*)(base + L.o_colp);
    Real* cols = (Real*)(base + L.o_cols);

    for (int i = threadIdx.x; i < a.nfull; i += blockDim.x) fl[i] = t.full[i];
    for (int i = threadIdx.x; i < a.ncut; i += blockDim.x) {
        cl[i] = t.cut[i];
        cw[i] = t.cutw[i];
    }
    const int nf = a.nframes;
    if (wv == 0) {
        // prefix of min(n_obj, capacity) over the frames (one wavefront)
        constexpr int PER = kGrMaxFrames / 64;
        int tot = 0;
        for (int q = 0; q < PER; ++q) {
            const int fr = lane * PER + q;
            if (fr < nf) tot += min(g.n_obj[fr], a.capacity);
        }
        int incl = tot;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(incl, o);
            if (lane >= o) incl += y;
        }
        int run = incl - tot;
        for (int q = 0; q < PER; ++q) {
            const int fr = lane * PER + q;
            fpre[fr] = run;
            if (fr < nf) run += min(g.n_obj[fr], a.capacity);
        }
        if (lane == 63) fpre[kGrMaxFrames] = incl;
    }
    __syncthreads();
    const int total = fpre[kGrMaxFrames];
    // sources of all frames, numbered consecutively, in 8 contiguous ranges
    // (one per XCD): neighbouring sources, whose windows overlap, share an L2
    const int chunk = (total + kXcds - 1) / kXcds;
    const int xcd = blockIdx.x % kXcds, per_xcd = gridDim.x / kXcds;
    const int o_end = min(total, (xcd + 1) * chunk);
    for (int o = xcd * chunk + (blockIdx.x / kXcds) * nw + wv; o < o_end; o += per_xcd * nw) {
        int lo = 0, hi = nf - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (fpre[mid] <= o) lo = mid;
            else hi = mid - 1;
        }
        const int f = lo, row = f * a.capacity + (o - fpre[f]);
        const FrameDesc& d = ONE ? d1 : desc[f];
        const double fx = floor(g.x[row] + 0.5), fy = floor(g.y[row] + 0.5);
        // a pixel so far out that no tap reaches the frame (or not a number):
        // zero sums
        const bool reach = fx >= -(double)R - 1.0 && fx <= (double)d.W + R && fy >= -(double)R - 1.0 &&
                           fy <= (double)d.H + R;
        const int cx = reach ? (int)fx : 0, cy = reach ? (int)fy : 0;
        const int bx0 = cx - R, by0 = cy - R;
        // the frame inside the window, in window coordinates
        const int wx_lo = max(0, -bx0), wx_hi = min(side - 1, d.W - 1 - bx0);
        const int wy_lo = max(0, -by0), wy_hi = min(side - 1, d.H - 1 - by0);
        const bool any = reach && wx_lo <= wx_hi && wy_lo <= wy_hi;
        const bool inside = wx_lo == 0 && wy_lo == 0 && wx_hi == side - 1 && wy_hi == side - 1;   // the whole window
        double my_s = 0.0, my_v = 0.0, my_a = 0.0;
        if (any) {
            const int cx_lo = bx0 + wx_lo, cx_hi = bx0 + wx_hi;
            const int ixlo = piece_of(cx_lo, d.W, d.mw);
            const int nix = min(piece_of(cx_hi, d.W, d.mw) - ixlo + 1, nixmax);
            wave_sync();
            for (int c = lane; c < side; c += 64) {
                const int px = bx0 + c;
                if (px >= 0 && px < d.W) {
                    const int ix = piece_of(px, d.W, d.mw);
                    colp[c] = min(ix - ixlo, nixmax - 1);
                    cols[c] = (Real)((double)px - piece_ref(ix, d.W, d.mw));
                }
            }
            const int nrow = wy_hi - wy_lo + 1;
            for (int e = lane; e < nrow * nix; e += 64) {
                const int rr = e / nix, pi = e - rr * nix;
                const int py = by0 + wy_lo + rr;
                const int jy = piece_of(py, d.H, d.mh);
                const double u = (double)py - piece_ref(jy, d.H, d.mh);
                tab[(wy_lo + rr) * nixmax + pi] = make_row<Real>(d.coef, d.nx, d.ny, ixlo + pi, jy, u);
            }
            wave_sync();
            // M (and R^2) over the window; zero off the frame
            for (int b = 0; b < n2; b += 64 * kGrUnroll) {
                int wi[kGrUnroll], wyv[kGrUnroll], wxv[kGrUnroll];
                bool in[kGrUnroll];
                float iv[kGrUnroll];
#pragma unroll
                for (int u = 0; u < kGrUnroll; ++u) {
                    const int i = b + u * 64 + lane;
                    wi[u] = i;
                    const int wy = (int)(((uint32_t)i * (uint32_t)a.div_magic) >> 20);
                    const int wx = i - wy * side;
                    wyv[u] = wy;
                    wxv[u] = wx;
                    in[u] = i < n2 && wx >= wx_lo && wx <= wx_hi && wy >= wy_lo && wy <= wy_hi;
                    iv[u] = in[u] ? load_px(d, bx0 + wx, by0 + wy) : 0.0f;
                }
#pragma unroll
                for (int u = 0; u < kGrUnroll; ++u) {
                    if (wi[u] >= n2) continue;
                    Real m = (Real)0, v = (Real)0;
                    if (in[u]) {
                        const RowT<Real> T = tab[wyv[u] * nixmax + colp[wxv[u]]];
                        const Real sx = cols[wxv[u]];
                        m = eval_M(T, sx, (Real)iv[u]);
                        if (a.want_var) {
                            const Real rv = eval_R(T, sx);
                            v = rv * rv;
                        }
                    }
                    Mw[wi[u]] = m;
                    if (a.want_var) Vw[wi[u]] = v;
                }
            }
            wave_sync();
            // Sums: the full lists lie one after the other, so 64 entries at
            // a time are read whatever list they belong to; radius k takes
            // the whole rounds before its end and, of the round that holds
            // its end, the entries below it.  Four radii are reduced at once.
            auto entry = [&](int pk, double wt, double& m, double& v, double& ar) __attribute__((always_inline)) {
                const int wy = pk >> 16, wx = pk & 0xffff, w = wy * side + wx;
                m = wt * (double)Mw[w];
                v = a.want_var ? wt * (double)Vw[w] : 0.0;
                ar = inside || (wx >= wx_lo && wx <= wx_hi && wy >= wy_lo && wy <= wy_hi) ? wt : 0.0;
            };
            double sm = 0.0, sv = 0.0, sa = 0.0;   // this lane's share of the whole rounds so far
            double em, ev, ea;                     // and of the round that starts at entry at0
            int at0 = 0;
            auto round = [&]() __attribute__((always_inline)) {
                em = ev = ea = 0.0;
                if (at0 + lane < a.nfull) entry(fl[at0 + lane], 1.0, em, ev, ea);
            };
            round();
            for (int k0 = 0; k0 < nr; k0 += 4) {
                double x[16];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    x[q] = x[4 + q] = x[8 + q] = x[12 + q] = 0.0;
                    const int k = k0 + q;
                    if (k >= nr) continue;
                    const int end = a.full_off[k + 1];
                    while (at0 + 64 <= end) {
                        sm += em;
                        sv += ev;
                        sa += ea;
                        at0 += 64;
                        round();
                    }
                    const bool below = at0 + lane < end;
                    double cm = sm + (below ? em : 0.0), cv = sv + (below ? ev : 0.0), ca = sa + (below ? ea : 0.0);
                    for (int e = a.cut_off[k] + lane; e < a.cut_off[k + 1]; e += 64) {
                        double m, v, ar;
                        entry(cl[e], cw[e], m, v, ar);
                        cm += m;
                        cv += v;
                        ca += ar;
                    }
                    x[q] = cm;
                    x[4 + q] = cv;
                    x[8 + q] = ca;
                }
                const WaveTotals<16> T(x);
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const double ts = T.total(q), tv = T.total(4 + q), ta = T.total(8 + q);
                    if (lane == k0 + q) {
                        my_s = ts;
                        my_v = tv;
                        my_a = ta;
                    }
                }
            }
        }
        if (lane < nr) {
            g.sum[(size_t)row * nr + lane] = my_s;
            if (g.var) g.var[(size_t)row * nr + lane] = my_v;
            g.area[(size_t)row * nr + lane] = my_a;
        }
        if (lane == 0 && g.flags) {
            const bool trunc = !reach || cx - R < 0 || cx + R >= d.W || cy - R < 0 || cy + R >= d.H;
            g.flags[row] = trunc ? kFlagTrunc : 0u;
        }
    }
}

size_t growth_lds_bytes(int nfull, int ncut, int side, int nixmax, int want_var, bool f64, int waves) {
    if (f64) {
        const GrLayout<double> L(nfull, ncut, side, nixmax, want_var);
        return (size_t)L.shared + (size_t)L.wave * waves;
    }
    const GrLayout<float> L(nfull, ncut, side, nixmax, want_var);
    return (size_t)L.shared + (size_t)L.wave * waves;
}

void launch_growth_table(const GrowArgs& a, const GrowTab& t, hipStream_t s) {
    k_growth_table<<<2 * a.nr, kGrTabThreads, 0, s>>>(a, t);
}

template <typename Real>
static hipError_t launch_growth_t(const FrameDesc* desc, const FrameDesc* one, const GrowArgs& a, const GrowTab& t,
                                  const GrowOut& g, int blocks, int waves, hipStream_t s) {
    const size_t lds = growth_lds_bytes(a.nfull, a.ncut, a.side, a.nixmax, a.want_var, sizeof(Real) == 8, waves);
    const int grid = kXcds * std::max(1, (blocks + kXcds - 1) / kXcds);
    if (one) {
        hipError_t e = hipFuncSetAttribute((const void*)k_growth<Real, true>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        k_growth<Real, true><<<grid, 64 * waves, lds, s>>>(desc, *one, a, t, g);
    } else {
        hipError_t e = hipFuncSetAttribute((const void*)k_growth<Real, false>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        k_growth<Real, false><<<grid, 64 * waves, lds, s>>>(desc, FrameDesc{}, a, t, g);
    }
    return hipGetLastError();
}

hipError_t launch_growth(const FrameDesc* desc, const FrameDesc* one, const GrowArgs& a, const GrowTab& t,
                         const GrowOut& g, int blocks, int waves, bool f64, hipStream_t s) {
    if (f64) return launch_growth_t<double>(desc, one, a, t, g, blocks, waves, s);
    return launch_growth_t<float>(desc, one, a, t, g, blocks, waves, s);
}

}  // namespace gpk
