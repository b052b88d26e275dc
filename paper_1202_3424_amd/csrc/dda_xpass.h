// Passes 1 and 5 of the matrix-vector product (see dda_passes.h): scatter
// with the forward x transform, and the inverse x transform with gather,
// carrying the solvers' vector updates and inner products.
#pragma once

#include "dda_passcommon.h"

namespace dda {
namespace passes {

// threads of a compile-time x-pass workgroup: one wavefront up to length
// 128, two beyond (a line of 3 x 256 values gives one wavefront 12 elements
// per thread, which serialises its dependent map and site loads)
constexpr int xthr(int L) { return L > 128 ? 128 : 64; }

// ------------------------------------------------------------------ pass 1

// AL: the plain product's launch also forms the 1/alpha that its gather
// reads, in a layer of workgroups of its own behind the right-hand sides',
// instead of a launch before it (389 sites: 22.3 us a product so, 19.4 here).
struct NoAlpha {};
template <typename T, int MODE, int LC, int NTHR, typename AL = NoAlpha>
__global__ __launch_bounds__(NTHR) void k_scatter_x(Geo g, SiteArgs a, typename V2<T>::t* grid, const double2* tw64,
                                                   int XLrt, int chk, const AL al) {
    using C = typename V2<T>::t;
    constexpr bool CT = LC > 0;
    extern __shared__ __align__(16) unsigned char smem[];
    const int q = blockIdx.z;
    if constexpr (!std::is_same_v<AL, NoAlpha>) {
        if (q == a.nrhs) {
            const int b = blockIdx.y * gridDim.x + blockIdx.x;
            for (int i = b * NTHR + threadIdx.x; i < al.n; i += gridDim.x * gridDim.y * NTHR) alpha_entry(al, i);
            return;
        }
    }
    const RhsState* st = a.st + q;
    if constexpr (!CT) {
        if (skip_rhs(st, chk)) return;
    }
    // the box of the sites (and of the map): the volume's input window
    int nx = g.i1[0] - g.i0[0], ny = g.i1[1] - g.i0[1];
    const int xw = g.i0[0];
    const int* map = a.map;
    const int Mx = CT ? LC : g.M[0];
    const int My = g.M[1];
    const int XL = CT ? 1 : XLrt;
    const int z = blockIdx.y;
    const int y0 = blockIdx.x * XL;
    // the workgroups of one right-hand side along y, and its partial-sum index
    int bx = gridDim.x;
    if (a.rg) {   // ragged batch: this right-hand side's target
        const RhsGeo& r = a.rg[q];
        if (z >= r.n[2] || y0 >= r.n[1]) return;
        nx = r.n[0];
        ny = r.n[1];
        map += r.map_off;
        bx = (ny + XL - 1) / XL;
    }
    const int nl = CT ? 1 : min(XL, ny - y0);
    const int nlines = 3 * nl;
    const int Lp = pad_len(Mx);
    C* lds;
    C* tws = nullptr;
    if constexpr (CT) {
        lds = (C*)smem;
    } else {
        tws = (C*)smem;
        lds = tws + even_up(Mx);
        load_twiddles<T, NTHR>(tws, tw64, g.ax[0]);
    }
    double2 beta = {0, 0}, omega = {0, 0}, alpha = {0, 0};
    double w_old = 0.0, w_new = 0.0;
    int pend = 0;
    if (MODE == SC_P) { beta = st->beta; omega = st->omega; alpha = st->alpha; pend = st->pend; }
    if (MODE == SC_S) alpha = st->alpha;
    if (MODE == SC_Q) { alpha = st->alpha; beta = st->beta; w_old = st->w_old; w_new = st->w_new; }
    if (MODE == SC_B0 || MODE == SC_B2) beta = st->beta;
    if (MODE == SC_B1 || MODE == SC_B3) alpha = st->alpha;
    const long long vb = (long long)q * a.n3;
    const int* mrow = map + ((long long)z * ny + y0) * nx;
    double ss[3] = {0.0, 0.0, 0.0};
    // forward transform of a line that is zero beyond xw + nx: with twice that <= Mx the
    // first radix pass never reads the upper half, which is then not filled
    // (always so at the compile-time lengths, which are even and >= 2 nx - 1)
    bool hin = false;
    if constexpr (CT) hin = ct_half_in_ok(LC) && 2 * (xw + nx) <= Mx;
    const int ext = hin ? Mx / 2 : Mx;
    const int tin = nl * ext * 3;
    // the site-vector values this mode reads at element i (all of them are
    // loaded before any update is stored, so that the loads of every element
    // a thread fills are in flight together)
    struct Ops {
        double2 o[6];
    };
    // element (site s, component c) of this mode's vectors: the plain
    // product may take its input in the caller's site order
    auto elem = [&](int s, int c) -> long long {
        if (MODE == SC_PLAIN && a.perm) s = a.perm[s];
        return vb + (long long)s * 3 + c;
    };
    auto load_ops = [&](long long i) {
        Ops v;
        if (MODE == SC_PLAIN || MODE == SC_CONJ) {
            v.o[0] = a.in[i];
        } else if (MODE == SC_P) {
            v.o[0] = a.r[i]; v.o[1] = a.p[i]; v.o[2] = a.v[i]; v.o[3] = a.x[i]; v.o[4] = a.t[i];
        } else if (MODE == SC_B0) {
            v.o[0] = a.r[i]; v.o[1] = a.p[i];
        } else if (MODE == SC_B1) {
            v.o[0] = a.r[i]; v.o[1] = a.v[i]; v.o[2] = a.x[i]; v.o[3] = a.p[i];
        } else if (MODE == SC_B2) {
            v.o[0] = a.r[i]; v.o[1] = a.p[i]; v.o[2] = a.t[i]; v.o[3] = a.v[i];
        } else if (MODE == SC_B3) {
            v.o[0] = a.r[i]; v.o[1] = a.v[i]; v.o[2] = a.t[i]; v.o[3] = a.u2[i]; v.o[4] = a.x[i]; v.o[5] = a.p[i];
        } else if (MODE == SC_Q) {
            v.o[0] = a.r[i]; v.o[1] = a.p[i]; v.o[2] = a.rhat[i]; v.o[3] = a.t[i]; v.o[4] = a.x[i];
        } else {   // SC_S
            v.o[0] = a.r[i]; v.o[1] = a.v[i]; v.o[2] = a.rhat[i];
        }
        return v;
    };
    // the product's input at element i after this mode's vector update from
    // the loaded values v, the update stored back (and summed) only where
    // `live` (a site of this line; elsewhere the value is unused)
    auto update = [&](long long i, const Ops& v, bool live) -> double2 {
        double2 u;
        if (MODE == SC_PLAIN) {
            u = v.o[0];
        } else if (MODE == SC_CONJ) {
            u = cconj(v.o[0]);
        } else if (MODE == SC_P) {
            // the previous iteration's end, if pending: x += alpha p + omega
            // s, r = s - omega t (s is held in r); then p = r + beta (p -
            // omega v)
            double2 rr = v.o[0];
            const double2 pp = v.o[1];
            if (pend) {
                const double2 xx = cadd(cadd(v.o[3], cmul(alpha, pp)), cmul(omega, rr));
                rr = csub(rr, cmul(omega, v.o[4]));
                if (live) {
                    a.x[i] = xx;
                    a.r[i] = rr;
                }
            }
            u = cadd(rr, cmul(beta, csub(pp, cmul(omega, v.o[2]))));
            if (live) a.p[i] = u;
        } else if (MODE == SC_B0) {
            // BiCGstab(2), first BiCG step: u_0 = r_0 - beta u_0
            u = csub(v.o[0], cmul(beta, v.o[1]));
            if (live) a.p[i] = u;
        } else if (MODE == SC_B1) {
            // r_0 -= alpha u_1, x += alpha u_0; product of r_0
            u = csub(v.o[0], cmul(alpha, v.o[1]));
            if (live) {
                a.r[i] = u;
                a.x[i] = cadd(v.o[2], cmul(alpha, v.o[3]));
            }
        } else if (MODE == SC_B2) {
            // second BiCG step: u_0 = r_0 - beta u_0, u_1 = r_1 - beta u_1; product of u_1
            u = csub(v.o[2], cmul(beta, v.o[3]));
            if (live) {
                a.p[i] = csub(v.o[0], cmul(beta, v.o[1]));
                a.v[i] = u;
            }
        } else if (MODE == SC_B3) {
            // r_0 -= alpha u_1, r_1 -= alpha u_2, x += alpha u_0; product of r_1
            u = csub(v.o[2], cmul(alpha, v.o[3]));
            if (live) {
                a.r[i] = csub(v.o[0], cmul(alpha, v.o[1]));
                a.t[i] = u;
                a.x[i] = cadd(v.o[4], cmul(alpha, v.o[5]));
            }
        } else if (MODE == SC_Q) {
            // QMR: the previous iteration's x += alpha p (p = 0 after a
            // start), the pending smoothing step (y, s) <- w_old (y, s) +
            // w_new (x, r), and p = r + beta p
            const double2 rr = v.o[0];
            u = cadd(rr, cmul(beta, v.o[1]));
            if (live) {
                const double2 sm = v.o[2], ym = v.o[3];
                const double2 xx = cadd(v.o[4], cmul(alpha, v.o[1]));
                a.x[i] = xx;
                a.p[i] = u;
                a.rhat[i] = double2{w_old * sm.x + w_new * rr.x, w_old * sm.y + w_new * rr.y};
                a.t[i] = double2{w_old * ym.x + w_new * xx.x, w_old * ym.y + w_new * xx.y};
            }
        } else {
            // s = r - alpha v, stored over r; |s|^2 and <rhat, s>
            u = csub(v.o[0], cmul(alpha, v.o[1]));
            if (live) {
                const double2 w = cdotc(v.o[2], u);
                a.r[i] = u;
                ss[0] += u.x * u.x + u.y * u.y;
                ss[1] += w.x;
                ss[2] += w.y;
            }
        }
        return u;
    };
    if constexpr (CT) {
        // one line: the site indices of every element this thread fills are
        // loaded first, then every operand (clamped to site 0 where there is
        // no site), so that the loads of all elements are in flight together
        constexpr int EXT = ct_half_in_ok(LC) ? LC / 2 : LC;
        constexpr int NPT = (3 * EXT + NTHR - 1) / NTHR;
        int sk[NPT];
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int idx = threadIdx.x + k * NTHR;
            const int e = idx / 3 - xw;
            sk[k] = (idx < tin && (unsigned)e < (unsigned)nx) ? mrow[e] : -1;
        }
        // (the status and the map are loaded together: a small launch is a
        // chain of load latencies)
        if (skip_rhs(st, chk)) return;
        Ops ok[NPT];
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int idx = threadIdx.x + k * NTHR;
            ok[k] = load_ops(elem(sk[k] >= 0 ? sk[k] : 0, idx % 3));
        }
        double2 uk[NPT];
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int idx = threadIdx.x + k * NTHR;
            const bool live = sk[k] >= 0;
            uk[k] = update(MODE == SC_PLAIN ? 0 : elem(live ? sk[k] : 0, idx % 3), ok[k], live);
        }
#pragma unroll
        for (int k = 0; k < NPT; ++k) {
            const int idx = threadIdx.x + k * NTHR;
            if (idx < tin) {
                C val;
                val.x = 0;
                val.y = 0;
                if (sk[k] >= 0) val = to_c<C>(uk[k]);
                lds[(idx % 3) * Lp + idx / 3] = val;
            }
        }
        // (a full-length input, never the case at these even lengths: zeros
        // beyond the half)
        for (int idx = 3 * EXT + threadIdx.x; idx < tin; idx += NTHR) {
            C val;
            val.x = 0;
            val.y = 0;
            lds[(idx % 3) * Lp + idx / 3] = val;
        }
    } else {
        const Divisor de(ext);
        for (int idx = threadIdx.x; idx < tin; idx += NTHR) {
            const int c = idx % 3;
            const int rest = idx / 3;
            const int yo = de.quot(rest);
            const int e = rest - yo * ext;
            C val;
            val.x = 0;
            val.y = 0;
            if ((unsigned)(e - xw) < (unsigned)nx) {
                const int s = mrow[yo * nx + e - xw];
                if (s >= 0) {
                    const long long i = elem(s, c);
                    val = to_c<C>(update(i, load_ops(i), true));
                }
            }
            lds[(yo * 3 + c) * Lp + e] = val;
        }
    }
    __syncthreads();
    C* gq = grid + ((long long)q * g.npts + ((long long)(g.i0[2] + z) * My + g.i0[1] + y0) * Mx) * 3;
    if constexpr (CT) {
        // the last pass writes the grid itself
        auto store = line_io([&](int line, int e, const C& v) { gq[e * 3 + line] = v; });
        if (hin) fft_lines_ct<T, -1, LC, 3, NTHR, true, false>(lds, tw64 + g.ax[0].tw, NoIO(), store);
        else fft_lines_ct<T, -1, LC, 3, NTHR>(lds, tw64 + g.ax[0].tw, NoIO(), store);
    } else {
        fft_lines<T, -1, NTHR>(lds, tws, nlines, Lp, g.ax[0]);
        const int tot = nl * Mx * 3;
        const Divisor dm(Mx);
        for (int idx = threadIdx.x; idx < tot; idx += NTHR) {
            const int c = idx % 3;
            const int rest = idx / 3;
            const int yo = dm.quot(rest);
            const int e = rest - yo * Mx;
            gq[idx] = lds[(yo * 3 + c) * Lp + e];
        }
    }
    if (MODE == SC_S) {
        // slots 5-7 of the block's entry; the gather of t (same grid) fills
        // slots 0-4 and one finalize reads both
        double* sh = (double*)(lds + nlines * Lp);
        const int blk = blockIdx.y * bx + blockIdx.x;
        publish_partial<3, NTHR, 5>(ss, a.partials + (long long)q * a.maxblk * PSTRIDE, blk, a.maxblk, sh);
    }
}

// ------------------------------------------------------------------ pass 5

// PRE (compile-time lengths): each element's site operands are loaded
// before the inverse transform, so their latency overlaps it, at the price
// of the registers that hold them (fewer waves per SIMD); else after it.
template <typename T, int MODE, int LC, int NTHR, bool PRE = false>
__global__ __launch_bounds__(NTHR) void k_gather_x(Geo g, SiteArgs a, const typename V2<T>::t* grid,
                                                  const double2* tw64, int XLrt, int chk) {
    using C = typename V2<T>::t;
    constexpr bool CT = LC > 0;
    extern __shared__ __align__(16) unsigned char smem[];
    const int q = blockIdx.z;
    const RhsState* st = a.st + q;
    if constexpr (!CT) {
        if (skip_rhs(st, chk)) return;
    }
    int nx = g.n[0], ny = g.n[1];
    const int* map = a.map;
    const int* mat = a.mat;
    const int Mx = CT ? LC : g.M[0];
    const int My = g.M[1];
    const int XL = CT ? 1 : XLrt;
    const int z = blockIdx.y;
    const int y0 = blockIdx.x * XL;
    int bx = gridDim.x;
    if (a.rg) {   // ragged batch: this right-hand side's target
        const RhsGeo& r = a.rg[q];
        if (z >= r.n[2] || y0 >= r.n[1]) return;
        nx = r.n[0];
        ny = r.n[1];
        map += r.map_off;
        mat += r.site_off;
        bx = (ny + XL - 1) / XL;
    }
    const int nl = CT ? 1 : min(XL, ny - y0);
    const int nlines = 3 * nl;
    const int Lp = pad_len(Mx);
    C* lds;
    C* tws = nullptr;
    if constexpr (CT) {
        lds = (C*)smem;
    } else {
        tws = (C*)smem;
        lds = tws + even_up(Mx);
        load_twiddles<T, NTHR>(tws, tw64, g.ax[0]);
    }
    const int* mrow = map + ((long long)z * ny + y0) * nx;
    const int tout = nl * nx * 3;
    // compile-time lengths (one line per workgroup): the site index and
    // material of each element this thread gathers are loaded before the
    // transform, so only the operand loads follow it (e < nx <= (L + 1) / 2
    // since L >= 2 nx - 1).  The material with 128 right-hand sides of 18,432
    // sites: 104 us here, 106 after the transform.
    constexpr int PF = CT ? (3 * ((LC + 1) / 2) + NTHR - 1) / NTHR : 1;
    int ps[PF];
    if constexpr (CT) {
#pragma unroll
        for (int k = 0; k < PF; ++k) {
            const int idx = threadIdx.x + k * NTHR;
            // (a field is gathered at every point, in box-scan order)
            if (MODE == GA_FIELD) ps[k] = idx < tout ? (z * ny + y0) * nx + idx / 3 : -1;
            else ps[k] = idx < tout ? mrow[idx / 3] : -1;
        }
        if (skip_rhs(st, chk)) return;   // (as in k_scatter_x)
    }
    const C* gq = grid + ((long long)q * g.npts + ((long long)z * My + y0) * Mx) * 3;
    // (compile-time lengths: the first pass reads the grid itself)
    if constexpr (!CT) {
        const int tot = nl * Mx * 3;
        const Divisor dm(Mx);
        for (int idx = threadIdx.x; idx < tot; idx += NTHR) {
            const int c = idx % 3;
            const int rest = idx / 3;
            const int yo = dm.quot(rest);
            const int e = rest - yo * Mx;
            lds[(yo * 3 + c) * Lp + e] = gq[idx];
        }
    }
    // the site operands of the gathered elements (what each mode reads
    // besides the product), loaded before the transform so that their
    // latency overlaps it
    const long long vb = (long long)q * a.n3;
    auto elem = [&](int s, int c) -> long long {   // (see k_scatter_x)
        if (MODE == GA_PLAIN && a.perm) s = a.perm[s];
        return vb + (long long)s * 3 + c;
    };
    auto operand = [&](long long i) -> double2 {
        if (MODE == GA_PLAIN || MODE == GA_CONJ) return a.in[i];
        if (MODE == GA_V || MODE == GA_Q) return a.p[i];
        if (MODE == GA_T || MODE == GA_B1) return a.r[i];
        if (MODE == GA_RES) return a.x[i];
        if (MODE == GA_B2) return a.v[i];
        return a.t[i];   // GA_B3
    };
    constexpr bool HAS_AUX = MODE == GA_V || MODE == GA_T || MODE == GA_B1 || MODE == GA_B2 || MODE == GA_B3 ||
                             MODE == GA_RES;
    auto auxiliary = [&](long long i) -> double2 {
        if (MODE == GA_RES) return a.b[i];
        if (MODE == GA_B3) return a.r[i];
        return a.rhat[i];
    };
    int pm[PF];
    double2 px[PF], pa[PF];
    // (clamped to site 0 where there is no site: the values are unused)
    if constexpr (CT && MODE != GA_FIELD) {
#pragma unroll
        for (int k = 0; k < PF; ++k) pm[k] = mat[ps[k] >= 0 ? ps[k] : 0];
    }
    if constexpr (CT && PRE && MODE != GA_FIELD) {
#pragma unroll
        for (int k = 0; k < PF; ++k) {
            const int idx = threadIdx.x + k * NTHR;
            const long long i = elem(ps[k] >= 0 ? ps[k] : 0, idx % 3);
            px[k] = operand(i);
            pa[k] = HAS_AUX ? auxiliary(i) : double2{0.0, 0.0};
        }
    }
    if constexpr (CT) {
        auto load = line_io([&](int line, int e) { return gq[e * 3 + line]; });
        // only e < nx is gathered: with 2 nx <= Mx the last pass skips the upper half
        if (ct_half_out_ok(LC) && 2 * nx <= Mx)
            fft_lines_ct<T, 1, LC, 3, NTHR, false, true>(lds, tw64 + g.ax[0].tw, load);
        else
            fft_lines_ct<T, 1, LC, 3, NTHR>(lds, tw64 + g.ax[0].tw, load);
    } else {
        __syncthreads();
        fft_lines<T, 1, NTHR>(lds, tws, nlines, Lp, g.ax[0]);
    }

    const double2* ai = a.ainv + (long long)q * a.nmat * 3;
    double acc[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    // element (line yo, point e, component c) at site s of material mt, with
    // its operand xo and auxiliary vector value xa (as loaded)
    auto site = [&](int c, int e, int yo, int s, int mt, double2 xo, double2 xa) {
        const long long i = elem(s, c);
        const double2 gv = to_d(lds[(yo * 3 + c) * Lp + e]);
        if constexpr (MODE == GA_FIELD) {   // the scattered field: no diagonal
            a.out[i] = double2{-gv.x, -gv.y};
            return;
        }
        const double2 d = ai[mt * 3 + c];
        const double2 xin = MODE == GA_CONJ ? cconj(xo) : xo;
        const double2 y = cadd(gv, cmul(d, xin));
        if (MODE == GA_PLAIN) {
            a.out[i] = y;
        } else if (MODE == GA_CONJ) {
            const double2 yc = cconj(y);
            a.out[i] = yc;
            acc[0] += yc.x * yc.x + yc.y * yc.y;
        } else if (MODE == GA_V) {
            a.v[i] = y;
            const double2 w = cdotc(xa, y);
            acc[0] += w.x;
            acc[1] += w.y;
            acc[2] += y.x * y.x + y.y * y.y;   // |v|^2: bounds <rhat, v> with |rhat|
        } else if (MODE == GA_T) {
            a.t[i] = y;
            const double2 w = cdotc(y, xin);    // <t, s>
            const double2 wr = cdotc(xa, y);    // <rhat, t>
            acc[0] += w.x;
            acc[1] += w.y;
            acc[2] += y.x * y.x + y.y * y.y;
            acc[3] += wr.x;
            acc[4] += wr.y;
        } else if (MODE == GA_Q) {
            a.v[i] = y;
            acc[0] += xin.x * y.x - xin.y * y.y;   // p^T v (bilinear)
            acc[1] += xin.x * y.y + xin.y * y.x;
            acc[2] += y.x * y.x + y.y * y.y;       // |v|^2 and |p|^2 bound |p^T v|
            acc[3] += xin.x * xin.x + xin.y * xin.y;
        } else if (MODE == GA_B1 || MODE == GA_B2) {
            // r_1 = A r_0 or u_2 = A u_1, and <rhat, .>
            if (MODE == GA_B1) a.t[i] = y;
            else a.u2[i] = y;
            const double2 w = cdotc(xa, y);
            acc[0] += w.x;
            acc[1] += w.y;
            acc[2] += y.x * y.x + y.y * y.y;
        } else if (MODE == GA_B3) {
            // r_2 = A r_1 and the minimal-residual sums |r_1|^2, <r_1, r_2>,
            // |r_2|^2, <r_1, r_0>, <r_2, r_0>
            a.r2[i] = y;
            const double2 r0 = xa;
            const double2 w12 = cdotc(xin, y), w10 = cdotc(xin, r0), w20 = cdotc(y, r0);
            acc[0] += xin.x * xin.x + xin.y * xin.y;
            acc[1] += w12.x;
            acc[2] += w12.y;
            acc[3] += y.x * y.x + y.y * y.y;
            acc[4] += w10.x;
            acc[5] += w10.y;
            acc[6] += w20.x;
            acc[7] += w20.y;
        } else {
            const double2 rr = csub(xa, y);
            a.r[i] = rr;
            acc[0] += rr.x * rr.x + rr.y * rr.y;
        }
    };
    if constexpr (CT) {
#pragma unroll
        for (int k = 0; k < PF; ++k) {
            const int idx = threadIdx.x + k * NTHR;
            if (idx < tout && ps[k] >= 0) {
                if constexpr (MODE == GA_FIELD) {
                    site(idx % 3, idx / 3, 0, ps[k], 0, double2{0.0, 0.0}, double2{0.0, 0.0});
                } else if constexpr (PRE) {
                    site(idx % 3, idx / 3, 0, ps[k], pm[k], px[k], pa[k]);
                } else {
                    const long long i = elem(ps[k], idx % 3);
                    site(idx % 3, idx / 3, 0, ps[k], pm[k], operand(i),
                         HAS_AUX ? auxiliary(i) : double2{0.0, 0.0});
                }
            }
        }
    } else {
        const Divisor dx(nx);
        for (int idx = threadIdx.x; idx < tout; idx += NTHR) {
            const int c = idx % 3;
            const int rest = idx / 3;
            const int yo = dx.quot(rest);
            const int e = rest - yo * nx;
            if constexpr (MODE == GA_FIELD) {
                site(c, e, yo, (z * ny + y0 + yo) * nx + e, 0, double2{0.0, 0.0}, double2{0.0, 0.0});
                continue;
            }
            const int s = mrow[yo * nx + e];
            if (s >= 0) {
                const long long i = elem(s, c);
                site(c, e, yo, s, mat[s], operand(i), HAS_AUX ? auxiliary(i) : double2{0.0, 0.0});
            }
        }
    }
    if constexpr (MODE != GA_PLAIN && MODE != GA_FIELD) {
        double* sh = (double*)(lds + nlines * Lp);
        const int blk = blockIdx.y * bx + blockIdx.x;
        if constexpr (MODE == GA_B3) {
            publish_partial<8, NTHR>(acc, a.partials + (long long)q * a.maxblk * PSTRIDE, blk, a.maxblk, sh);
        } else if constexpr (MODE == GA_T) {
            double a5[5] = {acc[0], acc[1], acc[2], acc[3], acc[4]};
            publish_partial<5, NTHR>(a5, a.partials + (long long)q * a.maxblk * PSTRIDE, blk, a.maxblk, sh);
        } else if constexpr (MODE == GA_Q) {
            double a4[4] = {acc[0], acc[1], acc[2], acc[3]};
            publish_partial<4, NTHR>(a4, a.partials + (long long)q * a.maxblk * PSTRIDE, blk, a.maxblk, sh);
        } else {
            double a3[3] = {acc[0], acc[1], acc[2]};
            publish_partial<3, NTHR>(a3, a.partials + (long long)q * a.maxblk * PSTRIDE, blk, a.maxblk, sh);
        }
    }
}

// ------------------------------------------------------------------ launchers

template <typename T, int MODE, typename AL = NoAlpha>
void scatter_dispatch(int chk, const Geo& g, const SiteArgs& a, typename V2<T>::t* grid, const double2* tw,
                      hipStream_t s, const AL& al = AL()) {
    using C = typename V2<T>::t;
    const int L = g.M[0];
    const int XL = x_lines_per_tile(g, a.nrhs, sizeof(T) == 4);
    dim3 grd((g.i1[1] - g.i0[1] + XL - 1) / XL, g.i1[2] - g.i0[2], a.nrhs + (std::is_same_v<AL, NoAlpha> ? 0 : 1));
    switch (L) {
#define DDA_CASE(LL)                                                                                            \
    case LL:                                                                                                   \
        DDA_LAUNCH((k_scatter_x<T, MODE, LL, xthr(LL), AL>), grd, dim3(xthr(LL)), smem_ct<C>(LL, 3), s, g, a, grid, \
                           tw, 1, chk, al);                                                                        \
        return;
        DDA_CT_LENGTHS(DDA_CASE)
#undef DDA_CASE
        default:
            DDA_LAUNCH((k_scatter_x<T, MODE, 0, NT, AL>), grd, dim3(NT), smem_rt<C>(L, 3 * XL), s, g, a, grid,
                               tw, XL, chk, al);
    }
}

template <typename T, int MODE>
void gather_dispatch(int chk, const Geo& g, const SiteArgs& a, const typename V2<T>::t* grid, const double2* tw,
                     hipStream_t s) {
    using C = typename V2<T>::t;
    const int L = g.M[0];
    const int XL = x_lines_per_tile(g, a.nrhs, sizeof(T) == 4);
    dim3 grd((g.n[1] + XL - 1) / XL, g.n[2], a.nrhs);
    // operands before the transform pay in launches of few right-hand sides
    // (latency-bound workgroups); with many, the launch is bandwidth-bound
    // and the registers they take cost more occupancy than they save
    // (measured: 2-RHS solves gain, the 128-RHS brick loses 10%)
    const bool pre = a.nrhs <= 16;
    switch (L) {
#define DDA_CASE(LL)                                                                                            \
    case LL:                                                                                                   \
        if (pre)                                                                                               \
            DDA_LAUNCH((k_gather_x<T, MODE, LL, xthr(LL), true>), grd, dim3(xthr(LL)), smem_ct<C>(LL, 3), s, g, \
                       a, grid, tw, 1, chk);                                                                   \
        else                                                                                                   \
            DDA_LAUNCH((k_gather_x<T, MODE, LL, xthr(LL), false>), grd, dim3(xthr(LL)), smem_ct<C>(LL, 3), s,   \
                       g, a, grid, tw, 1, chk);                                                                \
        return;
        DDA_CT_LENGTHS(DDA_CASE)
#undef DDA_CASE
        default:
            DDA_LAUNCH((k_gather_x<T, MODE, 0, NT>), grd, dim3(NT), smem_rt<C>(L, 3 * XL), s, g, a, grid,
                               tw, XL, chk);
    }
}

}  // namespace passes

// ------------------------------------------------------------------ entry points

template <typename T>
void launch_scatter_x(int mode, int chk, const Geo& g, const SiteArgs& a, typename V2<T>::t* grid, const double2* tw,
                      hipStream_t s, const AlphaArgs* alpha) {
    using namespace passes;
    switch (mode) {
        case SC_PLAIN:
            if (alpha) scatter_dispatch<T, SC_PLAIN, AlphaArgs>(chk, g, a, grid, tw, s, *alpha);
            else scatter_dispatch<T, SC_PLAIN>(chk, g, a, grid, tw, s);
            break;
        case SC_CONJ: scatter_dispatch<T, SC_CONJ>(chk, g, a, grid, tw, s); break;
        case SC_P: scatter_dispatch<T, SC_P>(chk, g, a, grid, tw, s); break;
        case SC_Q: scatter_dispatch<T, SC_Q>(chk, g, a, grid, tw, s); break;
        case SC_B0: scatter_dispatch<T, SC_B0>(chk, g, a, grid, tw, s); break;
        case SC_B1: scatter_dispatch<T, SC_B1>(chk, g, a, grid, tw, s); break;
        case SC_B2: scatter_dispatch<T, SC_B2>(chk, g, a, grid, tw, s); break;
        case SC_B3: scatter_dispatch<T, SC_B3>(chk, g, a, grid, tw, s); break;
        default: scatter_dispatch<T, SC_S>(chk, g, a, grid, tw, s); break;
    }
}

template <typename T>
void launch_gather_x(int mode, int chk, const Geo& g, const SiteArgs& a, const typename V2<T>::t* grid,
                     const double2* tw, hipStream_t s) {
    using namespace passes;
    switch (mode) {
        case GA_PLAIN: gather_dispatch<T, GA_PLAIN>(chk, g, a, grid, tw, s); break;
        case GA_CONJ: gather_dispatch<T, GA_CONJ>(chk, g, a, grid, tw, s); break;
        case GA_V: gather_dispatch<T, GA_V>(chk, g, a, grid, tw, s); break;
        case GA_T: gather_dispatch<T, GA_T>(chk, g, a, grid, tw, s); break;
        case GA_Q: gather_dispatch<T, GA_Q>(chk, g, a, grid, tw, s); break;
        case GA_B1: gather_dispatch<T, GA_B1>(chk, g, a, grid, tw, s); break;
        case GA_B2: gather_dispatch<T, GA_B2>(chk, g, a, grid, tw, s); break;
        case GA_B3: gather_dispatch<T, GA_B3>(chk, g, a, grid, tw, s); break;
        case GA_FIELD: gather_dispatch<T, GA_FIELD>(chk, g, a, grid, tw, s); break;
        default: gather_dispatch<T, GA_RES>(chk, g, a, grid, tw, s); break;
    }
}

#define DDA_INSTANTIATE_XPASSES(T)                                                                                \
    template void launch_scatter_x<T>(int, int, const Geo&, const SiteArgs&, V2<T>::t*, const double2*,           \
                                      hipStream_t, const AlphaArgs*);                                            \
    template void launch_gather_x<T>(int, int, const Geo&, const SiteArgs&, const V2<T>::t*, const double2*,      \
                                     hipStream_t);

}  // namespace dda
