// Passes 2-4 of the product (y forward, z with the tensor product, y
// inverse; see dda_passes.h) as one kernel per kx plane, for grids whose
// (y, z) plane fits one compute unit's LDS.
//
// What bounds it.  Run as three kernels, the passes write and read the padded
// plane three times (ten line-grid volumes of traffic) and each waits for the
// one before it; here the plane is read once, kept in LDS through all three
// transforms and written once (two volumes).  What is left is the LDS traffic
// of the exchanges and the arithmetic of the transforms.
//
// Layout.  A workgroup owns one kx of one right-hand side: three component
// planes, element (ky, z) of component c at c * CS + ky * ZS + z, z < nz only
// (the z padding lives in registers).
// ZS is odd and CS = 3 mod 8 (FP64) or 5 mod 16 (FP32) in elements, so that
// both the lines along y (lanes over z and c) and the columns along z
// (lanes over ky) touch distinct banks.  Every line is handled by Q = L / P
// lanes of one wavefront (the register-resident passes of dda_device.h, the
// same butterflies and twiddles as every other form, so bitwise-identical
// results), and a line's exchange goes through that line's own LDS words:
// LDS instructions of one wavefront execute in order, so no exchange needs a
// workgroup barrier, and the kernel has two in all.
#pragma once

#include "dda_passes.h"

namespace dda {
namespace plane {

using passes::tw_table;

// VGPRs of line data per thread in the z stage (three components of P values)
template <typename T> constexpr int z_vgprs(int LZ) { return 3 * ct_split(LZ) * (int)(2 * sizeof(T) / 4); }

// LDS words (elements) of one column's exchange: element (j, f) of the
// first group's output, f < P, j < Q, at (f / FG) * CS + (f % FG) * Q + j:
// a third of the f in each of the column's three component segments.
constexpr int ex_group(int L) { return (ct_split(L) + 2) / 3; }
constexpr int ex_words(int L) { return ex_group(L) * (L / ct_split(L)); }

// z stride: odd, at least the occupied z extent and an exchange segment
constexpr int z_stride(int LZ, int nz) {
    return (nz > ex_words(LZ) ? nz : ex_words(LZ)) | 1;
}
// component stride: at least LY * ZS, = 3 mod 8 (FP64) or 5 mod 16 (FP32)
constexpr int c_stride(int LY, int ZS, bool f32) {
    return f32 ? LY * ZS + (5 + 16 - LY * ZS % 16) % 16 : LY * ZS + (3 + 8 - LY * ZS % 8) % 8;
}
constexpr size_t PLANE_LDS = 163840;   // 160 KB per compute unit

constexpr size_t plane_bytes(int LY, int LZ, int nz, bool f32) {
    return (size_t)3 * c_stride(LY, z_stride(LZ, nz), f32) * (f32 ? sizeof(float2) : sizeof(double2));
}

// Lengths with a plane kernel: their product at every occupied extent the
// padding rule gives them (at most L / 2 on each axis).  z: three components
// of a column to a thread, up to 144 VGPRs of data, which leaves two
// wavefronts per SIMD.
constexpr bool plane_y(int L) { return L == 32 || L == 48 || L == 64 || L == 80 || L == 96 || L == 128; }
template <typename T> constexpr bool plane_z(int LZ) { return plane_y(LZ) && z_vgprs<T>(LZ) <= 144; }
// pairs whose plane fits with the largest occupied z extent, LZ / 2
template <typename T> constexpr bool plane_pair(int LY, int LZ) {
    return plane_y(LY) && plane_z<T>(LZ) && plane_bytes(LY, LZ, LZ / 2, sizeof(T) == 4) <= PLANE_LDS;
}

// Wavefronts per workgroup: one per group of z columns a wavefront takes at
// once, at most eight (two per SIMD at the registers the z stage holds), with
// three measured exceptions, which depend on whether the launch has more
// workgroups than compute units (many) or each has one to itself:
//   FP64 48 x 32, whose 39 KB let four workgroups share a compute unit, two
//   if many (128 right-hand sides: 308 us against 346 with three; with two
//   right-hand sides a product takes a tenth longer with two);
//   FP32 96 x 64 and 96 x 128, twelve at three per SIMD (two right-hand sides:
//   25.1 us against 26.0 and 44.6 against 49.2 with eight);
//   FP32 with LZ = 80, eight for the y lines (80 x 80, twenty right-hand sides:
//   181 us against 193 with five), but with LY = 32 and 48 only if not many:
//   256 workgroups 19 us against 22 with two and 23 against 30 with three,
//   12,288 workgroups of 32 x 80 733 against 327 (537 as three passes).
template <typename T> constexpr int plane_waves(int LY, int LZ, bool many) {
    const int nz = LY * (LZ / ct_split(LZ)) / 64;   // groups of z columns
    if (sizeof(T) == 8) return (many && LZ == 32 && nz == 3) ? 2 : (nz < 8 ? nz : 8);
    if (nz == 12) return 12;
    if (LZ == 80 && (LY >= 64 || !many)) return 8;
    return nz < 8 ? nz : 8;
}
// wavefronts per SIMD asked of the compiler: three where that needs no
// spilling (FP32, at most 72 VGPRs of data) and whole workgroups of at most
// six wavefronts fill them (96 x 32, 3,072 workgroups: 155 us at two, 131 at
// three)
template <typename T> constexpr int plane_occ(int LZ, int waves) {
    return sizeof(T) == 4 && (waves == 12 || (waves <= 6 && z_vgprs<T>(LZ) <= 72)) ? 3 : 2;
}
constexpr int PLANE_ALONE = 256;   // compute units

// Planes that few workgroups do not take (plane_use): at most PLANE_MIN of
// them, an eighth of the compute units, and a chain per workgroup longer than
// the launches it saves.  A product in a solve here and with the three passes,
// us: FP64 4 workgroups of 128 x 48 50 and 39, of 96 x 64 49 and 38, 32 of 128
// x 48 44 and 36; but 16 of 32 x 64 0.98 and 32 of 128 x 32 1.00 of the time.
// FP32 4 of 128 x 96 74 and 56, 8 of 32 x 96 50 and 43, 32 of 128 x 96 61 and
// 54; but 40 of 48 x 64 0.94.  With 64 the two are within a tenth.
constexpr int PLANE_MIN = 32;
template <typename T> constexpr bool plane_long(int LY, int LZ) {
    return sizeof(T) == 8 ? LZ > 32 && LY * LZ > 3072 : LZ == 96 || LY * LZ >= 5120;
}

// Orders the LDS accesses of one wavefront for the compiler (the hardware
// executes them in order).
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One-dimensional launch: workgroup b runs on XCD b % 8 (round-robin).
// Neighbouring kx share cache lines of the grid, which should meet in one
// XCD's L2.  Where a sixteenth of the row, W = Mx / 16 points, is a run of at
// least 192 bytes, an XCD takes one such run of kx and its mirror run (they
// share tensor rows), every right-hand side in turn; with shorter runs (and
// extents that do not split so) it takes a contiguous part of the
// (right-hand side, kx) order.  Measured, us the first way and the second, the
// kernel launched back to back:
// FP64 Mx 32 39.5 and 34.0, 48 42.6 and 40.2, 64 94.6 and 95.7, 96 305 and
// 312, 128 32.0 and 35.8 (two right-hand sides); FP32 Mx 96 178 and 168.
template <typename T> __host__ __device__ constexpr bool plane_runs(int Mx) {
    return Mx % (2 * passes::N_XCD) == 0 && Mx / (2 * passes::N_XCD) * 3 * 2 * (int)sizeof(T) >= 192;
}
template <typename T> __device__ __forceinline__ bool plane_tile(int Mx, int nrhs, int& kx, int& q) {
    const int j = blockIdx.x % passes::N_XCD, local = blockIdx.x / passes::N_XCD;
    if (plane_runs<T>(Mx)) {
        const int W = Mx / (2 * passes::N_XCD);
        const int i = local % (2 * W);
        q = local / (2 * W);
        kx = i < W ? j * W + i : Mx - (j + 1) * W + (i - W);
        return true;
    }
    const int t = j * (gridDim.x / passes::N_XCD) + local;
    q = t / Mx;
    kx = t % Mx;
    return q < nrhs;
}
inline unsigned plane_grid(int Mx, int nrhs) {
    const long long n = (long long)Mx * nrhs;
    return (unsigned)((n + passes::N_XCD - 1) / passes::N_XCD * passes::N_XCD);
}

// gp: the tensor octant as [Hx][Hz][6][plane_row(LY)] (lanes over ky read
// consecutive values, rows on cache-line boundaries).
template <typename T, int LY, int LZ, int NTHR, int WV>
__global__ __launch_bounds__(NTHR) __attribute__((amdgpu_waves_per_eu(WV))) void k_plane(Geo g, typename V2<T>::t* grid, const double2* tw64,
                                               const typename V2<T>::t* gp, const RhsState* st, int chk, int nrhs,
                                               int ZS, int CS) {
    using C = typename V2<T>::t;
    constexpr int PY = ct_split(LY), QY = LY / PY;
    constexpr int PZ = ct_split(LZ), QZ = LZ / PZ;
    constexpr int LPW = 64 / QY;             // y lines per wavefront
    constexpr int CPW = 64 / QZ;             // z columns per wavefront
    constexpr int NW = NTHR / 64;
    constexpr int FG = ex_group(LZ);
    static_assert(LY % CPW == 0, "whole wavefronts of columns");
    extern __shared__ __align__(16) unsigned char smem[];
    C* lds = (C*)smem;
    const int Mx = g.M[0];
    int kx, q;
    if (!plane_tile<T>(Mx, nrhs, kx, q)) return;
    if (passes::skip_rhs(st + q, chk)) return;
    int ny = g.n[1], nz = g.n[2];
    if (g.rg) {   // ragged batch: this right-hand side's target
        const RhsGeo& r = g.rg[q];
        ny = r.n[1];
        nz = r.n[2];
        gp = (const C*)r.gplane[sizeof(C) == sizeof(float2) ? 1 : 0];
    }
    // the input window (all of the box but for a near-field volume)
    const int iy0 = g.i0[1], iy1 = g.rg ? ny : g.i1[1], iz0 = g.i0[2], iz1 = g.rg ? nz : g.i1[2];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const auto* twy = tw_table<T>(g, tw64) + g.ax[1].tw;
    const auto* twz = tw_table<T>(g, tw64) + g.ax[2].tw;
    C* gq = grid + (long long)q * g.npts * 3 + (long long)kx * 3;
    const int nlines = 3 * nz;
    const int yt = lane / LPW;
    const long long ys = (long long)Mx * 3;

    // ---- y forward: line (z, c3), lanes yt = 0 .. QY-1
    for (int l0 = wave * LPW; l0 < nlines; l0 += NW * LPW) {
        const int ln = l0 + lane % LPW;
        const int z = ln / 3, c3 = ln % 3;
        const bool live = ln < nlines, fed = z >= iz0 && z < iz1;
        const C* src = gq + (long long)z * LY * ys + c3;
        C v[1][PY];
#pragma unroll
        for (int m = 0; m < PY; ++m) {
            const int e = yt + QY * m;
            if (2 * m < PY && fed && e >= iy0 && e < iy1) {
                v[0][m] = src[(long long)e * ys];
            } else {
                v[0][m].x = 0;
                v[0][m].y = 0;
            }
        }
        rf_group_a<T, -1, LY, true, 1>(v, twy);
        C* row = lds + c3 * CS + z;
        if (live) {
#pragma unroll
            for (int f = 0; f < PY; ++f) row[(yt * PY + f) * ZS] = v[0][f];
        }
        wave_fence();
        if (live) {
#pragma unroll
            for (int c = 0; c < PY / QY; ++c) {
#pragma unroll
                for (int jj = 0; jj < QY; ++jj) v[0][c * QY + jj] = row[(jj * PY + yt + QY * c) * ZS];
            }
        }
        wave_fence();
        rf_group_b<T, -1, LY, false, 1>(v, yt, twy);
        if (live) {
#pragma unroll
            for (int c = 0; c < PY / QY; ++c) {
#pragma unroll
                for (int gg = 0; gg < QY; ++gg) row[(yt + QY * c + PY * gg) * ZS] = v[0][c * QY + gg];
            }
        }
    }
    __syncthreads();

    // ---- z forward, tensor product, z inverse: column ky, lanes zt
    const int zt = lane / CPW;
    // LDS offset of the values (j, f = zt + QZ c) this lane reads in an exchange
    int rd[PZ / QZ];
#pragma unroll
    for (int c = 0; c < PZ / QZ; ++c) {
        const int f = zt + QZ * c;
        rd[c] = (f / FG) * CS + (f % FG) * QZ;
    }
    constexpr int HY = plane_row(LY), Hz = LZ / 2 + 1;
    for (int c0 = wave * CPW; c0 < LY; c0 += NW * CPW) {
        const int cy = c0 + lane % CPW;
        // the upper half in mirrored order: its tensor rows then ascend with
        // the lane, as the lower half's do
        const bool uy = cy > LY / 2;
        const int fy = uy ? cy - LY / 2 : cy;
        const int ky = uy ? LY - fy : cy;
        C* cb = lds + ky * ZS;
        C v[3][PZ];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
#pragma unroll
            for (int m = 0; m < PZ; ++m) {
                const int e = zt + QZ * m;
                if (2 * m < PZ && e < nz) {
                    v[a][m] = cb[a * CS + e];
                } else {
                    v[a][m].x = 0;
                    v[a][m].y = 0;
                }
            }
        }
        wave_fence();
        auto exchange = [&]() {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
#pragma unroll
                for (int f = 0; f < PZ; ++f) cb[(f / FG) * CS + (f % FG) * QZ + zt] = v[a][f];
                wave_fence();
#pragma unroll
                for (int c = 0; c < PZ / QZ; ++c) {
#pragma unroll
                    for (int jj = 0; jj < QZ; ++jj) v[a][c * QZ + jj] = cb[rd[c] + jj];
                }
                wave_fence();
            }
        };
        rf_group_a<T, -1, LZ, true, 3>(v, twz);
        exchange();
        rf_group_b<T, -1, LZ, false, 3>(v, zt, twz);
        {
            // y_a = sum_b Ghat_ab x_b at (kx, ky, kz = zt + QZ c + PZ gg): the
            // stored octant and the parities (diagonal even, ab odd in a and b)
            const bool ux = kx > Mx / 2;
            const int fx = ux ? Mx - kx : kx;
            const C* gx = gp + (long long)fx * Hz * 6 * HY + fy;
            const bool f1 = ux != uy;
#pragma unroll
            for (int c = 0; c < PZ / QZ; ++c) {
#pragma unroll
                for (int gg = 0; gg < QZ; ++gg) {
                    const int kz = zt + QZ * c + PZ * gg;
                    const bool uz = kz > LZ / 2;
                    const int fz = uz ? LZ - kz : kz;
                    const C* Gp = gx + fz * 6 * HY;
                    C G6[6];
#pragma unroll
                    for (int k = 0; k < 6; ++k) G6[k] = Gp[k * HY];
                    const bool f2 = ux != uz, f4 = uy != uz;
                    G6[1].x = f1 ? -G6[1].x : G6[1].x;
                    G6[1].y = f1 ? -G6[1].y : G6[1].y;
                    G6[2].x = f2 ? -G6[2].x : G6[2].x;
                    G6[2].y = f2 ? -G6[2].y : G6[2].y;
                    G6[4].x = f4 ? -G6[4].x : G6[4].x;
                    G6[4].y = f4 ? -G6[4].y : G6[4].y;
                    const int sl = c * QZ + gg;
                    const C X = v[0][sl], Y = v[1][sl], Z = v[2][sl];
                    v[0][sl] = passes::trow(G6[0], G6[1], G6[2], X, Y, Z);
                    v[1][sl] = passes::trow(G6[1], G6[3], G6[4], X, Y, Z);
                    v[2][sl] = passes::trow(G6[2], G6[4], G6[5], X, Y, Z);
                }
            }
        }
        // back to subsequences: X[kappa_c + P g] = X[zt + Q m], m = c + (P / Q) g
        {
            C w[3][PZ];
#pragma unroll
            for (int a = 0; a < 3; ++a) {
#pragma unroll
                for (int c = 0; c < PZ / QZ; ++c) {
#pragma unroll
                    for (int gg = 0; gg < QZ; ++gg) w[a][c + (PZ / QZ) * gg] = v[a][c * QZ + gg];
                }
            }
#pragma unroll
            for (int a = 0; a < 3; ++a) {
#pragma unroll
                for (int m = 0; m < PZ; ++m) v[a][m] = w[a][m];
            }
        }
        rf_group_a<T, 1, LZ, false, 3>(v, twz);
        exchange();
        rf_group_b<T, 1, LZ, true, 3>(v, zt, twz);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
#pragma unroll
            for (int c = 0; c < PZ / QZ; ++c) {
#pragma unroll
                for (int gg = 0; gg < QZ / 2; ++gg) {
                    const int e = zt + QZ * c + PZ * gg;
                    if (e < nz) cb[a * CS + e] = v[a][c * QZ + gg];
                }
            }
        }
        wave_fence();
    }
    __syncthreads();

    // ---- y inverse, y < ny stored
    for (int l0 = wave * LPW; l0 < nlines; l0 += NW * LPW) {
        const int ln = l0 + lane % LPW;
        const int z = ln / 3, c3 = ln % 3;
        const bool live = ln < nlines;
        C* row = lds + c3 * CS + z;
        C v[1][PY];
#pragma unroll
        for (int m = 0; m < PY; ++m) {
            if (live) {
                v[0][m] = row[(yt + QY * m) * ZS];
            } else {
                v[0][m].x = 0;
                v[0][m].y = 0;
            }
        }
        wave_fence();
        rf_group_a<T, 1, LY, false, 1>(v, twy);
        if (live) {
#pragma unroll
            for (int f = 0; f < PY; ++f) row[(yt * PY + f) * ZS] = v[0][f];
        }
        wave_fence();
        if (live) {
#pragma unroll
            for (int c = 0; c < PY / QY; ++c) {
#pragma unroll
                for (int jj = 0; jj < QY; ++jj) v[0][c * QY + jj] = row[(jj * PY + yt + QY * c) * ZS];
            }
        }
        rf_group_b<T, 1, LY, true, 1>(v, yt, twy);
        C* dst = gq + (long long)z * LY * ys + c3;
        if (live) {
#pragma unroll
            for (int c = 0; c < PY / QY; ++c) {
#pragma unroll
                for (int gg = 0; gg < QY / 2; ++gg) {
                    const int e = yt + QY * c + PY * gg;
                    if (e < ny) dst[(long long)e * ys] = v[0][c * QY + gg];
                }
            }
        }
    }
}

// ------------------------------------------------------------------ short lengths
// The same fusion for grids with y and z extents of at most 20, which have no
// compile-time kernels (targets of up to about ten sites across): the
// plane of one kx in LDS as y lines (z, c) and as z lines (ky, c), the
// runtime-planned transforms on each.  Bounded by latency, so the chain is
// kept short: a thread keeps its line through all the passes of an axis (one
// division), each pass reads one LDS buffer and writes the other (one
// barrier), the first and last pass of an axis read and write the grid or
// the other axis' order, and the tensor values are loaded at the start.
// 18^3 in FP64, us for two and for thirty-two right-hand sides: 9.8 and 20;
// through the general runtime transform, with copies between the axes, 15.9
// and 24; as three kernels 33 and 235.

constexpr int SHORT_MAX = 20;
// eight wavefronts: one butterfly, or two, of every pass for each thread
constexpr int SHORT_NT = 512;

// An axis' passes, at most three at these lengths, one word each: radix,
// product of the radices before, and that product's 10-bit reciprocal (exact
// quotients of values below SHORT_MAX).  Kernel arguments lie in host
// memory: few bytes, read at the start.
struct ShortPlan {
    int L, tw, nst;
    unsigned p0, p1, p2;
};
inline ShortPlan short_plan(const AxisPlan& ax) {
    ShortPlan p{};
    p.L = ax.L;
    p.tw = ax.tw;
    p.nst = ax.nst;   // (at least one: extents start at 2)
    if (p.nst > 3) throw std::invalid_argument("too many passes for a short axis");
    int ns = 1;
    for (int i = 0; i < p.nst; ++i) {
        const int r = ax.R[i];
        (i == 0 ? p.p0 : i == 1 ? p.p1 : p.p2) = (unsigned)(r | ns << 8 | (1024 + ns - 1) / ns << 16);
        ns *= r;
    }
    return p;
}
__device__ __forceinline__ unsigned short_word(const ShortPlan& p, int s) { return s == 0 ? p.p0 : s == 1 ? p.p1 : p.p2; }

// LDS values of one of the two buffers, and with the twiddles of both axes
constexpr int short_buffer(int LY, int LZ, int nz) {
    const int a = nz * (LY | 1), b = LY * (LZ | 1);
    return 3 * (a > b ? a : b);
}
constexpr size_t rt_values(int LY, int LZ, int nz) {
    return (size_t)2 * short_buffer(LY, LZ, nz) + ((LY + 1) & ~1) + ((LZ + 1) & ~1);
}

// One pass of one line (operations and order of fft_pass: bitwise the same):
// the line's elements lie ss apart at src, results go ds apart to dst;
// IN: only elements [e0, e1) are inputs, the others zero; OUT: only results
// e < e1 are stored.  Butterflies jb, jb + jn, ...
template <typename T, int RR, int DIR, bool IN, bool OUT>
__device__ __forceinline__ void short_pass(const typename V2<T>::t* src, int ss, typename V2<T>::t* dst, int ds,
                                           int e0, int e1, const typename V2<T>::t* tw, int L, unsigned w, int jb,
                                           int jn) {
    using C = typename V2<T>::t;
    const int Ns = w >> 8 & 255, inv = w >> 16;
    const int LR = L / RR;
    const int tstep = LR * inv >> 10;   // LR / Ns
    for (int j = jb; j < LR; j += jn) {
        C v[RR];
        const unsigned o = __umul24(j, ss);
#pragma unroll
        for (int r = 0; r < RR; ++r) {
            if (IN) {
                v[r].x = 0;
                v[r].y = 0;
                if (j + r * LR >= e0 && j + r * LR < e1) v[r] = src[o + r * LR * ss];
            } else {
                v[r] = src[o + r * LR * ss];
            }
        }
        const int k = j - __umul24(Ns, __umul24(j, inv) >> 10);
        if (Ns > 1) {
            const int kt = __umul24(k, tstep);
#pragma unroll
            for (int r = 1; r < RR; ++r) {
                C t = tw[r * kt];
                if (DIR > 0) t.y = -t.y;
                v[r] = cmul(v[r], t);
            }
        }
        Dft<RR, DIR, C>::run(v);
        const int b = (j - k) * RR + k;
        const unsigned d = __umul24(b, ds);
#pragma unroll
        for (int q = 0; q < RR; ++q)
            if (!OUT || b + q * Ns < e1) dst[d + q * Ns * ds] = v[q];
    }
}
template <typename T, int DIR, bool IN, bool OUT>
__device__ __forceinline__ void short_step(const typename V2<T>::t* src, int ss, typename V2<T>::t* dst, int ds,
                                           int e0, int e1, const typename V2<T>::t* tw, int L, unsigned w, int jb,
                                           int jn) {
    switch (w & 255) {
#define DDA_R(N) \
    case N: short_pass<T, N, DIR, IN, OUT>(src, ss, dst, ds, e0, e1, tw, L, w, jb, jn); break;
        DDA_R(8) DDA_R(5) DDA_R(4) DDA_R(3) DDA_R(2)
#undef DDA_R
    }
}

template <typename T>
__global__ __launch_bounds__(SHORT_NT) void k_plane_rt(Geo g, ShortPlan py, ShortPlan pz, typename V2<T>::t* grid,
                                                const double2* tw64, const typename V2<T>::t* ghat,
                                                const RhsState* st, int chk) {
    using C = typename V2<T>::t;
    extern __shared__ __align__(16) unsigned char smem[];
    const int kx = blockIdx.x, q = blockIdx.y;
    if (passes::skip_rhs(st + q, chk)) return;
    const int Mx = g.M[0], My = py.L, Mz = pz.L, ny = g.n[1], nz = g.n[2];
    const int Ly = My | 1, Lz = Mz | 1;
    C* twy = (C*)smem;
    C* twz = twy + ((My + 1) & ~1);
    C* buf = twz + ((Mz + 1) & ~1);
    const int other = short_buffer(My, Mz, nz);   // the second buffer's offset
    C* gq = grid + (long long)q * g.npts * 3 + (long long)kx * 3;
    const int ys = Mx * 3;
    const int tid = threadIdx.x;
    // this thread's y line (z, c) and z line (ky, c), and its butterflies
    const int nly = 3 * nz, nlz = 3 * My;
    const int jny = SHORT_NT / nly, jnz = SHORT_NT / nlz;
    const int ly = tid % nly, lz = tid % nlz;
    const int jby = tid / nly < jny ? tid / nly : My, jbz = tid / nlz < jnz ? tid / nlz : Mz;
    const int zy = ly / 3, cy = ly - 3 * zy, kz = lz / 3, cz = lz - 3 * kz;
    C* gl = gq + (long long)zy * My * ys + cy;

    // tensor values of this thread's point (ky, kz)
    static_assert(SHORT_NT >= SHORT_MAX * SHORT_MAX, "points of a plane");
    C G[6];
    const int p = min(tid, My * Mz - 1);
    const int h = (p * ((65536 + My - 1) / My)) >> 16, k = p - h * My;
    const bool ux = kx > Mx / 2, uy = k > My / 2, uz = h > Mz / 2;
    const C* Gp = ghat + (((long long)(uz ? Mz - h : h) * g.H[1] + (uy ? My - k : k)) * g.H[0] +
                          (ux ? Mx - kx : kx)) * 6;
#pragma unroll
    for (int c = 0; c < 6; ++c) G[c] = Gp[c];
    // diagonal components are even in every index, ab is odd in a and b
    if (ux != uy) { G[1].x = -G[1].x; G[1].y = -G[1].y; }
    if (ux != uz) { G[2].x = -G[2].x; G[2].y = -G[2].y; }
    if (uy != uz) { G[4].x = -G[4].x; G[4].y = -G[4].y; }
    for (int i = tid; i < My + Mz; i += SHORT_NT) {
        const double2 w = tw64[i < My ? py.tw + i : pz.tw + i - My];
        C* d = i < My ? twy + i : twz + i - My;
        d->x = (T)w.x;
        d->y = (T)w.y;
    }

    int at = 0;   // offset of the buffer that holds the data
    for (int s = 0; s < py.nst; ++s) {
        const unsigned w = short_word(py, s);
        C* o = buf + (other - at);
        const bool last = s == py.nst - 1;   // ... into z lines
        C* dst = last ? o + cy * Lz + zy : o + ly * Ly;
        const int ds = last ? 3 * Lz : 1;
        if (s == 0) {
            const int e1 = zy >= g.i0[2] && zy < g.i1[2] ? g.i1[1] : 0;
            short_step<T, -1, true, false>(gl, ys, dst, ds, g.i0[1], e1, twy, My, w, jby, jny);
        } else {
            short_step<T, -1, false, false>(buf + at + ly * Ly, 1, dst, ds, 0, 0, twy, My, w, jby, jny);
        }
        at = other - at;
        __syncthreads();
    }
    for (int s = 0; s < pz.nst; ++s) {
        const unsigned w = short_word(pz, s);
        const C* src = buf + at + lz * Lz;
        C* dst = buf + (other - at) + lz * Lz;
        if (s == 0) short_step<T, -1, true, false>(src, 1, dst, 1, 0, nz, twz, Mz, w, jbz, jnz);
        else short_step<T, -1, false, false>(src, 1, dst, 1, 0, 0, twz, Mz, w, jbz, jnz);
        at = other - at;
        __syncthreads();
    }
    if (tid < My * Mz) {
        C* b = buf + at + k * 3 * Lz + h;
        const C X = b[0], Y = b[Lz], Z = b[2 * Lz];
        b[0] = passes::trow(G[0], G[1], G[2], X, Y, Z);
        b[Lz] = passes::trow(G[1], G[3], G[4], X, Y, Z);
        b[2 * Lz] = passes::trow(G[2], G[4], G[5], X, Y, Z);
    }
    __syncthreads();
    for (int s = 0; s < pz.nst; ++s) {
        const unsigned w = short_word(pz, s);
        const C* src = buf + at + lz * Lz;
        C* o = buf + (other - at);
        if (s == pz.nst - 1)   // ... z < nz into y lines
            short_step<T, 1, false, true>(src, 1, o + cz * Ly + kz, 3 * Ly, 0, nz, twz, Mz, w, jbz, jnz);
        else
            short_step<T, 1, false, false>(src, 1, o + lz * Lz, 1, 0, 0, twz, Mz, w, jbz, jnz);
        at = other - at;
        __syncthreads();
    }
    for (int s = 0; s < py.nst; ++s) {
        const unsigned w = short_word(py, s);
        const C* src = buf + at + ly * Ly;
        if (s == py.nst - 1) {   // ... y < ny into the grid
            short_step<T, 1, false, true>(src, 1, gl, ys, 0, ny, twy, My, w, jby, jny);
            break;
        }
        short_step<T, 1, false, false>(src, 1, buf + (other - at) + ly * Ly, 1, 0, 0, twy, My, w, jby, jny);
        at = other - at;
        __syncthreads();
    }
}

// ------------------------------------------------------------------ launcher

template <typename T, int LY, int LZ, int NW>
void plane_launch_waves(int chk, const Geo& g, int nrhs, typename V2<T>::t* grid, const double2* tw,
                        const typename V2<T>::t* gp, const RhsState* st, hipStream_t s) {
    const int ZS = z_stride(LZ, g.n[2]), CS = c_stride(LY, ZS, sizeof(T) == 4);
    DDA_LAUNCH((k_plane<T, LY, LZ, 64 * NW, plane_occ<T>(LZ, NW)>), dim3(plane_grid(g.M[0], nrhs)), dim3(64 * NW),
               plane_bytes(LY, LZ, g.n[2], sizeof(T) == 4), s, g, grid, tw, gp, st, chk, nrhs, ZS, CS);
}

template <typename T, int LY, int LZ>
bool plane_launch(int chk, const Geo& g, int nrhs, typename V2<T>::t* grid, const double2* tw,
                  const typename V2<T>::t* gp, const RhsState* st, hipStream_t s) {
    if constexpr (plane_pair<T>(LY, LZ)) {
        if ((long long)g.M[0] * nrhs > PLANE_ALONE)
            plane_launch_waves<T, LY, LZ, plane_waves<T>(LY, LZ, true)>(chk, g, nrhs, grid, tw, gp, st, s);
        else
            plane_launch_waves<T, LY, LZ, plane_waves<T>(LY, LZ, false)>(chk, g, nrhs, grid, tw, gp, st, s);
        return true;
    }
    return false;
}

template <typename T, int LY>
bool plane_launch_z(int chk, const Geo& g, int nrhs, typename V2<T>::t* grid, const double2* tw,
                    const typename V2<T>::t* gp, const RhsState* st, hipStream_t s) {
    switch (g.M[2]) {
#define DDA_Z(L) \
    case L: return plane_launch<T, LY, L>(chk, g, nrhs, grid, tw, gp, st, s);
        DDA_Z(32) DDA_Z(48) DDA_Z(64) DDA_Z(80) DDA_Z(96) DDA_Z(128)
#undef DDA_Z
        default: return false;
    }
}

}  // namespace plane

// The short-length kernel takes grids of one target with at most 20 points
// along y and z, the lengths below the shortest compile-time one.  Measured,
// us for passes 2-4 here and as three kernels: 18 x 18, two right-hand sides
// 9.8 and 33, thirty-two 20 and 235; but 20 x 48, whose z pass has a
// compile-time kernel, 28 (this kernel's first form) and 19.
template <typename T> bool plane_short(const Geo& g) {
    return !g.rg && g.M[1] <= plane::SHORT_MAX && g.M[2] <= plane::SHORT_MAX &&
           plane::rt_values(g.M[1], g.M[2], g.n[2]) * sizeof(typename V2<T>::t) <= plane::PLANE_LDS;
}

template <typename T>
void launch_plane(int chk, const Geo& g, int nrhs, typename V2<T>::t* grid, const double2* tw,
                  const typename V2<T>::t* gp, const RhsState* st, hipStream_t s) {
    bool done = false;
    if (plane_short<T>(g)) {
        hipStream_t stream = s;
        DDA_LAUNCH((plane::k_plane_rt<T>), dim3(g.M[0], nrhs), dim3(plane::SHORT_NT),
                   plane::rt_values(g.M[1], g.M[2], g.n[2]) * sizeof(typename V2<T>::t), stream, g,
                   plane::short_plan(g.ax[1]), plane::short_plan(g.ax[2]), grid, tw, gp, st, chk);
        return;
    }
    switch (g.M[1]) {
#define DDA_Y(L) \
    case L: done = plane::plane_launch_z<T, L>(chk, g, nrhs, grid, tw, gp, st, s); break;
        DDA_Y(32) DDA_Y(48) DDA_Y(64) DDA_Y(80) DDA_Y(96) DDA_Y(128)
#undef DDA_Y
        default: break;
    }
    if (!done) throw std::invalid_argument("no plane kernel for this grid");
}

// Whether launch_plane can take this grid: a compiled pair of lengths whose
// plane, with the largest z extent such a grid holds, fits the LDS.
template <typename T> bool plane_fits(const Geo& g) {
    return plane_short<T>(g) ||
           (plane::plane_pair<T>(g.M[1], g.M[2]) && 2 * g.n[1] <= g.M[1] && 2 * g.n[2] <= g.M[2]);
}
// Whether it does: a launch within the grid limit, and enough workgroups.
template <typename T> PlaneUse plane_use(const Geo& g, int nrhs) {
    if (!plane_fits<T>(g)) return PLANE_NO;
    if (plane_short<T>(g)) return nrhs <= 65535 ? PLANE_YES : PLANE_NO;
    if ((long long)(g.M[0] + passes::N_XCD) * nrhs * 768 >= (1LL << 32)) return PLANE_NO;
    return (long long)g.M[0] * nrhs <= plane::PLANE_MIN && plane::plane_long<T>(g.M[1], g.M[2]) ? PLANE_FEW : PLANE_YES;
}

#define DDA_INSTANTIATE_PLANE(T)                                                                                \
    template void launch_plane<T>(int, const Geo&, int, V2<T>::t*, const double2*, const V2<T>::t*,              \
                                  const RhsState*, hipStream_t);                                                \
    template bool plane_fits<T>(const Geo&);                                                                    \
    template PlaneUse plane_use<T>(const Geo&, int);                                                            \
    template bool plane_short<T>(const Geo&);

}  // namespace dda
