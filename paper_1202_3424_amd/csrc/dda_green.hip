// The interaction tensor and its FFT octant (FP64, rounded to FP32 for the
// FP32-matvec mode).
//
// The tensor is sampled on separations -(n-1) .. n-1 of each axis (padded
// index m or m - M) and is even or odd in each of them: the diagonal
// components are even, ab is odd in a and in b, exactly (a mirrored sample
// differs by signs only, and rounding is symmetric).  Only the octant
// 0 .. M/2 of its FFT is kept.  So each axis transforms only lines at
// non-negative separations of the axes not yet transformed, takes the
// mirrored half of its line with the component's parity, and stores only
// frequencies 0 .. M/2 -- an eighth of the padded grid per array, instead of
// the whole grid read and written by every axis.  The arithmetic of each
// stored value is that of the full transform.
//
// 192^3 (n = 96): 178 us (57 + 59 + 62 for x, y and z), 1430 us as
// whole-grid passes with a kernel each for the samples and the octant; each
// of the three now moves about 87 MB in and out at 2.9 TB/s and is bounded by
// its LDS passes.
#include <stdexcept>

#include "dda_kernels.h"

namespace dda {

namespace {

__host__ __device__ inline int pad_len(int L) { return L | 1; }

// Off-diagonal interaction tensor (Draine 1988) at separation (dx, dy, dz):
// A_jl = exp(ikr)/r [k^2 (nn - I) + (ikr - 1)/r^2 (3nn - I)], its six
// distinct components xx, xy, xz, yy, yz, zz; zero at R = 0.
__device__ __forceinline__ void green_sample(int dx, int dy, int dz, double kd, double2 (&out)[6]) {
    if (dx == 0 && dy == 0 && dz == 0) {
        for (int c = 0; c < 6; ++c) out[c] = double2{0.0, 0.0};
        return;
    }
    const double X = dx, Y = dy, Z = dz;
    const double r2 = X * X + Y * Y + Z * Z;
    const double r = sqrt(r2);
    double sn, cs;
    sincos(kd * r, &sn, &cs);
    const double2 pref = {cs / r, sn / r};                       // exp(ikr)/r
    const double2 ikr1 = {-1.0 / r2, kd * r / r2};               // (ikr - 1)/r^2
    // A = pref [ (-k^2 - (ikr-1)/r^2) I + (k^2 + 3(ikr-1)/r^2) R R / r^2 ]
    const double2 ciso = cmul(pref, double2{-kd * kd - ikr1.x, -ikr1.y});
    const double2 cnn = cscale(cmul(pref, double2{kd * kd + 3.0 * ikr1.x, 3.0 * ikr1.y}), 1.0 / r2);
    const double R[3] = {X, Y, Z};
    const int ab[6][2] = {{0, 0}, {0, 1}, {0, 2}, {1, 1}, {1, 2}, {2, 2}};
#pragma unroll
    for (int c = 0; c < 6; ++c) {
        double2 v = cscale(cnn, R[ab[c][0]] * R[ab[c][1]]);
        if (ab[c][0] == ab[c][1]) v = cadd(v, ciso);
        out[c] = v;
    }
}

// x: the lines y < ny, z < nz sampled and transformed, out [nz][ny][Hx][6].
// XL lines per workgroup, three components at a time in LDS (the other three
// wait in registers, so that each point is sampled once); at most
// XL Mx / NT <= MAXP points per thread.  (Sampling only x >= 0 and mirroring
// the rest into LDS took longer, 75 us against 63: the transform, not the
// sampling, is the time.)
template <int MAXP>
__global__ __launch_bounds__(NT) void k_green_x(Geo g, double kd, double2* out, const double2* tw64, int XL) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int Mx = g.M[0], Hx = g.H[0], nx = g.n[0], ny = g.n[1];
    const int z = blockIdx.y;
    const int y0 = blockIdx.x * XL;
    const int nl = min(XL, ny - y0);
    const int Lp = pad_len(Mx);
    double2* tws = (double2*)smem;
    double2* lds = tws + ((Mx + 1) & ~1);
    load_twiddles<double>(tws, tw64, g.ax[0]);
    const Divisor dm(Mx), dh(Hx);
    double2 hold[MAXP][3];
#pragma unroll
    for (int i = 0; i < MAXP; ++i) {
        const int p = threadIdx.x + i * NT;
        if (p < nl * Mx) {
            const int yo = dm.quot(p), m = p - yo * Mx;
            double2 v[6];
            // the slots between +(n-1) and -(n-1) hold no separation
            const bool ok = m <= nx - 1 || m >= Mx - (nx - 1);
            if (ok) {
                green_sample(m <= nx - 1 ? m : m - Mx, y0 + yo, z, kd, v);
            } else {
                for (int c = 0; c < 6; ++c) v[c] = double2{0.0, 0.0};
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                lds[(yo * 3 + c) * Lp + m] = v[c];
                hold[i][c] = v[3 + c];
            }
        }
    }
    double2* o = out + ((long long)z * ny + y0) * Hx * 6;
    for (int half = 0; half < 2; ++half) {
        __syncthreads();
        fft_lines<double, -1>(lds, tws, 3 * nl, Lp, g.ax[0]);
        for (int idx = threadIdx.x; idx < nl * Hx * 3; idx += NT) {
            const int c = idx % 3;
            const int yo = dh.quot(idx / 3), e = idx / 3 - yo * Hx;
            o[((long long)yo * Hx + e) * 6 + 3 * half + c] = lds[(yo * 3 + c) * Lp + e];
        }
        if (half == 0) {
            __syncthreads();
#pragma unroll
            for (int i = 0; i < MAXP; ++i) {
                const int p = threadIdx.x + i * NT;
                if (p < nl * Mx) {
                    const int yo = dm.quot(p), m = p - yo * Mx;
#pragma unroll
                    for (int c = 0; c < 3; ++c) lds[(yo * 3 + c) * Lp + m] = hold[i][c];
                }
            }
        }
    }
}

// columns (of six components) per workgroup: about 3072 values of LDS
constexpr int green_cols(int L) {
    int p = 1;
    while (p * 2 * 6 * L <= 3072 && p < 16) p *= 2;
    return p;
}

// y (AXIS 1): in [nz][ny][Hx][6] -> out [nz][Hy][Hx][6], outer index z < nz.
// z (AXIS 2): in [nz][Hy][Hx][6] -> the octant [Hz][Hy][Hx][6] scaled by
// 1/M (so that the inverse transforms of the product need no further
// normalisation), FP64 and, where gh32 is given, FP32; outer index ky.
// LC: compile-time length, or 0 with TXrt columns per workgroup.
template <int AXIS, int LC>
__global__ __launch_bounds__(NT) void k_green_line(Geo g, const double2* in, double2* out, float2* gh32,
                                                  const double2* tw64, int TXrt) {
    constexpr bool CT = LC > 0;
    extern __shared__ __align__(16) unsigned char smem[];
    const AxisPlan& pl = g.ax[AXIS];
    const int L = CT ? LC : pl.L;
    const int TX = CT ? green_cols(CT ? LC : 1) : TXrt;
    const int Lp = pad_len(L);
    const int Hx = g.H[0], n = g.n[AXIS], H = g.H[AXIS];
    const int o = blockIdx.y;
    const int x0 = blockIdx.x * TX;
    const int nval = 6 * min(TX, Hx - x0), nlines = 6 * TX;
    double2* lds = (double2*)smem;
    double2* tws = nullptr;
    if constexpr (!CT) {
        tws = lds;
        lds = tws + ((L + 1) & ~1);
        load_twiddles<double>(tws, tw64, pl);
    }
    // strides of the line's element and of the outer index, in and out
    const long long row = (long long)Hx * 6;
    const long long se = AXIS == 1 ? row : g.H[1] * row;
    const double2* src = in + (AXIS == 1 ? (long long)o * n * row : (long long)o * row) + (long long)x0 * 6;
    const long long dst0 = (AXIS == 1 ? (long long)o * H * row : (long long)o * row) + (long long)x0 * 6;
    for (int idx = threadIdx.x; idx < nlines * L; idx += NT) {
        const int inner = idx % nlines;
        const int e = idx / nlines;
        double2 v = {0.0, 0.0};
        const bool lower = e < n, upper = e > L - n;
        if ((lower || upper) && inner < nval) {
            v = src[(lower ? e : L - e) * se + inner];
            // odd components: xy and yz in y, xz and yz in z
            const int c = inner % 6;
            if (!lower && (c == 4 || c == AXIS)) v = double2{-v.x, -v.y};
        }
        lds[inner * Lp + e] = v;
    }
    __syncthreads();
    if constexpr (CT) fft_lines_ct<double, -1, LC, 6 * green_cols(LC), NT>(lds, tw64 + pl.tw);
    else fft_lines<double, -1>(lds, tws, nlines, Lp, pl);
    const double sc = AXIS == 2 ? 1.0 / (double)g.npts : 1.0;
    for (int idx = threadIdx.x; idx < nlines * H; idx += NT) {
        const int inner = idx % nlines;
        const int e = idx / nlines;
        if (inner < nval) {
            const long long d = dst0 + e * se + inner;
            double2 v = lds[inner * Lp + e];
            if (AXIS == 2) {
                v = cscale(v, sc);
                if (gh32) gh32[d] = float2{(float)v.x, (float)v.y};
            }
            out[d] = v;
        }
    }
}

// The octant as [Hx][Hz][6][plane_row(My)] for the plane kernel, the padding
// of a row zero.
__global__ __launch_bounds__(NT) void k_green_plane(Geo g, const double2* gh64, double2* gp64, float2* gp32) {
    const int hyp = plane_row(g.M[1]);
    const long long i = (long long)blockIdx.x * NT + threadIdx.x;
    if (i >= (long long)g.H[0] * g.H[2] * 6 * hyp) return;
    const int hy = (int)(i % hyp);
    const int c = (int)(i / hyp % 6);
    const int hz = (int)(i / (6LL * hyp) % g.H[2]);
    const int hx = (int)(i / (6LL * hyp * g.H[2]));
    double2 v = {0.0, 0.0};
    if (hy < g.H[1]) v = gh64[(((long long)hz * g.H[1] + hy) * g.H[0] + hx) * 6 + c];
    if (gp64) gp64[i] = v;
    if (gp32) gp32[i] = float2{(float)v.x, (float)v.y};
}

template <int AXIS>
void green_line(const Geo& g, const double2* in, double2* out, float2* gh32, const double2* tw, int n_outer,
                hipStream_t s) {
    const int L = g.M[AXIS];
    auto smem = [](int l, int tx) { return ((size_t)((l + 1) & ~1) + (size_t)6 * tx * pad_len(l)) * sizeof(double2); };
    switch (L) {
#define DDA_G(LL)                                                                                              \
    case LL:                                                                                                   \
        hipLaunchKernelGGL((k_green_line<AXIS, LL>), dim3((g.H[0] + green_cols(LL) - 1) / green_cols(LL), n_outer), \
                           dim3(NT), smem(LL, green_cols(LL)), s, g, in, out, gh32, tw, 0);                    \
        return;
        DDA_G(32) DDA_G(48) DDA_G(64) DDA_G(80) DDA_G(96) DDA_G(128) DDA_G(160) DDA_G(192) DDA_G(256) DDA_G(384)
        DDA_G(512)
#undef DDA_G
        default: {
            // the runtime-planned transform takes at most Tile::EMAX values
            int TX = Tile<double>::EMAX / (6 * L);
            if (TX < 1) throw std::invalid_argument("tensor line above the LDS tile");
            if (TX > 16) TX = 16;
            hipLaunchKernelGGL((k_green_line<AXIS, 0>), dim3((g.H[0] + TX - 1) / TX, n_outer), dim3(NT), smem(L, TX),
                               s, g, in, out, gh32, tw, TX);
        }
    }
}

}  // namespace

size_t green_work_values(const Geo& g) {
    return (size_t)g.n[2] * g.H[0] * 6 * ((size_t)g.n[1] + g.H[1]);
}

void launch_green(const Geo& g, double kd, double2* work, double2* gh64, float2* gh32, const double2* tw,
                  hipStream_t s) {
    double2* A = work;
    double2* B = work + (size_t)g.n[2] * g.n[1] * g.H[0] * 6;
    constexpr int MAXP = (Tile<double>::EMAX / 3 + NT - 1) / NT;
    int XL = Tile<double>::EMAX / (3 * g.M[0]);
    if (XL < 1) throw std::invalid_argument("x extent above the LDS line tile");
    if (XL > g.n[1]) XL = g.n[1];
    const size_t sm = ((size_t)((g.M[0] + 1) & ~1) + (size_t)3 * XL * pad_len(g.M[0])) * sizeof(double2);
    hipLaunchKernelGGL(k_green_x<MAXP>, dim3((g.n[1] + XL - 1) / XL, g.n[2]), dim3(NT), sm, s, g, kd, A, tw, XL);
    green_line<1>(g, A, B, nullptr, tw, g.n[2], s);
    green_line<2>(g, B, gh64, gh32, tw, g.H[1], s);
}

void launch_green_plane(const Geo& g, const double2* gh64, double2* gp64, float2* gp32, hipStream_t s) {
    const long long n = (long long)plane_values(g);
    hipLaunchKernelGGL(k_green_plane, dim3((unsigned)((n + NT - 1) / NT)), dim3(NT), 0, s, g, gh64, gp64, gp32);
}

}  // namespace dda
