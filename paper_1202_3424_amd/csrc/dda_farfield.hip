// The far field: scattering amplitudes and cross sections over direction
// sets, and the direction sets of the angular averages.
#include "dda_kernels.h"

namespace dda {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------ far field
// Scattering amplitudes ("Scattering by Finite Targets: The Mueller Matrix";
// Draine 1988): per direction n and right-hand side, A = k^3 sum_j P_j
// exp(-i k n . r_j), then f_1 = theta . A, f_2 = phi . A and the differential
// cross section (|f_1|^2 + |f_2|^2) / k^2.  dirs holds n, theta, phi per
// direction.  On the lattice the phase factor separates by axis,
// exp(-i k n . r) = w_x(x) w_y(y) w_z(z), so one workgroup per direction
// tabulates the n_x + n_y + n_z factors of its direction in LDS and every
// term costs two complex products instead of a sine and cosine; the
// right-hand sides are taken FR at a time over the same factors, and DW
// directions at a time over the same loaded sites (each site's P is read
// once for all DW).  per > 0: direction d belongs to right-hand side d / per
// alone (every right-hand side with its own direction set in one launch;
// DW divides per) and its results go to entry d; there FR is 1.  Each term
// is accumulated as four fused multiply-adds in a fixed order.
// Deterministic sums (each direction: fixed per-thread order, then the
// workgroup reduction; the same for every DW and FR).
template <int DW, int FR>
__global__ __launch_bounds__(NT) void k_farfield(int nsites, const int* coords, const double2* P, long long n3,
                                                 int nrhs, const double* dirs, double k, int lox, int loy, int loz,
                                                 int nx, int ny, int nz, double2* f, double* dcs, int ndir,
                                                 int per) {
    extern __shared__ double2 wtab[];     // [DW][nx + ny + nz] phase factors of the group's directions
    __shared__ double sh[6 * FR * NT / 64];   // block_sum scratch: one value per wave and sum
    const int d0 = blockIdx.x * DW;
    const int nt = nx + ny + nz;
    for (int i = threadIdx.x; i < DW * nt; i += NT) {
        const int j = i / nt, ii = i % nt;
        const int d = min(d0 + j, ndir - 1);   // past the end: a copy of the last direction, not stored
        const double* dv = dirs + (long long)d * 9;
        const int a = ii < nx ? 0 : (ii < nx + ny ? 1 : 2);
        const int c = a == 0 ? lox + ii : (a == 1 ? loy + (ii - nx) : loz + (ii - nx - ny));
        double sn, cs;
        sincos(-k * dv[a] * c, &sn, &cs);
        wtab[i] = double2{cs, sn};
    }
    __syncthreads();
    const double k3 = k * k * k;
    // per = 0: the right-hand sides FR at a time along the grid's y
    const int qa = per > 0 ? d0 / per : (int)blockIdx.y * FR;
    const int qb = per > 0 ? qa + 1 : min(nrhs, qa + FR);
    for (int q0 = qa; q0 < qb; q0 += FR) {
        double acc[DW][6 * FR];
#pragma unroll
        for (int j = 0; j < DW; ++j)
#pragma unroll
            for (int i = 0; i < 6 * FR; ++i) acc[j][i] = 0.0;
        // a thread's sites s, s + NT, s + 2 NT, ... in that order, two per
        // iteration with both sites' loads issued first
        for (int s0 = threadIdx.x; s0 < nsites; s0 += 2 * NT) {
            int cc[2][3];
            double2 pv[2][FR][3];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int s = min(s0 + h * NT, nsites - 1);   // past the end: loaded, not added
                cc[h][0] = coords[s * 3 + 0] - lox;
                cc[h][1] = nx + coords[s * 3 + 1] - loy;
                cc[h][2] = nx + ny + coords[s * 3 + 2] - loz;
#pragma unroll
                for (int r = 0; r < FR; ++r) {
                    const double2* Pq = P + (long long)(q0 + r) * n3 + (long long)s * 3;
#pragma unroll
                    for (int c = 0; c < 3; ++c) pv[h][r][c] = q0 + r < qb ? Pq[c] : double2{0.0, 0.0};
                }
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (h == 1 && s0 + NT >= nsites) break;
#pragma unroll
                for (int j = 0; j < DW; ++j) {
                    const double2* wt = wtab + j * nt;
                    const double2 w = cmul(cmul(wt[cc[h][0]], wt[cc[h][1]]), wt[cc[h][2]]);
#pragma unroll
                    for (int r = 0; r < FR; ++r) {
#pragma unroll
                        for (int c = 0; c < 3; ++c) {
                            double& ar = acc[j][6 * r + 2 * c];
                            double& ai = acc[j][6 * r + 2 * c + 1];
                            ar = fma(pv[h][r][c].x, w.x, ar);
                            ar = fma(-pv[h][r][c].y, w.y, ar);
                            ai = fma(pv[h][r][c].x, w.y, ai);
                            ai = fma(pv[h][r][c].y, w.x, ai);
                        }
                    }
                }
            }
        }
#pragma unroll
        for (int j = 0; j < DW; ++j) {
            block_sum<6 * FR>(acc[j], sh);
            const int d = d0 + j;
            if (threadIdx.x == 0 && d < ndir) {
                const double* dv = dirs + (long long)d * 9;
                for (int r = 0; r < FR && q0 + r < qb; ++r) {
                    double2 f1 = {0.0, 0.0}, f2 = {0.0, 0.0};
                    for (int c = 0; c < 3; ++c) {
                        const double2 A = {k3 * acc[j][6 * r + 2 * c], k3 * acc[j][6 * r + 2 * c + 1]};
                        f1 = cadd(f1, double2{dv[3 + c] * A.x, dv[3 + c] * A.y});
                        f2 = cadd(f2, double2{dv[6 + c] * A.x, dv[6 + c] * A.y});
                    }
                    const long long o = per > 0 ? (long long)d : (long long)(q0 + r) * ndir + d;
                    f[o * 2 + 0] = f1;
                    f[o * 2 + 1] = f2;
                    dcs[o] = (f1.x * f1.x + f1.y * f1.y + f2.x * f2.x + f2.y * f2.y) / (k * k);
                }
            }
            __syncthreads();
        }
    }
}

// Direction sets of the angular averages ("Averaging over Scattering
// Directions"): for right-hand side q with incidence direction k, the frame
// (k, u, v), u the unit vector along k x e (e the x axis, or y where k is
// near x) and v = k x u, and the directions n = mu_i k + sqrt(1 - mu_i^2)
// (cos p_j u + sin p_j v), p_j = 2 pi j / n_phi, with their theta and phi
// unit vectors: dirs [ng][n_theta][n_phi][9] (n, theta, phi).
__global__ __launch_bounds__(NT) void k_avg_dirs(int ng, const double* kh, const double* mu, int n_theta, int n_phi,
                                                 double* dirs) {
    const long long nd = (long long)n_theta * n_phi;
    const long long idx = (long long)blockIdx.x * NT + threadIdx.x;
    if (idx >= (long long)ng * nd) return;
    const int q = (int)(idx / nd);
    const int i = (int)((idx % nd) / n_phi);
    const int j = (int)(idx % n_phi);
    const double* k = kh + 3 * q;
    const bool nx = fabs(k[0]) < 0.9;
    const double e[3] = {nx ? 1.0 : 0.0, nx ? 0.0 : 1.0, 0.0};
    double u[3] = {k[1] * e[2] - k[2] * e[1], k[2] * e[0] - k[0] * e[2], k[0] * e[1] - k[1] * e[0]};
    const double un = sqrt(u[0] * u[0] + u[1] * u[1] + u[2] * u[2]);
    for (double& x : u) x /= un;
    const double v[3] = {k[1] * u[2] - k[2] * u[1], k[2] * u[0] - k[0] * u[2], k[0] * u[1] - k[1] * u[0]};
    const double ct = mu[i], st = sqrt(fmax(0.0, 1.0 - ct * ct));
    const double p = 2.0 * M_PI * j / n_phi;
    double sp, cp;
    sincos(p, &sp, &cp);
    double* D = dirs + idx * 9;
    for (int m = 0; m < 3; ++m) {
        const double t = cp * u[m] + sp * v[m];
        D[m] = ct * k[m] + st * t;
        D[3 + m] = ct * t - st * k[m];
        D[6 + m] = -sp * u[m] + cp * v[m];
    }
}

// ------------------------------------------------------------------ dense boxes
// The same amplitudes by a contraction along x.  With x = xc + h about the
// box centre, a line (y, z) of sites gives
//   sum_x P(x) exp(-i t x) = exp(-i t xc) sum_{h >= 0} [cos(t h) E_h - i sin(t h) O_h],
// E_h = P(+h) + P(-h), O_h = P(+h) - P(-h), t = k n_x: two real products per
// component and pair of sites instead of a complex phase product and a
// complex multiply-add each, and a real matrix product (directions x h) (h x
// lines) for the FP64 matrix instructions.  The factors of y and z then
// multiply the line sums.  Bounded by the FP64 matrix rate: 6 multiply-adds
// per direction, right-hand side and point of the box (rounded up to 8 in x
// and 16 in y, a tile of 16 lines only as far from the centre as it has
// sites), 71 us of matrix instructions for the 51,488-site ellipsoid and 2 x
// 3,072 directions: 129 us and 14 for its two small kernels, 353 by the sum
// over sites.

constexpr int FF_LINES = 16;   // lines (along y) of a tile
constexpr int FF_DIRS = 16;    // directions of a wavefront
// planes of a workgroup: a constant, so that a sum's order depends on neither
// the directions nor the right-hand sides of the call
constexpr int FF_Z = 2;
// wavefronts of three components up to which a launch takes one component a
// wavefront instead
constexpr int FF_SPLIT = 1024;

// Phase factors of a tile of 16 directions: tab[q][tile] holds, in the order
// the lanes of k_ff_lines read them, (cos, sin)(t h) of lane (direction
// lane & 15, h = 4 ks + (lane >> 4)) as [KS][64], then exp(-i k n_y y) as
// [ny][16] and exp(-i k n_z z) as [nz][16].  Directions past the end copy the
// last one.  i: value of this thread; dirs, tab: of this right-hand side.
__device__ __forceinline__ void ff_factor(int i, int tile, int nx, int ny, int nz, int KS, const double* dirs, int nd,
                                          double k, int loy, int loz, double2* tab) {
    const int n = KS * 64 + (ny + nz) * FF_DIRS;
    if (i >= n) return;
    const int j = i - KS * 64;
    const double* dv = dirs + (long long)min(tile * FF_DIRS + (i & 15), nd - 1) * 9;
    double ph;
    if (j < 0) ph = k * dv[0] * (4 * (i >> 6) + ((i & 63) >> 4) + (nx & 1 ? 0.0 : 0.5));
    else if (j < ny * FF_DIRS) ph = -k * dv[1] * (loy + j / FF_DIRS);
    else ph = -k * dv[2] * (loz + j / FF_DIRS - ny);
    double2 w;
    sincos(ph, &w.y, &w.x);
    tab[(long long)tile * n + i] = w;
}

// The operands of k_ff_lines for right-hand side blockIdx.y: the first nfold
// workgroups fold P, the others form the phase factors (one launch: each part
// alone is mostly launch and load latency).
//
// The folded operands of every tile (16 lines of one z, one component), in
// the order in which a wavefront's lanes read them: value [q][tile][c][ks][p]
// of lane (k, l) is h = 4 ks + k of line y = 16 yb + l, {Re E, Im O} (p = 0)
// or {Im E, -Re O} (p = 1).  A workgroup forms four steps ks of one component
// of a tile; kt[tile][ks / 4]: steps of the tile up to its last one there with
// a site.
__global__ __launch_bounds__(NT) void k_ff_operands(const int* map, const int* perm, const double2* P, long long n3,
                                                    int nx, int ny, int nz, int KS, double2* fold, int* kt,
                                                    int nfold, const double* dirs, int nd, int dstride, double k,
                                                    int loy, int loz, double2* tab) {
    if ((int)blockIdx.x >= nfold) {
        const int per = (KS * 64 + (ny + nz) * FF_DIRS + NT - 1) / NT;   // workgroups of a tile of directions
        const int b = blockIdx.x - nfold, q = blockIdx.y;
        const int tiles = (nd + FF_DIRS - 1) / FF_DIRS;
        ff_factor(b % per * NT + threadIdx.x, b / per, nx, ny, nz, KS, dirs + (long long)q * dstride * 9, nd, k, loy,
                  loz, tab + (long long)q * tiles * (KS * 64 + (ny + nz) * FF_DIRS));
        return;
    }
    __shared__ int most;
    const int nyb = (ny + FF_LINES - 1) / FF_LINES, nkg = (KS + 3) / 4;
    const int tile = blockIdx.x / (3 * nkg), kg = blockIdx.x % nkg, q = blockIdx.y, c = blockIdx.x / nkg % 3;
    const int z = tile / nyb, yb = tile % nyb;
    const double2* Pq = P + (long long)q * n3;
    double2* out = fold + ((long long)q * nz * nyb + tile) * 3 * KS * 2 * 64;
    if (threadIdx.x == 0) most = 0;
    __syncthreads();
    const int half = nx / 2, odd = nx & 1;
    const int lane = threadIdx.x & 63, ks = kg * 4 + (threadIdx.x >> 6);
    if (ks < KS) {
        const int h = 4 * ks + (lane >> 4), y = yb * FF_LINES + (lane & 15);
        const int xp = half + h, xm = half - 1 + odd - h;
        int sp = -1, sm = -1;
        if (y < ny) {
            const int* row = map + ((long long)z * ny + y) * nx;
            if (xp < nx) sp = row[xp];
            if (xm >= 0 && xm != xp) sm = row[xm];
        }
        if (sp >= 0 || sm >= 0) atomicMax(&most, ks + 1);
        const long long ip = sp >= 0 ? 3LL * perm[sp] : 0, im = sm >= 0 ? 3LL * perm[sm] : 0;
        const double2 zero = {0.0, 0.0};
        const double2 a = sp >= 0 ? Pq[ip + c] : zero, b = sm >= 0 ? Pq[im + c] : zero;
        const double2 E = cadd(a, b);
        // the centre of an odd line is its own mirror point: O = 0
        const double2 O = xm == xp ? zero : csub(a, b);
        double2* o = out + ((long long)(c * KS + ks) * 2) * 64 + lane;
        o[0] = double2{E.x, O.y};
        o[64] = double2{E.y, -O.x};
    }
    __syncthreads();
    if (q == 0 && c == 0 && threadIdx.x == 0) kt[tile * nkg + kg] = most;
}

// Sums over the planes z of chunk blockIdx.y for 16 directions per
// wavefront: part[q][chunk][d][6] (Re, Im of the three components).  dirs
// [nd][9], per right-hand side dstride directions further on.  The matrix
// instruction (16 x 16 x 4) takes A[direction lane & 15][k = lane >> 4] and
// B[k][line lane & 15] and gives rows (lane >> 4) + 4 v of column lane & 15.
// Wavefronts share nothing: each keeps its factors of x in its own LDS.  NC:
// the components a wavefront takes, all three or one (blockIdx.y then counts
// the components of each chunk); their sums are separate, so the results are
// the same.
template <int NC>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(3))) void k_ff_lines(const double2* fold, const int* kt, int nx, int ny, int nz, int KS,
                                                const double2* tab, int nd, double* part) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int d0 = (blockIdx.x * (NT / 64) + wave) * FF_DIRS;
    if (d0 >= nd) return;
    double2* cst = (double2*)smem + (size_t)wave * KS * 64;   // [KS][lane] (cos, sin) of t h
    const int q = blockIdx.z;
    const int chunk = NC == 3 ? blockIdx.y : blockIdx.y / 3, c0 = NC == 3 ? 0 : blockIdx.y % 3;
    const int nchunk = NC == 3 ? gridDim.y : gridDim.y / 3;
    const int z0 = chunk * FF_Z, z1 = min(nz, z0 + FF_Z);
    const int nyb = (ny + FF_LINES - 1) / FF_LINES;
    tab += ((long long)q * ((nd + FF_DIRS - 1) / FF_DIRS) + d0 / FF_DIRS) * (KS * 64 + (ny + nz) * FF_DIRS);
    for (int ks = 0; ks < KS; ++ks) cst[ks * 64 + lane] = tab[ks * 64 + lane];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    // this lane's four directions (rows) and line (column)
    const int row = lane >> 4, col = lane & 15;
    const double2* fy = tab + KS * 64 + row;
    const double2* fz = fy + ny * FF_DIRS;
    double2 tot[4][NC];
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int c = 0; c < NC; ++c) tot[v][c] = double2{0.0, 0.0};
    const int nkg = (KS + 3) / 4, nzc = z1 - z0, nt = nyb * nzc;
    // tile i of this wavefront: line block i / nzc of plane z0 + i % nzc
    auto tile_of = [&](int i) { return (z0 + i % nzc) * nyb + i / nzc; };
    const double2* base = fold + ((long long)q * nz * nyb * 3 + c0) * KS * 2 * 64 + lane;
    const long long tstride = 3LL * KS * 2 * 64;
    double2 b0 = base[tile_of(0) * tstride], b1 = base[tile_of(0) * tstride + 64];
    for (int i = 0; i < nt; ++i) {
        const int tile = tile_of(i);
        int n = 1;   // (an empty tile takes one step of zeros)
        for (int j = 0; j < nkg; ++j) n = max(n, kt[tile * nkg + j]);
        n = __builtin_amdgcn_readfirstlane(n);
        double2 w[4];
#pragma unroll
        for (int v = 0; v < 4; ++v)
            w[v] = cmul(fz[(z0 + i % nzc) * FF_DIRS + 4 * v],
                        fy[min(i / nzc * FF_LINES + col, ny - 1) * FF_DIRS + 4 * v]);
        // one component at a time: two accumulators are enough to keep the
        // matrix unit busy, and the registers they leave let three wavefronts
        // share a SIMD (all six at once, two wavefronts: 136 us against 129 for
        // the ellipsoid)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            const double2* B = base + tile * tstride + c * KS * 128;
            const double2* Bn = c < NC - 1 ? B + KS * 128 : base + tile_of(min(i + 1, nt - 1)) * tstride;
            d4 T0 = {0.0, 0.0, 0.0, 0.0}, T1 = {0.0, 0.0, 0.0, 0.0};
            for (int ks = 0; ks < n; ++ks) {
                const double2 a = cst[ks * 64 + lane];
                // the next step's operands (after the last, the next
                // component's or tile's first) are loaded before the products
                const double2* src = ks + 1 < n ? B + (ks + 1) * 128 : Bn;
                const double2 n0 = src[0], n1 = src[64];
                T0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b0.x, T0, 0, 0, 0);
                T1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a.x, b1.x, T1, 0, 0, 0);
                T0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b0.y, T0, 0, 0, 0);
                T1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a.y, b1.y, T1, 0, 0, 0);
                b0 = n0;
                b1 = n1;
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                tot[v][c].x = fma(-T1[v], w[v].y, fma(T0[v], w[v].x, tot[v][c].x));
                tot[v][c].y = fma(T1[v], w[v].x, fma(T0[v], w[v].y, tot[v][c].y));
            }
        }
    }
    // over the 16 lines
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int d = d0 + row + 4 * v;
        double* o = part + (((long long)q * nchunk + chunk) * nd + d) * 6 + 2 * c0;
#pragma unroll
        for (int c = 0; c < NC; ++c) {
#pragma unroll
            for (int off = 8; off > 0; off >>= 1) {
                tot[v][c].x += __shfl_xor(tot[v][c].x, off, 64);
                tot[v][c].y += __shfl_xor(tot[v][c].y, off, 64);
            }
            if (col == 0 && d < nd) {
                o[2 * c] = tot[v][c].x;
                o[2 * c + 1] = tot[v][c].y;
            }
        }
    }
}

// A = k^3 times the chunks' sums in order and the phase of the box centre in
// x, projected on theta and phi; f and dcs [q][ostride].
__global__ __launch_bounds__(NT) void k_ff_project(const double* part, int nchunk, const double* dirs, int nd,
                                                  int dstride, double k, double xc, int ostride, double2* f,
                                                  double* dcs) {
    const int d = blockIdx.x * NT + threadIdx.x, q = blockIdx.y;
    if (d >= nd) return;
    const double* dv = dirs + ((long long)q * dstride + d) * 9;
    double s[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
    for (int h = 0; h < nchunk; ++h) {   // (unrolled: the loads do not wait for one another)
        const double* p = part + (((long long)q * nchunk + h) * nd + d) * 6;
        for (int i = 0; i < 6; ++i) s[i] += p[i];
    }
    double2 w;
    sincos(-k * dv[0] * xc, &w.y, &w.x);
    w = cscale(w, k * k * k);
    double2 f1 = {0.0, 0.0}, f2 = {0.0, 0.0};
    for (int c = 0; c < 3; ++c) {
        const double2 A = cmul(double2{s[2 * c], s[2 * c + 1]}, w);
        f1 = cadd(f1, double2{dv[3 + c] * A.x, dv[3 + c] * A.y});
        f2 = cadd(f2, double2{dv[6 + c] * A.x, dv[6 + c] * A.y});
    }
    const long long o = (long long)q * ostride + d;
    f[o * 2 + 0] = f1;
    f[o * 2 + 1] = f2;
    dcs[o] = (f1.x * f1.x + f1.y * f1.y + f2.x * f2.x + f2.y * f2.y) / (k * k);
}

}  // namespace

// directions per workgroup of the far field: four where the direction sets
// allow it and the launch still has at least FF_MIN_WG workgroups (each
// site's P then serves four directions), else one
constexpr int FF_DW = 4;
constexpr int FF_MIN_WG = 512;
void launch_farfield(int nsites, const int* coords, const double2* P, int nrhs, const double* dirs, int ndir,
                     double k, const int lo[3], const int n[3], double2* f, double* dcs, hipStream_t s) {
    const size_t nt = (size_t)(n[0] + n[1] + n[2]);
    const int npair = (nrhs + 1) / 2;   // grid y: the right-hand sides two at a time
    if ((long long)((ndir + FF_DW - 1) / FF_DW) * npair >= FF_MIN_WG) {
        hipLaunchKernelGGL((k_farfield<FF_DW, 2>), dim3((ndir + FF_DW - 1) / FF_DW, npair), dim3(NT),
                           FF_DW * nt * sizeof(double2), s, nsites, coords, P, 3LL * nsites, nrhs, dirs, k, lo[0],
                           lo[1], lo[2], n[0], n[1], n[2], f, dcs, ndir, 0);
    } else {
        hipLaunchKernelGGL((k_farfield<1, 2>), dim3(ndir, npair), dim3(NT), nt * sizeof(double2), s, nsites, coords,
                           P, 3LL * nsites, nrhs, dirs, k, lo[0], lo[1], lo[2], n[0], n[1], n[2], f, dcs, ndir, 0);
    }
}
void launch_avg_dirs(int ng, const double* kh, const double* mu, int n_theta, int n_phi, double* dirs,
                     hipStream_t s) {
    const long long tot = (long long)ng * n_theta * n_phi;
    hipLaunchKernelGGL(k_avg_dirs, dim3((unsigned)((tot + NT - 1) / NT)), dim3(NT), 0, s, ng, kh, mu, n_theta, n_phi,
                       dirs);
}
void launch_farfield_sets(int nsites, const int* coords, const double2* P, int nrhs, const double* dirs, int per,
                          double k, const int lo[3], const int n[3], double2* f, double* dcs, hipStream_t s) {
    const size_t nt = (size_t)(n[0] + n[1] + n[2]);
    const int ndt = per * nrhs;
    if (per % FF_DW == 0 && ndt >= FF_DW * FF_MIN_WG) {
        hipLaunchKernelGGL((k_farfield<FF_DW, 1>), dim3(ndt / FF_DW), dim3(NT), FF_DW * nt * sizeof(double2), s, nsites,
                           coords, P, 3LL * nsites, nrhs, dirs, k, lo[0], lo[1], lo[2], n[0], n[1], n[2], f, dcs,
                           ndt, per);
    } else {
        hipLaunchKernelGGL((k_farfield<1, 1>), dim3(ndt), dim3(NT), nt * sizeof(double2), s, nsites, coords, P,
                           3LL * nsites, nrhs, dirs, k, lo[0], lo[1], lo[2], n[0], n[1], n[2], f, dcs, ndt, per);
    }
}

// Which form.  A list of directions (nset 0): of the target alone, so that a
// direction's sum does not depend on the others of the call; the sets of an
// average, of nset directions each: of that count too (never of the right-hand
// sides).  The line form's work grows with the rounded box, the sum's with the
// sites: for 48^3 boxes, 2 x 3,072 directions, 297 against 453 us a call at two
// points a site, 297 against 265 at four.  Below 8,192 sites it costs a few us
// of launches and latency that only many directions win back.  One right-hand
// side, us a call by lines and by the sum: 16^3, 74 directions 55 and 53, 3,072
// 89 and 109; 48 x 10 x 10 58 and 54, 89 and 111; 21^3 60 % full 60 and 56, 102
// and 118; 26^3 60 % full (10,514 sites) 61 and 60, 112 and 136.  Boxes of eight
// points along x or fewer, half empty when rounded: 8 x 8 x 128 62 and 57, 128
// and 125.
bool far_lines(int nsites, const int n[3], int nset) {
    const long long v = 8LL * ((n[0] + 7) / 8) * FF_LINES * ((n[1] + FF_LINES - 1) / FF_LINES) * n[2];
    if (nsites < 4096 || v > 3LL * nsites) return false;
    const bool half = v < 2LL * nsites;
    if (nsites >= 8192) return half || n[0] > 8;
    if (10 * v <= 11LL * nsites) return true;
    return half ? nset >= 1024 : n[0] > 8 && nset >= 2048;
}
namespace {
// Work memory is at most FF_WORK, by groups of directions and of right-hand
// sides, or what one right-hand side's folded operands (at most 3 times its P
// by the rule above) and FF_DMIN directions take.
constexpr size_t FF_WORK = (size_t)512 << 20;
constexpr int FF_DMIN = 4096;
struct LineSizes {
    int KS, tiles, nchunk, nkg;
    int nd;                       // directions of a launch
    size_t fold, kt, part, tab;   // bytes: kt of the launch, the others per right-hand side
    LineSizes(const int n[3], int nd_) {
        KS = ((n[0] + 1) / 2 + 3) / 4;
        tiles = n[2] * ((n[1] + FF_LINES - 1) / FF_LINES);
        nchunk = (n[2] + FF_Z - 1) / FF_Z;
        fold = (size_t)tiles * 3 * KS * 2 * 64 * sizeof(double2);
        nkg = (KS + 3) / 4;
        kt = ((size_t)tiles * nkg * sizeof(int) + 255) & ~(size_t)255;
        const size_t pd = (size_t)nchunk * 6 * sizeof(double);   // part and tab of a direction
        const size_t td = (size_t)(KS * 4 + n[1] + n[2]) * sizeof(double2);
        const size_t most = (fold < FF_WORK ? FF_WORK - fold : 0) / (pd + td) / FF_DMIN * FF_DMIN;
        nd = most >= (size_t)nd_ ? nd_ : (int)(most > FF_DMIN ? most : FF_DMIN);
        if (nd > nd_) nd = nd_;
        part = nd * pd;
        tab = (size_t)((nd + FF_DIRS - 1) / FF_DIRS) * FF_DIRS * td;
    }
    // right-hand sides of a launch, at least one
    int group(int nrhs) const {
        const size_t most = FF_WORK / (fold + part + tab);
        return (int)(most < 1 ? 1 : (most < (size_t)nrhs ? most : (size_t)nrhs));
    }
};
}  // namespace
size_t far_lines_bytes(const int n[3], int nrhs, int nd) {
    const LineSizes z(n, nd);
    return z.kt + (size_t)z.group(nrhs) * (z.fold + z.part + z.tab);
}
void launch_far_lines(const int* map, const int* perm, const double2* P, long long n3, int nrhs, const double* dirs,
                      int nd, int dstride, double k, const int lo[3], const int n[3], void* work, double2* f,
                      double* dcs, hipStream_t s) {
    const LineSizes z(n, nd);
    const int grp = z.group(nrhs);
    int* kt = (int*)work;
    double2* fold = (double2*)((char*)work + z.kt);
    double2* tab = (double2*)((char*)fold + (size_t)grp * z.fold);
    double* part = (double*)((char*)tab + (size_t)grp * z.tab);
    const size_t sm = (size_t)(NT / 64) * z.KS * 64 * sizeof(double2);
    const int nf = z.KS * 64 + (n[1] + n[2]) * FF_DIRS;
    const int per_wg = FF_DIRS * (NT / 64);
    const int groups = (nd + z.nd - 1) / z.nd;
    for (int g = 0; g < groups * ((nrhs + grp - 1) / grp); ++g) {
        const int q0 = g / groups * grp, d0 = g % groups * z.nd;
        const int nq = nrhs - q0 < grp ? nrhs - q0 : grp, ng = nd - d0 < z.nd ? nd - d0 : z.nd;
        const double* dq = dirs + ((size_t)q0 * dstride + d0) * 9;
        // (P is folded with the first directions of its group)
        const int nfold = d0 == 0 ? z.tiles * z.nkg * 3 : 0;
        hipLaunchKernelGGL(k_ff_operands, dim3(nfold + ((nf + NT - 1) / NT) * ((ng + FF_DIRS - 1) / FF_DIRS), nq),
                           dim3(NT), 0, s, map, perm, P + (size_t)q0 * n3, n3, n[0], n[1], n[2], z.KS, fold, kt,
                           nfold, dq, ng, dstride, k, lo[1], lo[2], tab);
        // one component a wavefront where that still leaves no more wavefronts
        // than the card holds at once (three per SIMD): a wavefront's tiles are
        // a chain of load latencies.  One right-hand side of 9,261 sites (21^3),
        // 74 directions: 17.2 us with three components, 9.1 with one; 722
        // directions 16.5 and 12.3
        if ((long long)((ng + FF_DIRS - 1) / FF_DIRS) * z.nchunk * nq <= FF_SPLIT)
            hipLaunchKernelGGL(k_ff_lines<1>, dim3((ng + per_wg - 1) / per_wg, 3 * z.nchunk, nq), dim3(NT), sm, s, fold,
                               kt, n[0], n[1], n[2], z.KS, tab, ng, part);
        else
            hipLaunchKernelGGL(k_ff_lines<3>, dim3((ng + per_wg - 1) / per_wg, z.nchunk, nq), dim3(NT), sm, s, fold, kt,
                               n[0], n[1], n[2], z.KS, tab, ng, part);
        const size_t o = (size_t)q0 * nd + d0;
        hipLaunchKernelGGL(k_ff_project, dim3((ng + NT - 1) / NT, nq), dim3(NT), 0, s, part, z.nchunk, dq, ng, dstride,
                           k, lo[0] + 0.5 * (n[0] - 1), nd, f + o * 2, dcs + o);
    }
}

}  // namespace dda
