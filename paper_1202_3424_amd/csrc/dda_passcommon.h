// What the matvec kernels share: the compile-time lengths, precision
// conversions, the skip rule, the tensor product's rows and LDS sizes.
#pragma once

#include <stdexcept>
#include <type_traits>

#include "dda_kernels.h"

namespace dda {
namespace passes {

// lengths with compile-time kernels
#define DDA_CT_LENGTHS(X) X(32) X(48) X(64) X(80) X(96) X(128) X(160) X(192) X(256) X(384) X(512)

template <typename C> __device__ __forceinline__ C to_c(double2 u) {
    C c;
    c.x = u.x;
    c.y = u.y;
    return c;
}
template <typename C> __device__ __forceinline__ double2 to_d(C u) {
    double2 c;
    c.x = (double)u.x;
    c.y = (double)u.y;
    return c;
}

__device__ __forceinline__ bool skip_rhs(const RhsState* st, int chk) {
    return chk != CHK_NONE && st->status != ST_ACTIVE;
}

// g_a X + g_b Y + g_c Z for one row of the symmetric tensor product, each
// part one expression so that it contracts to a multiply and five fused
// multiply-adds (every pass-3 form uses this, so all stay bitwise identical)
template <typename C>
__device__ __forceinline__ C trow(const C& ga, const C& gb, const C& gc, const C& X, const C& Y, const C& Z) {
    C r;
    r.x = ga.x * X.x - ga.y * X.y + gb.x * Y.x - gb.y * Y.y + gc.x * Z.x - gc.y * Z.y;
    r.y = ga.x * X.y + ga.y * X.x + gb.x * Y.y + gb.y * Y.x + gc.x * Z.y + gc.y * Z.x;
    return r;
}

inline __host__ __device__ int pad_len(int L) { return L | 1; }
inline __host__ __device__ int even_up(int L) { return (L + 1) & ~1; }

// LDS of a runtime-length kernel: [twiddles (L)][tile (nlines * Lp)][scratch];
// of a compile-time kernel: [tile][scratch].
template <typename C> inline size_t smem_rt(int L, int nlines) {
    return ((size_t)even_up(L) + (size_t)nlines * pad_len(L)) * sizeof(C) + 8 * (NT / 64) * sizeof(double) + 64;
}
template <typename C> inline size_t smem_ct(int L, int nlines) {
    return (size_t)nlines * pad_len(L) * sizeof(C) + 8 * (NT / 64) * sizeof(double) + 64;
}

}  // namespace passes
}  // namespace dda
