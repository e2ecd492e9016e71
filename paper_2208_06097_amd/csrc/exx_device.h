// Device helpers shared by the exx kernels (k_exx.hip, k_scatter.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

#include "sea_internal.h"

// k mod N in [0, N) for any k
__device__ __forceinline__ int wrap_idx(int k, int N) {
    int m = k % N;
    return m < 0 ? m + N : m;
}

// A pointer read from device memory (a cell record) is generic to the
// compiler, and loads through it become flat loads, which also count on the
// scalar-load counter and so serialize behind scalar loads; the arrays these
// pointers address are always in global memory.
template <typename T>
using global_ptr = __attribute__((address_space(1))) const T*;
template <typename T>
__device__ __forceinline__ global_ptr<T> as_global(const T* p) {
    return (global_ptr<T>)p;
}

// orbital value from an FP64 or FP32 array
__device__ __forceinline__ double load_phi(const void* phi, int f32, size_t off) {
    return f32 ? (double)as_global((const float*)phi)[off] : as_global((const double*)phi)[off];
}

// The multipole sum's parts along a line parallel to axis AX, from the pair's
// monomial coefficients cf (84 of them, for dx^a dy^b dz^c with a + b + c <= 6,
// a the outer index, then b, then c): with the other two displacement
// components fixed (d[AX] is ignored), P_l(s) = sum_{e <= l} q[l][e] s^e for
// the displacement s along AX.
template <int AX>
__device__ __forceinline__ void me_line_coeffs(const double* cf, const double d[3], double q[SEA_LMAX + 1][SEA_LMAX + 1]) {
#pragma unroll
    for (int l = 0; l <= SEA_LMAX; ++l)
#pragma unroll
        for (int e = 0; e <= SEA_LMAX; ++e) q[l][e] = 0.0;
    double pw[3][7];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        pw[k][0] = 1.0;
#pragma unroll
        for (int e = 1; e <= 6; ++e) pw[k][e] = (k == AX) ? 1.0 : pw[k][e - 1] * d[k];
    }
    int t = 0;
#pragma unroll
    for (int ea = 0; ea <= 6; ++ea)
#pragma unroll
        for (int eb = 0; eb <= 6 - ea; ++eb)
#pragma unroll
            for (int ec = 0; ec <= 6 - ea - eb; ++ec) {
                const int e = AX == 0 ? ea : (AX == 1 ? eb : ec);
                q[ea + eb + ec][e] += cf[t++] * pw[0][ea] * pw[1][eb] * pw[2][ec];
            }
}

// 1/sqrt(x) for x > 0: the hardware estimate refined by two Newton steps
// y <- y (3 - x y^2) / 2 (each roughly doubles the correct bits, from about
// 23 to full double precision), a handful of FMAs instead of a correctly
// rounded square root and division.
__device__ __forceinline__ double rsqrt_nr(double x) {
    double y = __builtin_amdgcn_rsq(x);
    y = y * fma(-0.5 * x * y, y, 1.5);
    y = y * fma(-0.5 * x * y, y, 1.5);
    return y;
}

// Multipole potential (Eq. 10) on the line: sum_l P_l(s) r^-(2l+1), r^2 = s^2 + rt2
__device__ __forceinline__ double me_line_potential(const double q[SEA_LMAX + 1][SEA_LMAX + 1], double s, double rt2) {
    const double rinv = rsqrt_nr(s * s + rt2), rinv2 = rinv * rinv;
    double v = 0.0, pw = rinv;
#pragma unroll
    for (int l = 0; l <= SEA_LMAX; ++l) {
        double p = q[l][l];
#pragma unroll
        for (int e = l - 1; e >= 0; --e) p = p * s + q[l][e];
        v += p * pw;
        pw *= rinv2;
    }
    return v;
}
