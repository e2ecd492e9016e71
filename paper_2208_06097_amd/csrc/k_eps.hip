// Epsilon-driven domains (Eq. 16) and absolute-overlap pair screening
// (Eq. 17): the two grid reductions they need.
//
//   k_eps_marginals  m[o][a][k] = sum over the plane perpendicular to axis a
//                    at index k of |phi_o|^2, all three axes in one pass over
//                    phi (x and y as partial sums per group of z planes);
//   k_eps_marg_sum   sums the partials;
//   k_eps_overlap    S_p = dV sum over pair p's box of |phi_i phi_j|
//                    (one workgroup per candidate pair, wrapped indices).
//
// The interval search, the box intersections and the screening decision are
// host work (sea_api.hip); every sum here accumulates in FP64.
#include "sea_internal.h"

namespace {

constexpr int EP_BS = 256;

__device__ __forceinline__ double ld_phi(const void* phi, int f32, size_t off) {
    return f32 ? (double)(((const float*)phi)[off]) : ((const double*)phi)[off];
}

__device__ __forceinline__ int wrap_i(int k, int N) {
    int m = k % N;
    return m < 0 ? m + N : m;
}

__device__ __forceinline__ double block_sum_d(double v, double* red) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) red[wid] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < EP_BS / 64; ++w) t += red[w];
    return t;  // valid in thread 0
}

// Marginals of one orbital's planes z0 .. z0 + EM_ZC - 1; grid (plane groups,
// n_occ).  Memory bound (phi read once; one workgroup per marginal entry read
// it three times, the x marginals at one element per 64-byte segment: 7.8 ms
// for 256 orbitals on 120^3, now 0.67 ms = 5.3 TB/s).  A wavefront takes every
// fourth row y of the group's planes, a lane the points x = lane + 64 j: the
// EM_ZC planes of a row are EM_ZC x EM_XB loads in flight per lane, one
// wavefront sum per row serves all of them.  Every sum has a fixed order.
constexpr int EM_ZC = 8;   // planes per workgroup
constexpr int EM_XB = 2;   // 64-point x blocks per sweep over the rows
template <typename T>
__global__ __launch_bounds__(EP_BS) void k_eps_marginals(const T* __restrict__ phi, int N0, int N1, int N2, int nmax,
                                                         double* __restrict__ m, double* __restrict__ part) {
    __shared__ double red[EP_BS / 64][EM_XB * 64];
    __shared__ double zred[EP_BS / 64][EM_ZC];
    const int o = blockIdx.y, z0 = blockIdx.x * EM_ZC, nz = min(EM_ZC, N2 - z0);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const size_t pl = (size_t)N0 * N1;
    const T* p = phi + ((size_t)o * N2 + z0) * pl;
    double* px = part + ((size_t)o * gridDim.x + blockIdx.x) * (N0 + N1);
    double* py = px + N0;
    double zs[EM_ZC];
#pragma unroll
    for (int z = 0; z < EM_ZC; ++z) zs[z] = 0.0;
    for (int xb = 0; xb < N0; xb += EM_XB * 64) {
        double xs[EM_XB];
#pragma unroll
        for (int j = 0; j < EM_XB; ++j) xs[j] = 0.0;
        for (int y = w; y < N1; y += EP_BS / 64) {
            T f[EM_ZC][EM_XB];
#pragma unroll
            for (int z = 0; z < EM_ZC; ++z)
#pragma unroll
                for (int j = 0; j < EM_XB; ++j) {
                    const int x = xb + 64 * j + lane;
                    f[z][j] = (z < nz && x < N0) ? p[z * pl + (size_t)y * N0 + x] : T(0);
                }
            double ys = 0.0;
#pragma unroll
            for (int z = 0; z < EM_ZC; ++z)
#pragma unroll
                for (int j = 0; j < EM_XB; ++j) {
                    const double q = (double)f[z][j] * (double)f[z][j];
                    xs[j] += q;
                    ys += q;
                    zs[z] += q;
                }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) ys += __shfl_down(ys, off, 64);
            if (lane == 0) py[y] = xb ? py[y] + ys : ys;
        }
        __syncthreads();   // (the previous sweep's sums have been read)
#pragma unroll
        for (int j = 0; j < EM_XB; ++j) red[w][64 * j + lane] = xs[j];
        __syncthreads();
        const int t = threadIdx.x;
        if (t < EM_XB * 64 && xb + t < N0) px[xb + t] = (red[0][t] + red[1][t]) + (red[2][t] + red[3][t]);
    }
#pragma unroll
    for (int z = 0; z < EM_ZC; ++z) {
        double v = zs[z];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
        if (lane == 0) zred[w][z] = v;
    }
    __syncthreads();
    const int t = threadIdx.x;
    if (t < nz) m[((size_t)o * 3 + 2) * nmax + z0 + t] = (zred[0][t] + zred[1][t]) + (zred[2][t] + zred[3][t]);
}

// m[o][0], m[o][1] from the plane groups' partials; grid n_occ
__global__ __launch_bounds__(EP_BS) void k_eps_marg_sum(const double* __restrict__ part, int groups, int N0, int N1,
                                                        int nmax, double* __restrict__ m) {
    const int o = blockIdx.x, n = N0 + N1;
    for (int t = threadIdx.x; t < n; t += EP_BS) {
        double s = 0.0;
#pragma unroll 4
        for (int g = 0; g < groups; ++g) s += part[((size_t)o * groups + g) * n + t];
        m[((size_t)o * 3 + (t < N0 ? 0 : 1)) * nmax + (t < N0 ? t : t - N0)] = s;
    }
}

// one workgroup per candidate pair
__global__ __launch_bounds__(EP_BS) void k_eps_overlap(const void* __restrict__ phi, int f32, int N0, int N1, int N2,
                                                       double dV, const sea_pair* __restrict__ pairs,
                                                       double* __restrict__ S) {
    __shared__ double red[EP_BS / 64];
    const sea_pair P = pairs[blockIdx.x];
    const size_t Ng = (size_t)N0 * N1 * N2;
    const size_t oi = (size_t)P.i * Ng, oj = (size_t)P.j * Ng;
    const long n = (long)P.n[0] * P.n[1] * P.n[2];
    double s = 0.0;
    for (long t = threadIdx.x; t < n; t += EP_BS) {
        const int x = (int)(t % P.n[0]), y = (int)((t / P.n[0]) % P.n[1]), z = (int)(t / ((long)P.n[0] * P.n[1]));
        const size_t g = ((size_t)wrap_i(P.lo[2] + z, N2) * N1 + wrap_i(P.lo[1] + y, N1)) * N0 + wrap_i(P.lo[0] + x, N0);
        s += fabs(ld_phi(phi, f32, oi + g) * ld_phi(phi, f32, oj + g));
    }
    s = block_sum_d(s, red);
    if (threadIdx.x == 0) S[blockIdx.x] = dV * s;
}

}  // namespace

static int eps_groups(const int* N) { return (N[2] + EM_ZC - 1) / EM_ZC; }
size_t eps_marginals_part_doubles(const int* N, int n_occ) {
    return (size_t)n_occ * eps_groups(N) * ((size_t)N[0] + N[1]);
}

hipError_t launch_eps_marginals(const void* phi, int f32, const int* N, int n_occ, int nmax, double* m, double* part,
                                hipStream_t s) {
    const dim3 grid(eps_groups(N), n_occ);
    if (f32)
        hipLaunchKernelGGL(k_eps_marginals<float>, grid, dim3(EP_BS), 0, s, (const float*)phi, N[0], N[1], N[2], nmax, m,
                           part);
    else
        hipLaunchKernelGGL(k_eps_marginals<double>, grid, dim3(EP_BS), 0, s, (const double*)phi, N[0], N[1], N[2], nmax,
                           m, part);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_eps_marg_sum, dim3(n_occ), dim3(EP_BS), 0, s, part, eps_groups(N), N[0], N[1], nmax, m);
    return hipGetLastError();
}

hipError_t launch_eps_overlap(const void* phi, int f32, const int* N, double dV, const sea_pair* pairs, int n_pairs,
                              double* S, hipStream_t s) {
    if (n_pairs <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_eps_overlap, dim3(n_pairs), dim3(EP_BS), 0, s, phi, f32, N[0], N[1], N[2], dV, pairs, S);
    return hipGetLastError();
}
