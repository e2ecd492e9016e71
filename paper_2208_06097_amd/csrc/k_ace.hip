// ACE kernels (Eq. 18, App. A) on the small matrix: symmetrization,
// Cholesky, triangular inverse and the energy's sum of squares.  The
// tall-skinny products over the grid are in k_ace_mfma.hip.
//
// All orbital arrays are orbital-major (rows of length n_grid).
#include "sea_internal.h"
#include "k_ace.h"

namespace {

// ---------------------------------------------------------------------------
// small-matrix kernels (one workgroup)

__global__ void k_symmetrize(const double* __restrict__ M, int n, double* __restrict__ Mb) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n * n) return;
    const int i = t / n, j = t % n;
    Mb[t] = 0.5 * (M[(size_t)i * n + j] + M[(size_t)j * n + i]);
}

constexpr int CH_BS = 1024;

// Wave-wide sum (64 lanes).
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Blocked right-looking Cholesky (lower, row-major) of A into L, in place
// in L, blocks of CB: for each block column kb, one workgroup factors the
// diagonal block in LDS (column by column), a grid of workgroups solves the
// panel below it against that factor (a wavefront per row, forward
// substitution with the row's entries on the lanes), and a grid of
// 64 x 64 tiles subtracts the panel's rank-CB product from the lower
// trailing matrix.  flag[0] = 1-based index of the first non-positive
// pivot, 0 on success; every kernel stops once it is set.
constexpr int CB = 64;

__global__ __launch_bounds__(256) void k_chol_init(const double* __restrict__ A, int n, double* __restrict__ L,
                                                   int* __restrict__ flag) {
    const size_t t = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (t == 0) flag[0] = 0;
    if (t >= (size_t)n * n) return;
    const int i = (int)(t / n), j = (int)(t % n);
    L[t] = j <= i ? A[t] : 0.0;
}

// The block's lower triangle in registers, 4 x 4 elements a thread of a 16 x 16
// grid.  Step j takes the updated, unscaled column j from LDS, subtracts its
// product from the columns behind and leaves column j + 1 in the other buffer: one
// barrier and one reciprocal a step, on four wavefronts (a block of 64 59 -> 43 us
// against scaled columns, four barriers and 16 wavefronts; 16 wavefronts of this
// form 75: their divisions).  Columns are scaled at the end.
constexpr int CD_BS = 256, CD_G = 16, CD_E = CB / CD_G;
__global__ __launch_bounds__(CD_BS) void k_chol_diag(int n, int kb, double* __restrict__ L, int* __restrict__ flag) {
    __shared__ double col[2][CB], piv[CB];
    if (flag[0]) return;
    const int nb = min(CB, n - kb);
    const int tx = threadIdx.x % CD_G, ty = threadIdx.x / CD_G;
    double D[CD_E][CD_E];
#pragma unroll
    for (int a = 0; a < CD_E; ++a)
#pragma unroll
        for (int b = 0; b < CD_E; ++b) {
            const int r = ty + CD_G * a, c = tx + CD_G * b;
            D[a][b] = (r < nb && c <= r) ? L[(size_t)(kb + r) * n + kb + c] : 0.0;
            if (c == 0) col[0][r] = D[a][b];
        }
    for (int j = 0; j < nb; ++j) {
        __syncthreads();
        const double* cj = col[j & 1];
        const double p = cj[j];
        if (!(p > 0.0)) {
            if (threadIdx.x == 0) flag[0] = kb + j + 1;
            return;
        }
        if (threadIdx.x == 0) piv[j] = p;
        const double rp = 1.0 / p;
        double lr[CD_E];
#pragma unroll
        for (int a = 0; a < CD_E; ++a) lr[a] = cj[ty + CD_G * a];
#pragma unroll
        for (int b = 0; b < CD_E; ++b) {
            const int c = tx + CD_G * b;
            const double lc = cj[c] * rp;
#pragma unroll
            for (int a = 0; a < CD_E; ++a) {
                if (c > j) D[a][b] -= lr[a] * lc;   // (above the diagonal: not read)
                if (c == j + 1) col[(j + 1) & 1][ty + CD_G * a] = D[a][b];
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < CD_E; ++b) {
        const int c = tx + CD_G * b;
        if (c >= nb) continue;
        const double root = sqrt(piv[c]);
#pragma unroll
        for (int a = 0; a < CD_E; ++a) {
            const int r = ty + CD_G * a;
            if (r < nb && c <= r) L[(size_t)(kb + r) * n + kb + c] = r == c ? root : D[a][b] / root;
        }
    }
}

// rows kb + CB + 16 blockIdx.x + wave: L[i][kb..kb+CB) <- (that row) L11^-T
__global__ __launch_bounds__(CH_BS) void k_chol_trsm(int n, int kb, double* __restrict__ L, const int* __restrict__ flag) {
    __shared__ double D[CB][CB + 1];
    if (flag[0]) return;
    for (int t = threadIdx.x; t < CB * CB; t += CH_BS) {
        const int r = t / CB, c = t % CB;
        D[r][c] = c <= r ? L[(size_t)(kb + r) * n + kb + c] : 0.0;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = kb + CB + blockIdx.x * (CH_BS / 64) + wave;
    if (i >= n) return;
    double* row = L + (size_t)i * n + kb;
    double a = row[lane];
    for (int k = 0; k < CB; ++k) {
        const double yk = __shfl(a, k, 64) / D[k][k];
        if (lane == k) a = yk;
        else if (lane > k) a -= D[lane][k] * yk;
    }
    row[lane] = a;
}

// lower 64 x 64 tiles (ti >= tc) of the trailing matrix from kb + CB on:
// L[i][c] -= sum_m L[i][kb+m] L[c][kb+m]
__global__ __launch_bounds__(256) void k_chol_syrk(int n, int kb, double* __restrict__ L, const int* __restrict__ flag) {
    __shared__ double Pi[CB][CB + 1], Pc[CB][CB + 1];
    if (flag[0]) return;
    int ti = 0, rem = blockIdx.x;
    while (rem > ti) {
        rem -= ti + 1;
        ++ti;
    }
    const int tc = rem;
    const int r0 = kb + CB + ti * CB, c0 = kb + CB + tc * CB;
    for (int t = threadIdx.x; t < CB * CB; t += 256) {
        const int r = t / CB, m = t % CB;
        Pi[r][m] = r0 + r < n ? L[(size_t)(r0 + r) * n + kb + m] : 0.0;
        Pc[r][m] = c0 + r < n ? L[(size_t)(c0 + r) * n + kb + m] : 0.0;
    }
    __syncthreads();
    for (int t = threadIdx.x; t < CB * CB; t += 256) {
        const int r = t / CB, c = t % CB;
        const int i = r0 + r, j = c0 + c;
        if (i >= n || j > i) continue;
        double s = 0.0;
#pragma unroll 8
        for (int m = 0; m < CB; ++m) s += Pi[r][m] * Pc[c][m];
        L[(size_t)i * n + j] -= s;
    }
}

// X = L^{-1} (lower): workgroup c (one wavefront) forms column c by forward
// substitution, x_i = (delta_ic - sum_{c<=k<i} L[i][k] x_k) / L[i][i].  Lane l
// holds x_k, k = l mod 64, in R registers (n <= 64 R) and rows of L are loaded
// TR_AHEAD steps before their dot product, so that a step is a wave sum and a
// division and no trip to memory (32: 17 -> 13 us, 256: 180 -> 103, 257: 163 -> 131, 512:
// 432 -> 265, 513: 427 -> 367, 1024: 1372 -> 748).  At R = 16 that takes 230
// registers; larger matrices keep the column in LDS.
constexpr int TR_MAX = 4096, TR_AHEAD = 4;
template <int R>
__global__ __launch_bounds__(64) void k_trtri_small(const double* __restrict__ L, int n, double* __restrict__ X) {
    const int c = blockIdx.x, lane = threadIdx.x;
    double x[R], row[TR_AHEAD][R], diag[TR_AHEAD];
#pragma unroll
    for (int q = 0; q < R; ++q) x[q] = 0.0;
    // row i of L (its part below the diagonal; lanes past it read the diagonal)
    auto load = [&](int i, double (&r)[R], double& d) {
        const int ii = min(i, n - 1);
#pragma unroll
        for (int q = 0; q < R; ++q) r[q] = L[(size_t)ii * n + min(64 * q + lane, ii)];
        d = L[(size_t)ii * n + ii];
    };
    for (int i = lane; i < c; i += 64) X[(size_t)i * n + c] = 0.0;
#pragma unroll
    for (int u = 0; u < TR_AHEAD; ++u) load(c + u, row[u], diag[u]);
    for (int i0 = c; i0 < n; i0 += TR_AHEAD) {
#pragma unroll
        for (int u = 0; u < TR_AHEAD; ++u) {
            const int i = i0 + u;
            double s = 0.0;
#pragma unroll
            for (int q = 0; q < R; ++q) s += 64 * q + lane < i ? row[u][q] * x[q] : 0.0;
            s = wave_sum(s);
            const double xi = ((i == c ? 1.0 : 0.0) - s) / diag[u];
            if (i < n) {
#pragma unroll
                for (int q = 0; q < R; ++q)
                    if (64 * q + lane == i) x[q] = xi;
                if (lane == 0) X[(size_t)i * n + c] = xi;
            }
            load(i + TR_AHEAD, row[u], diag[u]);
        }
    }
}
__global__ __launch_bounds__(64) void k_trtri_lower(const double* __restrict__ L, int n, double* __restrict__ X) {
    __shared__ double x[TR_MAX];
    const int c = blockIdx.x;
    const int lane = threadIdx.x;
    for (int i = lane; i < c; i += 64) X[(size_t)i * n + c] = 0.0;
    for (int i = c; i < n; ++i) {
        double s = 0.0;
        for (int k = c + lane; k < i; k += 64) s += L[(size_t)i * n + k] * x[k];
        s = wave_sum(s);
        const double xi = ((i == c ? 1.0 : 0.0) - s) / L[(size_t)i * n + i];
        if (lane == 0) {
            x[i] = xi;
            X[(size_t)i * n + c] = xi;
        }
        __syncthreads();
    }
}

// Symmetric eigendecomposition A = Q diag(lambda) Q^T (App. A) by parallel
// cyclic Jacobi in one workgroup: each round rotates n/2 disjoint (p, q)
// planes chosen by a round-robin tournament (index 0 fixed, the others
// rotating), so every pair of indices meets once per sweep; rows, then
// columns and the eigenvector matrix are updated in separate phases.  The
// rotation zeroing A[p][q] uses t = tan(angle) = sgn(th)/(|th| + sqrt(th^2
// + 1)), th = (A[q][q] - A[p][p]) / (2 A[p][q]).  Sweeps stop when the
// off-diagonal Frobenius norm is below 1e-15 of the whole, or after 40.
// A (n x n, overwritten), V (n x n, eigenvectors in columns), lam (n).
constexpr int JB_BS = 1024;
constexpr int JB_MAXP = 2048;   // pairs per round (n <= 4096)

__global__ __launch_bounds__(JB_BS) void k_jacobi_eig(double* __restrict__ A, int n, double* __restrict__ V,
                                                      double* __restrict__ lam) {
    __shared__ double cs[JB_MAXP], sn[JB_MAXP];
    __shared__ int pp[JB_MAXP], qq[JB_MAXP];
    __shared__ double red[JB_BS / 64];
    __shared__ int done;
    const int m = n + (n & 1);      // even count; index n (if any) is a dummy
    const int np = m / 2;
    for (int t = threadIdx.x; t < n * n; t += JB_BS) V[t] = (t / n == t % n) ? 1.0 : 0.0;
    __syncthreads();
    for (int sweep = 0; sweep < 40; ++sweep) {
        // convergence test on the off-diagonal part
        double off = 0.0, tot = 0.0;
        for (int t = threadIdx.x; t < n * n; t += JB_BS) {
            const double v = A[t] * A[t];
            tot += v;
            if (t / n != t % n) off += v;
        }
        off = wave_sum(off);
        tot = wave_sum(tot);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = off;
        __syncthreads();
        if (threadIdx.x == 0) {
            double o2 = 0.0;
            for (int w = 0; w < JB_BS / 64; ++w) o2 += red[w];
            red[0] = o2;
        }
        __syncthreads();
        const double offs = red[0];
        __syncthreads();
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = tot;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t2 = 0.0;
            for (int w = 0; w < JB_BS / 64; ++w) t2 += red[w];
            done = !(offs > 1e-30 * t2);
        }
        __syncthreads();
        if (done) break;
        for (int r = 0; r < m - 1; ++r) {
            for (int k = threadIdx.x; k < np; k += JB_BS) {
                auto idx = [&](int t) { return t == 0 ? 0 : ((t - 1 + r) % (m - 1)) + 1; };
                int p = idx(k), q = idx(m - 1 - k);
                if (p > q) { const int tmp = p; p = q; q = tmp; }
                double c = 1.0, sv = 0.0;
                if (q < n) {
                    const double apq = A[(size_t)p * n + q];
                    if (apq != 0.0) {
                        const double th = (A[(size_t)q * n + q] - A[(size_t)p * n + p]) / (2.0 * apq);
                        const double t = (th >= 0.0 ? 1.0 : -1.0) / (fabs(th) + sqrt(th * th + 1.0));
                        c = 1.0 / sqrt(t * t + 1.0);
                        sv = t * c;
                    }
                }
                cs[k] = c;
                sn[k] = sv;
                pp[k] = p;
                qq[k] = q;
            }
            __syncthreads();
            // rows p, q <- P^T A
            for (int t = threadIdx.x; t < np * n; t += JB_BS) {
                const int k = t / n, j = t % n;
                const int p = pp[k], q = qq[k];
                if (q >= n || sn[k] == 0.0) continue;
                const double a = A[(size_t)p * n + j], b = A[(size_t)q * n + j];
                A[(size_t)p * n + j] = cs[k] * a - sn[k] * b;
                A[(size_t)q * n + j] = sn[k] * a + cs[k] * b;
            }
            __syncthreads();
            // columns p, q <- A P and V P
            for (int t = threadIdx.x; t < np * n; t += JB_BS) {
                const int k = t / n, i = t % n;
                const int p = pp[k], q = qq[k];
                if (q >= n || sn[k] == 0.0) continue;
                const double a = A[(size_t)i * n + p], b = A[(size_t)i * n + q];
                A[(size_t)i * n + p] = cs[k] * a - sn[k] * b;
                A[(size_t)i * n + q] = sn[k] * a + cs[k] * b;
                const double va = V[(size_t)i * n + p], vb = V[(size_t)i * n + q];
                V[(size_t)i * n + p] = cs[k] * va - sn[k] * vb;
                V[(size_t)i * n + q] = sn[k] * va + cs[k] * vb;
            }
            __syncthreads();
        }
    }
    for (int i = threadIdx.x; i < n; i += JB_BS) lam[i] = A[(size_t)i * n + i];
}

__global__ void k_transpose(const double* __restrict__ X, int n, double* __restrict__ Y) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n * n) return;
    Y[(size_t)(t % n) * n + t / n] = X[t];
}

// T[k][i] = Q[i][k] / sqrt(|lambda_k|) (zero for |lambda_k| <= 1e-14 max|lambda|),
// the map W -> zeta = W Q |Lambda|^{-1/2} in the layout of the xi product.
__global__ void k_eig_transform(const double* __restrict__ Q, const double* __restrict__ lam, int n,
                                double* __restrict__ T) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n * n) return;
    const int k = t / n, i = t % n;
    double lmax = 0.0;
    for (int q = 0; q < n; ++q) lmax = fmax(lmax, fabs(lam[q]));
    const double l = fabs(lam[k]);
    T[t] = l > 1e-14 * lmax ? Q[(size_t)i * n + k] / sqrt(l) : 0.0;
}

constexpr int SQ_BS = 1024, SQ_U = 8;   // (256 x 256: 61 -> 11 us against 256 threads, a load at a time)

__global__ __launch_bounds__(SQ_BS) void k_neg_sum_squares(const double* __restrict__ S, int mn, double* out) {
    __shared__ double red[SQ_BS / 64];
    double s = 0.0;
    for (int t0 = threadIdx.x; t0 < mn; t0 += SQ_BS * SQ_U) {
        double v[SQ_U];
#pragma unroll
        for (int u = 0; u < SQ_U; ++u) v[u] = t0 + u * SQ_BS < mn ? S[t0 + u * SQ_BS] : 0.0;
#pragma unroll
        for (int u = 0; u < SQ_U; ++u) s += v[u] * v[u];
    }
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < SQ_BS / 64; ++w) t += red[w];
        out[0] = -t;
    }
}

}  // namespace

// ---------------------------------------------------------------------------

hipError_t ace_symmetrize(const double* M, int n, double* Mb, hipStream_t s) {
    hipLaunchKernelGGL(k_symmetrize, dim3((n * n + 255) / 256), dim3(256), 0, s, M, n, Mb);
    return hipGetLastError();
}

hipError_t ace_cholesky(const double* A, int n, double* L, int* flag, hipStream_t s) {
    hipLaunchKernelGGL(k_chol_init, dim3((unsigned)(((size_t)n * n + 255) / 256)), dim3(256), 0, s, A, n, L, flag);
    for (int kb = 0; kb < n; kb += CB) {
        hipLaunchKernelGGL(k_chol_diag, dim3(1), dim3(CD_BS), 0, s, n, kb, L, flag);
        const int m = n - kb - CB;
        if (m <= 0) break;
        hipLaunchKernelGGL(k_chol_trsm, dim3((m + CH_BS / 64 - 1) / (CH_BS / 64)), dim3(CH_BS), 0, s, n, kb, L, flag);
        const int T = (m + CB - 1) / CB;
        hipLaunchKernelGGL(k_chol_syrk, dim3(T * (T + 1) / 2), dim3(256), 0, s, n, kb, L, flag);
    }
    return hipGetLastError();
}

hipError_t ace_trtri(const double* L, int n, double* X, hipStream_t s) {
    if (n > TR_MAX) return hipErrorInvalidValue;
    if (n <= 64) hipLaunchKernelGGL(k_trtri_small<1>, dim3(n), dim3(64), 0, s, L, n, X);
    else if (n <= 256) hipLaunchKernelGGL(k_trtri_small<4>, dim3(n), dim3(64), 0, s, L, n, X);
    else if (n <= 512) hipLaunchKernelGGL(k_trtri_small<8>, dim3(n), dim3(64), 0, s, L, n, X);
    else if (n <= 1024) hipLaunchKernelGGL(k_trtri_small<16>, dim3(n), dim3(64), 0, s, L, n, X);
    else hipLaunchKernelGGL(k_trtri_lower, dim3(n), dim3(64), 0, s, L, n, X);
    return hipGetLastError();
}

hipError_t ace_eig(double* A, int n, double* V, double* lam, hipStream_t s) {
    if (n > 2 * JB_MAXP) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_jacobi_eig, dim3(1), dim3(JB_BS), 0, s, A, n, V, lam);
    return hipGetLastError();
}

hipError_t ace_transpose(const double* X, int n, double* Y, hipStream_t s) {
    hipLaunchKernelGGL(k_transpose, dim3((n * n + 255) / 256), dim3(256), 0, s, X, n, Y);
    return hipGetLastError();
}

hipError_t ace_eig_transform(const double* Q, const double* lam, int n, double* T, hipStream_t s) {
    hipLaunchKernelGGL(k_eig_transform, dim3((n * n + 255) / 256), dim3(256), 0, s, Q, lam, n, T);
    return hipGetLastError();
}

hipError_t ace_neg_sum_squares(const double* S, int mn, double* out, hipStream_t s) {
    hipLaunchKernelGGL(k_neg_sum_squares, dim3(1), dim3(SQ_BS), 0, s, S, mn, out);
    return hipGetLastError();
}
