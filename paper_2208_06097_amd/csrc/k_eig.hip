// Exact correction of a pair solve: x += A^-1 (b - A x) for the pairs whose
// spectral start misses the target.
//
// A, the O(h^12) Laplacian (negated) with zero values beyond the domain, is
// a sum of one-axis matrices, A = Tx + Ty + Tz with T the symmetric banded
// Toeplitz matrix of the stencil, so the eigenvectors Q of T on each axis
// diagonalize it: A^-1 = (Q x Q x Q) diag(1 / (tx + ty + tz)) (Q x Q x Q)^T.
// One iteration of CG preconditioned by A^-1 is this correction (its step is
// 1), and it ends at the rounding of b - A x; the sine transform of the start
// (k_dst.hip) inverts the odd continuation A_odd instead, cheaper per pass
// for odd lengths (its second even/odd fold) and exact enough for most
// domains, but as a preconditioner of CG it took up to five iterations of
// three passes, three stencil sweeps and a dot product.
//
// T is symmetric about the middle, so its eigenvectors are even or odd
// (index them 2 i and 2 i + 1) and a transform folds to two products of half
// the size:
//   forward  y_{2i}   = sum_k Qe[k][i] (a_k + a_{n-1-k}),  y_{2i+1} = sum_k Qo[k][i] (a_k - a_{n-1-k})
//   inverse  a_k = P_k + M_k, a_{n-1-k} = P_k - M_k,
//            P_k = sum_i Qe[k][i] y_{2i}, M_k = sum_i Qo[k][i] y_{2i+1}
// with k < ceil(n/2) (the middle entry of an odd length belongs to P alone).
// The eigenvectors of T depend on n alone: they are found once per device and
// kept in static arrays of the code object.
#include <mutex>

#include "sea_internal.h"

namespace {

constexpr int EG_N = 64;        // longest axis
constexpr int EG_H = 32;        // half of it
constexpr int EG_BS = 256;
constexpr int EG_LD = 66;       // LDS row pitch (doubles): rows on the lanes meet every bank
constexpr int EG_TAB = 2048;    // operand table entries per length and direction
constexpr int EG_PG = 8;        // workgroups per pair and pass, at most
// second-derivative weights of the O(h^12) central difference (App. C)
constexpr double kW[7] = {-5369.0 / 1800.0, 12.0 / 7.0, -15.0 / 56.0, 10.0 / 189.0,
                          -1.0 / 112.0, 2.0 / 1925.0, -1.0 / 16632.0};

// Operand tables of length n at (n - 1) * EG_TAB: entry ((par * 2 + b) * 8 +
// kk) * 64 + lane with row = 16 b + lane % 16 and k = 4 kk + lane / 16 is the
// matrix-core operand of lane `lane` at k step kk for output block b:
// forward Q_par[k][row] (row: the mode), inverse Q_par[row][k] (k: the mode).
__device__ double g_fwd[EG_N * EG_TAB];
__device__ double g_inv[EG_N * EG_TAB];
__device__ double g_mu[EG_N * EG_N];   // eigenvalues at h = 1 of length n at (n - 1) * 64, by mode

// Eigenvectors of one parity of one length by the cyclic Jacobi method (round-
// robin order: the 16 rotations of a round touch disjoint rows).  grid (n - 1, parity)
__global__ __launch_bounds__(EG_BS) void k_eig_tables() {
    __shared__ double A[EG_H][EG_H + 1], V[EG_H][EG_H + 1];
    __shared__ double cs[EG_H / 2][2];
    __shared__ int rot[EG_H / 2][2];
    const int n = blockIdx.x + 1, par = blockIdx.y, h = n / 2;
    const int N = par ? h : n - h;   // size of this parity's block
    auto T = [](int d) { d = d < 0 ? -d : d; return d <= 6 ? -kW[d] : 0.0; };
    for (int t = threadIdx.x; t < EG_H * EG_H; t += EG_BS) {
        const int k = t / EG_H, l = t % EG_H;
        double v = 0.0;
        if (k < N && l < N) {
            // basis (e_k +- e_{n-1-k}) / sqrt 2, and the middle point (k = h, n odd)
            const bool mk = k == h, ml = l == h;
            if (mk && ml) v = T(0);
            else if (mk || ml) v = sqrt(2.0) * T(k - l);
            else v = T(k - l) + (par ? -1.0 : 1.0) * T(k - (n - 1 - l));
        }
        A[k][l] = v;
        V[k][l] = k == l ? 1.0 : 0.0;
    }
    __syncthreads();
    for (int sweep = 0; sweep < 12; ++sweep)
        for (int r = 0; r < EG_H - 1; ++r) {
            if (threadIdx.x < EG_H / 2) {
                // round-robin pairs of round r: 31 stays, the others rotate
                const int t = threadIdx.x, m = EG_H - 1;
                const int p0 = t == 0 ? m : (r + t) % m, q0 = t == 0 ? r % m : (r + m - t) % m;
                const int p = min(p0, q0), q = max(p0, q0);
                double c = 1.0, s = 0.0;
                const double apq = A[p][q];
                if (fabs(apq) > 0.0) {
                    const double th = (A[q][q] - A[p][p]) / (2.0 * apq);
                    const double tt = (th >= 0.0 ? 1.0 : -1.0) / (fabs(th) + sqrt(th * th + 1.0));
                    c = 1.0 / sqrt(tt * tt + 1.0);
                    s = tt * c;
                }
                cs[t][0] = c;
                cs[t][1] = s;
                rot[t][0] = p;
                rot[t][1] = q;
            }
            __syncthreads();
            for (int t = threadIdx.x; t < EG_H / 2 * EG_H; t += EG_BS) {   // rows p, q
                const int k = t / EG_H, l = t % EG_H, p = rot[k][0], q = rot[k][1];
                const double c = cs[k][0], s = cs[k][1], ap = A[p][l], aq = A[q][l];
                A[p][l] = c * ap - s * aq;
                A[q][l] = s * ap + c * aq;
            }
            __syncthreads();
            for (int t = threadIdx.x; t < EG_H / 2 * EG_H; t += EG_BS) {   // columns p, q
                const int k = t / EG_H, l = t % EG_H, p = rot[k][0], q = rot[k][1];
                const double c = cs[k][0], s = cs[k][1];
                const double ap = A[l][p], aq = A[l][q], vp = V[l][p], vq = V[l][q];
                A[l][p] = c * ap - s * aq;
                A[l][q] = s * ap + c * aq;
                V[l][p] = c * vp - s * vq;
                V[l][q] = s * vp + c * vq;
            }
            __syncthreads();
        }
    // Q[k][i]: entry k < ceil(n/2) of eigenvector i of this parity
    auto Q = [&](int k, int i) -> double {
        if (k >= N || i >= N) return 0.0;
        return k == h ? V[k][i] : V[k][i] * sqrt(0.5);
    };
    for (int t = threadIdx.x; t < EG_TAB / 2; t += EG_BS) {
        const int b = t >> 9, kk = (t >> 6) & 7, lane = t & 63;
        const int row = 16 * b + (lane & 15), k = 4 * kk + (lane >> 4);
        const size_t e = (size_t)(n - 1) * EG_TAB + par * (EG_TAB / 2) + t;
        g_fwd[e] = Q(k, row);
        g_inv[e] = Q(row, k);
    }
    for (int i = threadIdx.x; i < N; i += EG_BS) g_mu[(n - 1) * EG_N + 2 * i + par] = A[i][i];
}

struct EigArgs {
    const sea_pair* pairs;
    const DevCell* cells;
    const int* pair_cell;
    const int* list;     // pairs to correct
    const int* count;    // how many
    size_t stride;       // pair layout
    size_t pstride;      // padded planes
    const double* in;
    double* out;
    double* xadd;        // inverse pass: added to this array (pair layout)
};

typedef double f64x4 __attribute__((ext_vector_type(4)));

// both parities' operands of output block b of length n
__device__ __forceinline__ void eg_ops(const double* tab, int n, int b, int lane, double t[16]) {
    const double* p = tab + (size_t)(n - 1) * EG_TAB + lane;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
        t[kk] = p[((0 + b) * 8 + kk) * 64];
        t[8 + kk] = p[((2 + b) * 8 + kk) * 64];
    }
}

// the operand pair of step k of one line: folded values (forward) or the two
// parities' modes (inverse); entries beyond the line meet zero operands
template <bool FWD>
__device__ __forceinline__ void eg_pair(const double* row, int n, int k, double& p, double& m) {
    if constexpr (FWD) {
        const double a0 = row[k];
        const int k2 = n - 1 - k;
        const double a1 = k2 > k ? row[k2] : 0.0;
        p = a0 + a1;
        m = a0 - a1;
    } else {
        p = row[2 * k];
        m = row[2 * k + 1];
    }
}

// Transforms the lines of blocks bp, bp + 1 (the rows of B) for output block
// hb.  DATA_A: lines are the A operand (result item v: line lane / 16 + 4 v,
// output index lane % 16), else the B operand (the other way round).
template <bool FWD, bool DATA_A>
__device__ __forceinline__ void eg_lines(const double* B, int n, int bp, int r, int g, const double t[16],
                                         f64x4 acc[2][2]) {
#pragma unroll
    for (int a = 0; a < 2; ++a) acc[a][0] = acc[a][1] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kk = 0; kk < 8; ++kk)
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            double p, m;
            eg_pair<FWD>(B + (16 * (bp + a) + r) * EG_LD, n, 4 * kk + g, p, m);
            if constexpr (DATA_A) {
                acc[a][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(p, t[kk], acc[a][0], 0, 0, 0);
                acc[a][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(m, t[8 + kk], acc[a][1], 0, 0, 0);
            } else {
                acc[a][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(t[kk], p, acc[a][0], 0, 0, 0);
                acc[a][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(t[8 + kk], m, acc[a][1], 0, 0, 0);
            }
            if (a == 1 && (kk & 1)) __builtin_amdgcn_sched_barrier(0);   // bounds the reads in flight
        }
}

// Where output index i of a transform of length n goes: forward the modes 2 i
// and 2 i + 1, inverse the points i and n - 1 - i; -1 where there is none.
// f(position, value)
template <bool FWD, typename F>
__device__ __forceinline__ void eg_emit(int n, int i, double even, double odd, F&& f) {
    if constexpr (FWD) {
        if (2 * i < n) f(2 * i, even);
        if (2 * i + 1 < n) f(2 * i + 1, odd);
    } else {
        const int j = n - 1 - i;
        if (i <= j) f(i, even + odd);
        if (i < j) f(j, even - odd);
    }
}

// 2-D transform of the z planes of the listed pairs: forward (pair layout in,
// padded planes out) or inverse (padded in, added to x).  One plane in LDS
// through both products, as in the sine-transform pass; memory bound.  A
// workgroup takes (pair, group) items in turn, so a launch with nothing
// listed costs a few microseconds.
template <bool FWD>
__global__ __launch_bounds__(EG_BS, 3) void k_eig_plane(EigArgs d) {
    __shared__ double B[EG_N * EG_LD];
    const int items = d.count[0] * EG_PG;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
    const int hb = w & 1, bp = 2 * (w >> 1);
    for (int it = blockIdx.x; it < items; it += gridDim.x) {
        // entries outside the plane only ever meet zero operands: finite from
        // the start, whatever the previous pair left
        __syncthreads();
        for (int t = threadIdx.x; t < EG_N * EG_LD; t += EG_BS) B[t] = 0.0;
        const int pid = d.list[it / EG_PG];
        const sea_pair P = d.pairs[pid];
        const int nx = P.n[0], ny = P.n[1], nz = P.n[2], npl = nx * ny;
        double tx[16], ty[16];
        eg_ops(FWD ? g_fwd : g_inv, nx, hb, lane, tx);
        eg_ops(FWD ? g_fwd : g_inv, ny, hb, lane, ty);
        const int pin = dst_plane_pitch(npl, !FWD), pout = dst_plane_pitch(npl, FWD);
        const double* in = d.in + (size_t)pid * (FWD ? d.stride : d.pstride);
        double* out = FWD ? d.out + (size_t)pid * d.pstride : d.xadd + (size_t)pid * d.stride;
        for (int z = it % EG_PG; z < nz; z += EG_PG) {
            __syncthreads();   // the previous plane has been written out
            for (int e = threadIdx.x; e < npl; e += EG_BS) B[e / nx * EG_LD + e % nx] = in[(size_t)z * pin + e];
            __syncthreads();
            f64x4 acc[2][2];
            // along x, written transposed (row: the x mode or point)
            eg_lines<FWD, true>(B, nx, bp, r, g, tx, acc);
            __syncthreads();
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    eg_emit<FWD>(nx, 16 * hb + r, acc[a][0][v], acc[a][1][v], [&](int c, double q) {
                        B[c * EG_LD + 16 * (bp + a) + g + 4 * v] = q;
                    });
            __syncthreads();
            // along y
            eg_lines<FWD, false>(B, ny, bp, r, g, ty, acc);
            __syncthreads();
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const int c = 16 * (bp + a) + r;
                if (c < nx)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        eg_emit<FWD>(ny, 16 * hb + g + 4 * v, acc[a][0][v], acc[a][1][v],
                                     [&](int j, double q) { B[j * EG_LD + c] = q; });
            }
            __syncthreads();
            for (int e = threadIdx.x; e < npl; e += EG_BS) {
                const double q = B[e / nx * EG_LD + e % nx];
                if (FWD) out[(size_t)z * pout + e] = q;
                else out[(size_t)z * pout + e] += q;
            }
        }
    }
}

// Along z per column: forward transform, division by the eigenvalue, inverse
// transform (padded planes in and out).
__global__ __launch_bounds__(EG_BS, 3) void k_eig_zline(EigArgs d) {
    __shared__ double U[EG_N * EG_LD];
    __shared__ double lxy[EG_N];
    const int items = d.count[0] * EG_PG;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
    const int hb = w & 1, bp = 2 * (w >> 1);
    for (int it = blockIdx.x; it < items; it += gridDim.x) {
        __syncthreads();
        for (int t = threadIdx.x; t < EG_N * EG_LD; t += EG_BS) U[t] = 0.0;
        const int pid = d.list[it / EG_PG];
        const sea_pair P = d.pairs[pid];
        const int nx = P.n[0], ny = P.n[1], nz = P.n[2], ncol = nx * ny, pp = dst_plane_pitch(ncol, 1);
        double tf[16], ti[16];
        eg_ops(g_fwd, nz, hb, lane, tf);
        eg_ops(g_inv, nz, hb, lane, ti);
        const DevCell& C = d.cells[d.pair_cell[pid]];
        const double ihx = 1.0 / (C.h[0] * C.h[0]), ihy = 1.0 / (C.h[1] * C.h[1]), ihz = 1.0 / (C.h[2] * C.h[2]);
        const double lz = lane < nz ? g_mu[(nz - 1) * EG_N + lane] * ihz : 0.0;
        const double* in = d.in + (size_t)pid * d.pstride;
        double* out = d.out + (size_t)pid * d.pstride;
        for (int c0 = it % EG_PG * EG_N; c0 < ncol; c0 += EG_PG * EG_N) {
            const int col = c0 + lane;
            __syncthreads();
            for (int z = w; z < nz; z += EG_BS / 64) U[lane * EG_LD + z] = col < ncol ? in[(size_t)z * pp + col] : 0.0;
            if (w == 0) {
                double l = 1.0;
                if (col < ncol) l = g_mu[(ny - 1) * EG_N + col / nx] * ihy + g_mu[(nx - 1) * EG_N + col % nx] * ihx;
                lxy[lane] = l;
            }
            __syncthreads();
            f64x4 acc[2][2];
            eg_lines<true, false>(U, nz, bp, r, g, tf, acc);
            __syncthreads();
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    eg_emit<true>(nz, 16 * hb + g + 4 * v, acc[a][0][v], acc[a][1][v],
                                  [&](int j, double q) { U[(16 * (bp + a) + r) * EG_LD + j] = q; });
            __syncthreads();
            if (lane < nz)   // wave w divides columns w, w + 4, ..., lane the mode
                for (int c = w; c < EG_N; c += EG_BS / 64) U[c * EG_LD + lane] /= lxy[c] + lz;
            __syncthreads();
            eg_lines<false, false>(U, nz, bp, r, g, ti, acc);
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                const int cc = c0 + 16 * (bp + a) + r;
                if (cc < ncol)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        eg_emit<false>(nz, 16 * hb + g + 4 * v, acc[a][0][v], acc[a][1][v],
                                       [&](int j, double q) { out[(size_t)j * pp + cc] = q; });
            }
        }
    }
}

constexpr int kMaxDevices = 64;
std::mutex g_eig_mu;
bool g_eig_ready[kMaxDevices] = {};

}  // namespace

// Fills the current device's tables, once per device of the process.
hipError_t eig_tables_setup(int dev) {
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_eig_mu);
    if (g_eig_ready[dev]) return hipSuccess;
    hipStream_t s = nullptr;
    hipError_t e = hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_eig_tables, dim3(EG_N, 2), dim3(EG_BS), 0, s);
    e = hipGetLastError();
    const hipError_t e2 = hipStreamSynchronize(s);
    (void)hipStreamDestroy(s);
    if (e == hipSuccess) e = e2;
    g_eig_ready[dev] = e == hipSuccess;
    return e;
}

hipError_t launch_eig_correct(const ExxArgs& a, double* r, double* tmp, const int* list, const int* count, int n_cu,
                              hipStream_t s) {
    if (a.n_pairs <= 0) return hipSuccess;
    const long items = (long)a.n_pairs * EG_PG;
    const unsigned nb = (unsigned)(items < 3L * n_cu ? items : 3L * n_cu);
    EigArgs d{};
    d.pairs = a.pairs;
    d.cells = a.cells;
    d.pair_cell = a.pair_cell;
    d.list = list;
    d.count = count;
    d.stride = a.stride;
    d.pstride = a.pstride;
    d.in = r;
    d.out = tmp;
    hipLaunchKernelGGL(k_eig_plane<true>, dim3(nb), dim3(EG_BS), 0, s, d);
    d.in = tmp;
    d.out = r;
    hipLaunchKernelGGL(k_eig_zline, dim3(nb), dim3(EG_BS), 0, s, d);
    d.in = r;
    d.out = nullptr;
    d.xadd = a.v;
    hipLaunchKernelGGL(k_eig_plane<false>, dim3(nb), dim3(EG_BS), 0, s, d);
    return hipGetLastError();
}
