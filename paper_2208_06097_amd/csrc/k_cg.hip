// CG Poisson solves (Eq. 9) on the pair domains, one workgroup per pair,
// persistent over a pair queue.
//
// Each workgroup owns a whole pair: the domain (nx, ny <= 64) is marched
// plane by plane in z.  A wavefront covers one x-row of 64 points; every
// thread owns COLS (x, y) columns and keeps the 13 values p(z-6..z+6) of
// each column in registers.  x neighbours come from wavefront DPP shifts
// (zero fill at the wave edge is the zero boundary), y neighbours from the
// current plane in LDS (rows of 64 with 6 zero halo rows each side).  One
// LDS barrier per plane (double-buffered plane); no halo re-reads from HBM.
//
// One CG iteration is two sweeps (8 words of state traffic per point):
//   A: p = r + beta p (in place), d = <p, A p>           reads r, p; writes p
//   B: c += alpha p, r -= alpha A p, rr = <r, r>          reads p, c, r; writes c, r
// where A p is recomputed in B instead of being stored.  A start guess
// enters as the first FP64 residual update, so no separate start-residual
// pass is needed.
//
// Paired iterate updates (XC variants, 7 words per iteration on average):
// c is read and written only every second sweep B.  Iteration k-1 leaves
// its step alpha_{k-1} p_{k-1} pending; sweep B of iteration k adds both
// steps at once, recovering p_{k-1} = (p_k - r_k) / beta_{k-1} from the p_k
// and r_k it reads anyway:
//   c += (alpha_{k-1} / beta_{k-1} + alpha_k) p_k - (alpha_{k-1} / beta_{k-1}) r_k.
// When beta_{k-1} is small (the recovery would amplify rounding) the
// pending step is added to c before sweep A of iteration k, while p still
// holds p_{k-1}, and before a residual refresh likewise.  Any
// rounding in c is caught by the FP64 refresh, which recomputes the
// residual from x.
//
// Precision: the CG state (c, r, p) is T (double or float), with reliable
// updates (residual replacement, as in mixed-precision CG of Sleijpen and
// van der Vorst): the FP64 residual r64 starts at b; whenever the recursive
// residual has dropped by another decade (FP32 state) or has met the target,
// one more sweep applies r64 -= A c with FP64 arithmetic and x += c in FP64,
// and the recursive residual is replaced by (T) r64 while the search
// direction p is kept, so the Krylov process is never restarted.  Residual
// norms and dot products accumulate in FP64.  A separate kernel recomputes
// the true residual b - A x in FP64 at exit and the pair energy.
#include <algorithm>
#include <type_traits>

#include "cg_team_join.h"
#include "sea_internal.h"

namespace {

__constant__ double kCw[7] = {-5369.0 / 1800.0, 12.0 / 7.0,      -15.0 / 56.0,     10.0 / 189.0,
                              -1.0 / 112.0,     2.0 / 1925.0,    -1.0 / 16632.0};

constexpr int LW = 64;                 // LDS row length (x)
constexpr int LH = 64 + 2 * SEA_HALO;  // LDS rows per plane (y with halo)
constexpr int PL = 64 * 64;            // slot-array plane pitch (elements)
constexpr int RZ_XCD = 8;              // workgroup k runs on XCD k mod 8

// Cubic grid: -Lap_h f = w0 f + sum_k wk (six neighbours at distance k).
template <typename T>
struct SW {
    T w[7];
};

template <typename T>
__device__ __forceinline__ SW<T> make_sw(double ih2) {
    SW<T> w;
#pragma unroll
    for (int k = 0; k < 7; ++k) w.w[k] = (T)(-kCw[k] * ih2 * (k == 0 ? 3.0 : 1.0));
    return w;
}


// Wavefront shifts by one lane with zero fill at the edge (DPP wave_shl:1 /
// wave_shr:1).  The stencil only uses sums f(x+k) + f(x-k), so it does not
// depend on which of the two is the left shift.
__device__ __forceinline__ float wshl1(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xF, 0xF, true));
}
__device__ __forceinline__ float wshr1(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xF, 0xF, true));
}
__device__ __forceinline__ double wshl1(double v) {
    int2 t = *reinterpret_cast<int2*>(&v);
    t.x = __builtin_amdgcn_update_dpp(0, t.x, 0x130, 0xF, 0xF, true);
    t.y = __builtin_amdgcn_update_dpp(0, t.y, 0x130, 0xF, 0xF, true);
    return *reinterpret_cast<double*>(&t);
}
__device__ __forceinline__ double wshr1(double v) {
    int2 t = *reinterpret_cast<int2*>(&v);
    t.x = __builtin_amdgcn_update_dpp(0, t.x, 0x138, 0xF, 0xF, true);
    t.y = __builtin_amdgcn_update_dpp(0, t.y, 0x138, 0xF, 0xF, true);
    return *reinterpret_cast<double*>(&t);
}

template <int NT>
__device__ __forceinline__ double block_sum(double v, double* lds) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0) lds[wid] = v;
    __syncthreads();
    if (wid == 0) {
        double t = (lane < NT / 64) ? lds[lane] : 0.0;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) t += __shfl_down(t, off, 64);
        if (lane == 0) lds[NT / 64] = t;
    }
    __syncthreads();
    const double r = lds[NT / 64];
    __syncthreads();
    return r;
}

// residual history entry t of pair pid (a.hist set, t <= a.hist_len)
__device__ __forceinline__ void hist_put(const ExxArgs& a, int pid, int t, double r2, double b2) {
    if (a.hist && t <= a.hist_len) a.hist[(size_t)pid * (a.hist_len + 1) + t] = b2 > 0.0 ? sqrt(r2 / b2) : 0.0;
}

__device__ __forceinline__ int wrap_idx(int k, int N) {
    int m = k % N;
    return m < 0 ? m + N : m;
}

__device__ __forceinline__ double load_phi(const void* phi, int f32, size_t off) {
    typedef __attribute__((address_space(1))) const float gfloat;
    typedef __attribute__((address_space(1))) const double gdouble;
    return f32 ? (double)((gfloat*)phi)[off] : ((gdouble*)phi)[off];
}

// a value that all lanes hold, in scalar registers
__device__ __forceinline__ double uniform(double v) {
    int2 t = *reinterpret_cast<int2*>(&v);
    t.x = __builtin_amdgcn_readfirstlane(t.x);
    t.y = __builtin_amdgcn_readfirstlane(t.y);
    return *reinterpret_cast<double*>(&t);
}

struct Empty {};

// z-march of A applied to a field f.  The input of plane z is produced in
// two steps so its global loads overlap plane work: fetch(c, z) issues the
// loads DEPTH steps before plane z enters the register queue, make(c, z, F)
// turns them into f when it does (DEPTH = 1: loads issued at the start of
// the step that consumes them; DEPTH = 2: one step earlier, twice the bytes
// in flight for more registers).  pre(c, z) prefetches per-column data for
// the output plane z before the barrier; out(c, z, A f, f, PV) consumes it.
// Column c of this thread is (x, y) = (tx, ty + TY c).  Plane nz of every
// slot array is zero and every fetch beyond the domain reads it (it stays in
// cache), so the march never moves padding through HBM.
template <typename T, typename TC, int NT, int COLS, int DEPTH, typename F, typename PV, typename FetchF,
          typename MakeF, typename PreF, typename OutF>
__device__ __forceinline__ void zmarch(int nz, T* lds, const SW<TC>& w, FetchF&& fetch, MakeF&& make, PreF&& pre,
                                       OutF&& out) {
    static_assert(DEPTH == 1 || DEPTH == 2, "prefetch depth");
    constexpr int TY = NT / 64;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    T q[COLS][13];
#pragma unroll
    for (int c = 0; c < COLS; ++c) {
#pragma unroll
        for (int k = 0; k < 6; ++k) q[c][k] = T(0);
#pragma unroll
        for (int s = 0; s < 7; ++s) q[c][6 + s] = make(c, s, fetch(c, min(s, nz)));
    }
    F nb[COLS];
    if constexpr (DEPTH == 2) {
#pragma unroll
        for (int c = 0; c < COLS; ++c) nb[c] = fetch(c, min(7, nz));
    }
    for (int z = 0; z < nz; ++z) {
        F nxt[COLS];
        if constexpr (DEPTH == 1) {
#pragma unroll
            for (int c = 0; c < COLS; ++c) nxt[c] = fetch(c, min(z + 7, nz));
        } else {
#pragma unroll
            for (int c = 0; c < COLS; ++c) {
                nxt[c] = nb[c];
                nb[c] = fetch(c, min(z + 8, nz));
            }
        }
        PV pv[COLS];
#pragma unroll
        for (int c = 0; c < COLS; ++c) pv[c] = pre(c, z);
        T* pl = lds + (z & 1) * (LW * LH) + (ty + SEA_HALO) * LW + tx;
#pragma unroll
        for (int c = 0; c < COLS; ++c) pl[TY * c * LW] = q[c][6];
        lds_sync();
#pragma unroll
        for (int c = 0; c < COLS; ++c) {
            __builtin_amdgcn_sched_barrier(0);
            const T* row = pl + TY * c * LW;
            TC s = w.w[0] * (TC)q[c][6];
            T u = q[c][6], d = q[c][6];
#pragma unroll
            for (int k = 1; k <= SEA_HALO; ++k) {
                u = wshl1(u);
                d = wshr1(d);
                s += w.w[k] * (((TC)u + (TC)d) + ((TC)row[k * LW] + (TC)row[-k * LW]) +
                               ((TC)q[c][6 + k] + (TC)q[c][6 - k]));
            }
            out(c, z, s, q[c][6], pv[c]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < COLS; ++c) {
#pragma unroll
            for (int k = 0; k < 12; ++k) q[c][k] = q[c][k + 1];
            q[c][12] = make(c, z + 7, nxt[c]);
        }
    }
}

// -Lap_h x at interior point (x,y,z) read straight from global memory (zero
// outside the interior); used for the FP64 outer residual only.
__device__ __forceinline__ double apply_A_global(const double* __restrict__ p, int id, int x, int y, int z, int nx,
                                                 int ny, int nz, double ih2) {
    const int sy = nx, sz = nx * ny;
    double s = -3.0 * kCw[0] * ih2 * p[id];
#pragma unroll
    for (int k = 1; k <= SEA_HALO; ++k) {
        const double ax = (x - k >= 0 ? p[id - k] : 0.0) + (x + k < nx ? p[id + k] : 0.0);
        const double ay = (y - k >= 0 ? p[id - k * sy] : 0.0) + (y + k < ny ? p[id + k * sy] : 0.0);
        const double az = (z - k >= 0 ? p[id - k * sz] : 0.0) + (z + k < nz ? p[id + k * sz] : 0.0);
        s += -kCw[k] * ih2 * (ax + ay + az);
    }
    return s;
}

// FP32 z-march: the reliable-update trigger replaces the recursive residual
// by the FP64 one whenever it has dropped by another factor Delta (squared
// here).
//
// Exit target: the FP64 residual must reach `target` x rel_tol.  FP32 state
// loses the Galerkin orthogonality of CG, which makes the pair energies'
// error first order in the residual with a larger constant; at 0.3 x rel_tol
// the FP32 form's E_xx error matches the FP64 form's at rel_tol (64-molecule
// cell: |dE| 1.6e-7 Ha vs 6e-8 Ha; 1.1e-6 Ha at 1.0 x rel_tol) for about 4%
// more iterations.
template <typename T>
struct Delta;
template <>
struct Delta<float> {
    static constexpr double v2 = 1e-2;
    static constexpr double target = 0.3;
};

template <typename T>
struct F2 {
    T a, b;
};
template <typename T>
struct PVsel {
    using type = F2<T>;
};

// Whether a pair's start meets the exit test |b - A x|^2 <= tol2 |b|^2,
// from the residual sweep's norms per row tile, summed in a fixed order (the
// residual kernel's second launch and the CG take the same decision).
__device__ __forceinline__ bool start_meets_target(const ExxArgs& a, int pid, double tol2, double& b2, double& q2) {
    b2 = 0.0;
    q2 = 0.0;
    for (int t = 0; t < RZ_TILES; ++t) {
        b2 += a.rnorm[((size_t)pid * RZ_TILES + t) * 2];
        q2 += a.rnorm[((size_t)pid * RZ_TILES + t) * 2 + 1];
    }
    return q2 == q2 && b2 == b2 && q2 <= tol2 * b2;
}

// Access to one slot array at element col0 + off, off uniform across the
// workgroup (plane and column offsets).  BUF: raw buffer instructions with
// the array in a buffer resource (scalar registers), the lane's column in
// one 32-bit VGPR and the uniform offset in a scalar register, so the state
// arrays cost no 64-bit address registers; otherwise plain global pointers.
template <typename T, bool BUF>
struct SlotIO;
template <typename T>
struct SlotIO<T, false> {
    T* p;
    __device__ SlotIO(T* base, int, int col0) : p(base + col0) {}
    __device__ __forceinline__ T ld(int off) const { return p[off]; }
    __device__ __forceinline__ void st(int off, T v) const { p[off] = v; }
};
template <>
struct SlotIO<float, true> {
    __amdgpu_buffer_rsrc_t rs;
    int voff;
    __device__ SlotIO(float* base, int n_elems, int col0)
        : rs(__builtin_amdgcn_make_buffer_rsrc(base, 0, n_elems * (int)sizeof(float), 0x00020000)),
          voff(col0 * (int)sizeof(float)) {}
    __device__ __forceinline__ float ld(int off) const {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, voff, off * (int)sizeof(float), 0));
    }
    __device__ __forceinline__ void st(int off, float v) const {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rs, voff, off * (int)sizeof(float), 0);
    }
};

template <typename T, int NT, int COLS, bool PREFETCH, int DEPTH, bool BUF, bool XC>
__device__ void solve_pair(const ExxArgs& a, int pid, T* lds, double* red, T* __restrict__ cc, T* __restrict__ rr,
                           T* __restrict__ pp, double* __restrict__ r64) {
    const DevCell& C = a.cells[a.pair_cell[pid]];
    const double ih2 = 1.0 / (C.h[0] * C.h[0]);
    const SW<T> w = make_sw<T>(ih2);
    const SW<double> wd = make_sw<double>(ih2);
    // Slot arrays (cc, rr, pp, r64) use a padded 64 x 64 plane: element
    // (x,y,z) at (z*64 + y)*64 + x, planes 0..nz; cells outside the domain
    // (including all of plane nz) stay zero in cc, rr, pp and r64.
    constexpr int TY = NT / 64;
    const sea_pair P = a.pairs[pid];
    const int nx = P.n[0], ny = P.n[1], nz = P.n[2];
    const int npad = PL * (nz + 1);
    const double* __restrict__ b = a.b + (size_t)pid * a.stride;
    double* __restrict__ x = a.v + (size_t)pid * a.stride;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const double tol2 = Delta<T>::target * Delta<T>::target * a.rel_tol * a.rel_tol;
    T msk[COLS];
#pragma unroll
    for (int c = 0; c < COLS; ++c) msk[c] = (tx < nx && ty + TY * c < ny) ? T(1) : T(0);
    const int col0 = ty * 64 + tx;  // column c at col0 + c*TY*64 within a plane
    const SlotIO<T, BUF> io_c(cc, npad, col0), io_r(rr, npad, col0), io_p(pp, npad, col0);

    // step alpha p of the previous iteration not yet added to c (XC)
    T pend = T(0);
    // c += pend p over the padded grid (the p array holds the pending step's
    // direction when this runs)
    auto flush = [&]() {
        for (int q = threadIdx.x; q < npad; q += NT) cc[q] += pend * pp[q];
        pend = T(0);
        __syncthreads();
    };

    // FP64 residual update: r64 -= A c and x += c, one z-march; returns |r64|^2
    auto refresh = [&]() -> double {
        double uacc = 0.0;
        if (XC && pend != T(0)) flush();
        zmarch<T, double, NT, COLS, 1, T, double>(
            nz, lds, wd, [&](int c, int z) -> T { return io_c.ld(z * PL + c * TY * 64); },
            [&](int, int, T v) -> T { return v; },
            [&](int c, int z) -> double { return r64[z * PL + col0 + c * TY * 64]; },
            [&](int c, int z, double s, T ctr, double rv) {
                const int id = z * PL + col0 + c * TY * 64;
                const double rn = (double)msk[c] * (rv - s);
                r64[id] = rn;
                uacc += rn * rn;
                if (msk[c] != T(0)) x[(z * ny + ty + TY * c) * nx + tx] += (double)ctr;
            });
        return block_sum<NT>(uacc, red);
    };

    // r64 = b on the padded grid, x = 0.  A start guess x0 (in x on entry)
    // enters as the first increment c = (T) x0, so that x and r64 = b - A x
    // stay consistent in FP64 from the start.  With start_res the start is
    // kept in FP64 in x and r64 = b - A x comes precomputed in bres; with
    // rnorm too, the norms of the residual sweep decide first whether the
    // start already meets the target (bres is then not written).
    const bool sres = a.x_nonzero && a.start_res;
    const bool fold = a.x_nonzero && !a.start_res;
    if (sres && a.rnorm) {
        double b2, q2;
        if (start_meets_target(a, pid, tol2, b2, q2)) {
            if (threadIdx.x == 0) {
                a.stats[pid].iters = 0;
                a.stats[pid].converged = 1;
                a.stats[pid].rel_res = b2 > 0.0 ? sqrt(q2 / b2) : 0.0;
                hist_put(a, pid, 0, q2, b2);
            }
            return;
        }
    }
    const double* __restrict__ br = sres ? a.bres + (size_t)pid * a.stride : nullptr;
    double bb = 0.0, r2 = 0.0;
    for (int q = threadIdx.x; q < npad; q += NT) {
        const int xx = q & 63, yy = (q >> 6) & 63, zz = q >> 12;
        double rv = 0.0;
        T c0 = T(0);
        if (xx < nx && yy < ny && zz < nz) {
            const int id = (zz * ny + yy) * nx + xx;
            const double bv = b[id];
            bb += bv * bv;
            rv = sres ? br[id] : bv;
            if (fold) c0 = (T)x[id];
            if (!sres) x[id] = 0.0;
        }
        r64[q] = rv;
        if (fold) cc[q] = c0;
        r2 += rv * rv;
    }
    bb = block_sum<NT>(bb, red);
    r2 = block_sum<NT>(r2, red);
    if (fold) r2 = refresh();

    int it = 0, conv = 0;
    // inner state from r64: r = (T) r64, c = 0 (p is kept across replacements)
    auto reset = [&](bool zero_p) -> double {
        double r2t = 0.0;
        for (int q = threadIdx.x; q < npad; q += NT) {
            const T rt = (T)r64[q];
            rr[q] = rt;
            cc[q] = T(0);
            if (zero_p) pp[q] = T(0);
            r2t += (double)rt * (double)rt;
        }
        return block_sum<NT>(r2t, red);
    };
    double rho = 0.0, rupd = r2;
    T beta = T(0);
    if (threadIdx.x == 0) hist_put(a, pid, 0, r2, bb);
    if (!(r2 == r2) || !(bb == bb)) conv = -1;
    else if (r2 <= tol2 * bb) conv = 1;
    else if (a.max_iter <= 0) conv = 0;
    else rho = reset(true);
    while (conv == 0 && rho > 0.0) {
        // XC: a pending step whose recovery would need a small beta is
        // written now, while p still holds its direction
        if (XC && pend != T(0) && !((double)beta >= a.xc_beta_min)) flush();
        // sweep A: p = r + beta p, <p, A p>
        double dacc = 0.0;
        zmarch<T, T, NT, COLS, DEPTH, F2<T>, Empty>(
            nz, lds, w,
            [&](int c, int z) -> F2<T> {
                const int o = z * PL + c * TY * 64;
                return F2<T>{io_r.ld(o), io_p.ld(o)};
            },
            [&](int c, int z, F2<T> f) -> T {
                const T pn = f.a + beta * f.b;
                // beyond the domain pn = 0 (r and p read the zero plane):
                // the store lands on plane nz, which stays zero
                io_p.st(min(z, nz) * PL + c * TY * 64, pn);
                return pn;
            },
            [&](int, int) { return Empty{}; },
            [&](int, int, T s, T ctr, Empty) { dacc += (double)ctr * (double)s; });
        const double pAp = block_sum<NT>(dacc, red);
        const T al = (T)(rho / pAp);
        // coefficients of this sweep's update c += cp p + cr r (XC: none when
        // this step is left pending)
        const bool with_c = !XC || pend != T(0);
        const T cp = XC ? (pend != T(0) ? pend / beta + al : T(0)) : al;
        const T cr = XC && pend != T(0) ? -(pend / beta) : T(0);
        // sweep B: c += alpha p, r -= alpha A p, <r, r>
        using PV = typename PVsel<T>::type;
        double racc = 0.0;
        auto fetch_p = [&](int c, int z) -> T { return io_p.ld(z * PL + c * TY * 64); };
        auto make_p = [&](int, int, T v) -> T { return v; };
        if constexpr (PREFETCH) {
            zmarch<T, T, NT, COLS, DEPTH, T, PV>(
                nz, lds, w, fetch_p, make_p,
                [&](int c, int z) -> PV {
                    const int o = z * PL + c * TY * 64;
                    return PV{with_c ? io_c.ld(o) : T(0), io_r.ld(o)};
                },
                [&](int c, int z, T s, T ctr, PV v) {
                    const int o = z * PL + c * TY * 64;
                    const T rn = msk[c] * (v.b - al * s);
                    if (with_c) {
                        if constexpr (XC) io_c.st(o, v.a + cp * ctr + cr * v.b);
                        else io_c.st(o, v.a + al * ctr);
                    }
                    io_r.st(o, rn);
                    racc += (double)rn * (double)rn;
                });
        } else {
            zmarch<T, T, NT, COLS, DEPTH, T, Empty>(
                nz, lds, w, fetch_p, make_p, [&](int, int) { return Empty{}; },
                [&](int c, int z, T s, T ctr, Empty) {
                    const int o = z * PL + c * TY * 64;
                    const T rv = io_r.ld(o);
                    const T rn = msk[c] * (rv - al * s);
                    if (with_c) {
                        if constexpr (XC) io_c.st(o, io_c.ld(o) + cp * ctr + cr * rv);
                        else io_c.st(o, io_c.ld(o) + al * ctr);
                    }
                    io_r.st(o, rn);
                    racc += (double)rn * (double)rn;
                });
        }
        const double rn2 = block_sum<NT>(racc, red);
        if constexpr (XC) pend = with_c ? T(0) : al;
        ++it;
        if (threadIdx.x == 0) hist_put(a, pid, it, rn2, bb);
        const bool nan = !(rn2 == rn2);
        if (!nan && rn2 > tol2 * bb && rn2 > Delta<T>::v2 * rupd && it < a.max_iter) {
            beta = (T)(rn2 / rho);
            rho = rn2;
            continue;
        }
        // reliable update in FP64: r64 -= A c, x += c
        r2 = refresh();
        if (!(r2 == r2)) { conv = -1; break; }
        if (r2 <= tol2 * bb) { conv = 1; break; }
        if (it >= a.max_iter) break;
        // continue the same Krylov process from the replaced residual
        const double r2t = reset(false);
        beta = (T)(r2t / rho);
        rho = r2t;
        rupd = r2;
    }
    // r64 = b - A x up to the FP64 rounding of the increments: it is the
    // residual reported for this pair
    if (threadIdx.x == 0) {
        a.stats[pid].iters = it;
        a.stats[pid].converged = conv;
        a.stats[pid].rel_res = bb > 0.0 ? sqrt(r2 / bb) : 0.0;
    }
}

template <typename T, int NT, int COLS, bool PREFETCH, int DEPTH, bool BUF, bool XC>
__global__ __launch_bounds__(NT) void k_cg_zm(ExxArgs a) {
    extern __shared__ unsigned char smem[];
    T* lds = reinterpret_cast<T*>(smem);
    __shared__ double red[NT / 64 + 1];
    __shared__ int pid_sh;
    for (int i = threadIdx.x; i < 2 * LW * LH; i += NT) lds[i] = T(0);
    char* slot = reinterpret_cast<char*>(a.slots) + (size_t)blockIdx.x * 4 * a.slot_stride * sizeof(double);
    T* cc = reinterpret_cast<T*>(slot);
    T* rr = cc + a.slot_stride;
    T* pp = rr + a.slot_stride;
    double* r64 = reinterpret_cast<double*>(slot + 3 * a.slot_stride * sizeof(double));
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) {   // the next pair, of those that no team has taken
            int qi, pid = -1;
            while ((qi = atomicAdd(a.queue_ctr, 1)) < a.n_pairs) {
                pid = a.order ? a.order[qi] : qi;  // largest domains first
                const bool team = a.team != ZM_ALL && cg_team_takes(a.pairs[pid]);
                if (team ? a.team != ZM_BESIDE && a.stats[pid].converged == CG_TEAM_LEFT : a.team != ZM_LEFT) break;
            }
            pid_sh = qi < a.n_pairs ? pid : -1;
        }
        __syncthreads();
        const int pid = pid_sh;
        if (pid < 0) break;
        solve_pair<T, NT, COLS, PREFETCH, DEPTH, BUF, XC>(a, pid, lds, red, cc, rr, pp, r64);
    }
}

// ---------------------------------------------------------------------------
// FP32-state CG on a team of workgroups.  One workgroup per pair streams 8
// words a point and iteration through memory (the arrays of 256 pairs, 0.8 GB,
// fit no cache), forms A p twice and leaves most of the chip idle in the last
// round of a pair list.  Here TM_G workgroups own TM_ZP planes each of one
// domain and keep r and A p in registers and p in LDS; c alone is in memory
// (read and written once an iteration) and p's planes go through it to the
// neighbours.  Same recurrences, point for point, as the z-march above with
// reliable updates; only the FP64 sums are added in another order.
// Measured per iteration of a 63^3 domain: 36 us on 8 CUs alone, 47 with all 32
// teams at work, which is 1.5 us a pair on the whole chip; the z-march with a pair on
// every CU takes 2.0 us a pair.  288 such pairs 289 -> 160 ms, 8 of them 107 -> 13 ms;
// over long lists, without a nearly empty last round, 0.8 of the z-march's time.
// About 17 of the 47 us are the vector ALUs, the rest the three meetings and a third
// of r and A p, which the compiler spills.
//
// What a workgroup writes for others (p's planes, c, flags, partial sums) goes
// past the caches that are not shared, in both directions (device scope).  Two
// kinds of meeting: a flag with the number of the meeting, stored when all of the
// workgroup's writes are complete, which the neighbours (p's planes) or all (c
// before a residual update) wait for; and a sum, whose parts are their own flags
// (an empty slot is all zero bits, a zero part is stored as -0), one trip through
// memory.  The c update fills the wait for the sums.
//
// A workgroup fills a CU (LDS), and only workgroups that already run form a team
// (cg_team_join.h), of one XCD (8 of its 32 CUs) on a device with nothing else to
// do: whatever else holds CUs, a team that has begun can end.  Pairs that no team
// takes, because none came together within TM_JOIN_MS, go to the z-march, which is
// launched after the teams.  The limit is some kernels of other streams long; a
// stream restricted to fewer than 8 CUs of an XCD pays it once a call.
// Waits inside a team are bounded all the same: past TM_SPIN polls (about a minute)
// the pair ends as failed, whichever member's wait it was.
constexpr int TM_G = 8, TM_ZP = 8, TM_NT = 1024;
constexpr int TM_TY = TM_NT / 64, TM_C = 64 / TM_TY;   // rows of threads; columns of a thread
constexpr unsigned TM_SPIN = 1u << 26;
constexpr int TM_JOIN_MS = 20;
static_assert(TM_G * TM_ZP >= CG_TEAM_MAX && TM_ZP >= SEA_HALO, "planes of the largest domain; halos from the neighbours");
struct TeamCtl {
    unsigned flag[TM_G];        // meetings reached by each workgroup
    int pid[2];                 // the team's pair, by parity (-1: none left)
    int pad[6];
    double part[4][TM_G];       // parts of four successive sums
};
static_assert(sizeof(TeamCtl) <= CG_TEAM_CTL && (CG_TEAM_CTL & 7) == 0, "control block");
// After the teams' control blocks: the queue's counter and the classes' words, a
// line each.
static_assert((1 + RZ_XCD) * 64 <= CG_TEAM_TAIL, "control block's tail");
template <typename T>
__device__ __forceinline__ T ld_dev(const T* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void st_dev(T* p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A class's word in memory (team_join); patience also ends with the queue.
struct TeamWord {
    unsigned* word;
    const int* queue;
    int n_pairs;
    long long t0, limit;   // wall clock ticks
    __device__ unsigned load() const { return ld_dev(word); }
    __device__ unsigned cas(unsigned expected, unsigned desired) const { return atomicCAS(word, expected, desired); }
    __device__ bool expired() const { return wall_clock64() - t0 >= limit || ld_dev(queue) >= n_pairs; }
    __device__ void pause() const { __builtin_amdgcn_s_sleep(8); }
};

// One of the team's arrays of 64 x 64 planes in memory, the lane's column in a
// VGPR and the (uniform) plane and row offset in a scalar register; device
// scope, past the caches that CUs and XCDs keep for themselves.
struct TeamIO {
    static constexpr int DEVICE = 16;   // cache policy: sc1
    __amdgpu_buffer_rsrc_t rs;
    int voff;
    __device__ TeamIO(float* base, int n_elems, int col0)
        : rs(__builtin_amdgcn_make_buffer_rsrc(base, 0, n_elems * (int)sizeof(float), 0x00020000)),
          voff(col0 * (int)sizeof(float)) {}
    __device__ __forceinline__ float ld(int off) const {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, voff, off * (int)sizeof(float), DEVICE));
    }
    __device__ __forceinline__ void st(int off, float v) const {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rs, voff, off * (int)sizeof(float), DEVICE);
    }
    // the lane's own element, not an offset from its column
    __device__ __forceinline__ float at(int elem) const {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, elem * (int)sizeof(float), 0, DEVICE));
    }
};

struct Team {
    TeamCtl* ctl;
    int g;                       // this workgroup's number in the team
    unsigned seq = 0;            // meetings so far
    int n_sum = 0;               // sums so far
    double* red;                 // LDS: one per wavefront
    double* tot;                 // LDS: the last sum
    int* fail;                   // LDS

    // All writes of this workgroup are complete and its flag says so.
    __device__ __forceinline__ void publish() {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        ++seq;
        if (threadIdx.x == 0) st_dev(&ctl->flag[g], seq);
    }
    // Waits until workgroups lo..hi have published as often as this one;
    // false once the wait has run out.
    __device__ __forceinline__ bool wait(int lo, int hi) {
        const int t = lo + (int)threadIdx.x;
        if (threadIdx.x < TM_G && t <= hi) {
            unsigned n = 0;
            while ((int)(ld_dev(&ctl->flag[t]) - seq) < 0) {
                __builtin_amdgcn_s_sleep(1);
                if (++n > TM_SPIN) {
                    *fail = 1;
                    break;
                }
            }
        }
        __syncthreads();
        return *fail == 0;
    }
    __device__ __forceinline__ bool sync() {
        publish();
        return wait(0, TM_G - 1);
    }
    // The team's sum of every thread's t, in a fixed order.  begin stores this
    // workgroup's part, end waits for all.  A slot is cleared two sums before it
    // is used again: its last readers have by then added to the sum between.
    __device__ __forceinline__ void begin(double t) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = t;
        __syncthreads();
        if (threadIdx.x == 0) {
            t = 0.0;
            for (int w = 0; w < TM_NT / 64; ++w) t += red[w];
            if (t == 0.0) t = -0.0;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the slot's clearing, two sums ago
            st_dev(&ctl->part[n_sum & 3][g], t);
            st_dev(&ctl->part[(n_sum + 2) & 3][g], 0.0);
        }
    }
    __device__ __forceinline__ bool end(double& total) {
        if (threadIdx.x < 64) {
            const int lane = threadIdx.x;
            double t = 0.0;
            if (lane < TM_G) {
                unsigned n = 0;
                while (__double_as_longlong(t = ld_dev(&ctl->part[n_sum & 3][lane])) == 0) {
                    __builtin_amdgcn_s_sleep(1);
                    if (++n > TM_SPIN) {
                        *fail = 1;
                        break;
                    }
                }
            }
#pragma unroll
            for (int off = TM_G / 2; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
            if (lane == 0) *tot = t;
        }
        ++n_sum;
        __syncthreads();
        total = *tot;
        return *fail == 0;
    }
    __device__ __forceinline__ bool sum(double t, double& total) {
        begin(t);
        return end(total);
    }
};

// What a pair's solve came to (DevStat's fields).
struct TeamEnd {
    int iters, converged;
    double rel_res;
};

// One pair; false once a wait has run out.  Thread (tx, ty) owns the points
// (tx, ty + TM_TY c, TM_ZP g + z).
// pl: LDS planes of p with SEA_HALO zero rows on either side; cc, ph: the
// team's c and exported p (planes of 64 x 64), r64: the FP64 residual.
__device__ __forceinline__ bool team_solve(const ExxArgs& a, int pid, Team& tm, float* pl, const TeamIO& cc,
                                           const TeamIO& ph, double* r64, TeamEnd& end) {
    const DevCell& C = a.cells[a.pair_cell[pid]];
    const double ih2 = 1.0 / (C.h[0] * C.h[0]);
    SW<float> w = make_sw<float>(ih2);
#pragma unroll
    for (int k = 0; k < 7; ++k) w.w[k] = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(w.w[k])));
    const sea_pair P = a.pairs[pid];
    const int nx = P.n[0], ny = P.n[1], nz = P.n[2];
    const double* __restrict__ b = a.b + (size_t)pid * a.stride;
    double* __restrict__ x = a.v + (size_t)pid * a.stride;
    int tid = threadIdx.x;
    const int z0 = TM_ZP * tm.g, nown = min(max(nz - z0, 0), TM_ZP);   // this workgroup's planes: z0 + [0, nown)
    const double tol2 = Delta<float>::target * Delta<float>::target * a.rel_tol * a.rel_tol;
    const bool lead = tm.g == 0 && threadIdx.x == 0;
    auto msk = [&](int c) { return ((tid & 63) < nx && (tid >> 6) + TM_TY * c < ny) ? 1.0f : 0.0f; };
    auto off = [&](int c, int z) { return (z0 + z) * PL + c * TM_TY * 64; };   // and the lane's column
    // Uniform values that each unrolled part takes anew: kept across the
    // iterations, the offsets and conditions of all points (and, through their
    // spills, vector registers) would be held throughout.
    // A value that is computed where it stands (the compiler would otherwise
    // load everything of a sweep first and do the sums in the reduction).
    auto here = [](auto& v) { asm volatile("" : "+v"(v)); };
    auto fresh = [](int v) {
        asm volatile("" : "+s"(v));
        return v;
    };
    float* const own = pl + threadIdx.x + SEA_HALO * LW;   // + z LH LW + TM_TY c LW
    float r[TM_C][TM_ZP], ap[TM_C][TM_ZP];

    // r64 -= A c and x += c in FP64 (c of the whole domain in memory); |r64|^2
    auto refresh = [&](double& out) -> bool {
        asm volatile("" : "+v"(tid));
        if (!tm.sync()) return false;   // every workgroup's c
        const SW<double> wd = make_sw<double>(ih2);
        double uacc = 0.0;
#pragma unroll
        for (int c = 0; c < TM_C; ++c) {
            const int y = (tid >> 6) + TM_TY * c;
#pragma unroll 1
            for (int z = 0; z < nown; ++z) {
                const int q = off(c, z) + tid;
                const float ctr = cc.at(q);
                double s = wd.w[0] * (double)ctr;
                float u = ctr, d = ctr;
#pragma unroll
                for (int k = 1; k <= SEA_HALO; ++k) {
                    u = wshl1(u);
                    d = wshr1(d);
                    // rows and planes outside: read at the point itself, taken as zero
                    const bool yu = y + k < 64, yd = y - k >= 0, zu = z0 + z + k < nz, zd = z0 + z - k >= 0;
                    const float yp = cc.at(q + (yu ? k * 64 : 0)), ym = cc.at(q - (yd ? k * 64 : 0));
                    const float zp = cc.at(q + (zu ? k * PL : 0)), zm = cc.at(q - (zd ? k * PL : 0));
                    s += wd.w[k] * (((double)u + (double)d) + ((double)(yu ? yp : 0.0f) + (double)(yd ? ym : 0.0f)) +
                                    ((double)(zu ? zp : 0.0f) + (double)(zd ? zm : 0.0f)));
                }
                const double rn = (double)msk(c) * (r64[tid + off(c, z)] - s);
                r64[tid + off(c, z)] = rn;
                uacc += rn * rn;
                if (msk(c) != 0.0f) x[((z0 + z) * ny + y) * nx + (tid & 63)] += (double)ctr;
            }
        }
        return tm.sum(uacc, out);
    };
    // inner state from r64: r = (float) r64, c = 0; |r|^2
    auto reset = [&](bool zero_p, double& out) -> bool {
        asm volatile("" : "+v"(tid));
        double uacc = 0.0;
#pragma unroll
        for (int c = 0; c < TM_C; ++c) {
            const int o = fresh(off(c, 0));
#pragma unroll
            for (int z = 0; z < TM_ZP; ++z) {
                r[c][z] = (float)r64[tid + o + z * PL];
                cc.st(o + z * PL, 0.0f);
                uacc += (double)r[c][z] * (double)r[c][z];
                here(r[c][z]);
                here(uacc);
                if (zero_p) own[z * (LH * LW) + TM_TY * c * LW] = 0.0f;
            }
        }
        return tm.sum(uacc, out);
    };

    const bool sres = a.x_nonzero && a.start_res, fold = a.x_nonzero && !a.start_res;
    if (sres && a.rnorm) {
        double b2, q2;
        if (start_meets_target(a, pid, tol2, b2, q2)) {
            end = TeamEnd{0, 1, b2 > 0.0 ? sqrt(q2 / b2) : 0.0};
            if (lead) hist_put(a, pid, 0, q2, b2);
            return true;
        }
    }
    const double* __restrict__ br = sres ? a.bres + (size_t)pid * a.stride : nullptr;
    double bb = 0.0, r2 = 0.0;
    {
        double bacc = 0.0, racc = 0.0;
#pragma unroll
        for (int c = 0; c < TM_C; ++c) {
#pragma unroll 1
            for (int z = 0; z < TM_ZP; ++z) {
                double rv = 0.0;
                float c0 = 0.0f;
                if (z < nown && msk(c) != 0.0f) {
                    const int id = ((z0 + z) * ny + (tid >> 6) + TM_TY * c) * nx + (tid & 63);
                    const double bv = b[id];
                    bacc += bv * bv;
                    rv = sres ? br[id] : bv;
                    if (fold) c0 = (float)x[id];
                    if (!sres) x[id] = 0.0;
                }
                r64[tid + off(c, z)] = rv;
                if (fold) cc.st(off(c, z), c0);
                racc += rv * rv;
            }
        }
        if (!tm.sum(bacc, bb) || !tm.sum(racc, r2)) return false;
    }
    if (fold && !refresh(r2)) return false;

    int it = 0, conv = 0;
    double rho = 0.0, rupd = r2;
    float beta = 0.0f;
    if (lead) hist_put(a, pid, 0, r2, bb);
    if (!(r2 == r2) || !(bb == bb)) conv = -1;
    else if (r2 <= tol2 * bb) conv = 1;
    else if (a.max_iter <= 0) conv = 0;
    else if (!reset(true, rho)) return false;
    while (conv == 0 && rho > 0.0) {
        // p = r + beta p, its planes out to the neighbours
#pragma unroll
        for (int c = 0; c < TM_C; ++c) {
            const int o = fresh(off(c, 0));
#pragma unroll
            for (int z = 0; z < TM_ZP; ++z) {
                float* q = own + z * (LH * LW) + TM_TY * c * LW;
                const float pn = r[c][z] + beta * *q;
                *q = pn;
                ph.st(o + z * PL, pn);
            }
        }
        tm.publish();
        if (!tm.wait(max(tm.g - 1, 0), min(tm.g + 1, TM_G - 1))) return false;
        // A p and <p, A p>, a column at a time, the next column's halo planes on
        // the way; planes outside the team's are read at an own plane and taken
        // as zero (planes past the domain within them are zero)
        float hl[SEA_HALO], hu[SEA_HALO];
        auto halo = [&](int c) {
            const int o = fresh(off(c, 0));
#pragma unroll
            for (int k = 0; k < SEA_HALO; ++k) {
                hl[k] = ph.ld(o + (tm.g > 0 ? (k - SEA_HALO) * PL : 0));
                hu[k] = ph.ld(o + (tm.g < TM_G - 1 ? (TM_ZP + k) * PL : 0));
            }
        };
        halo(0);
        double dacc = 0.0;
#pragma unroll
        for (int c = 0; c < TM_C; ++c) {
            __builtin_amdgcn_sched_barrier(0);
            float q[TM_ZP + 2 * SEA_HALO];
#pragma unroll
            for (int k = 0; k < SEA_HALO; ++k) {
                q[k] = tm.g > 0 ? hl[k] : 0.0f;
                q[SEA_HALO + TM_ZP + k] = tm.g < TM_G - 1 ? hu[k] : 0.0f;
            }
            if (c + 1 < TM_C) halo(c + 1);
#pragma unroll
            for (int z = 0; z < TM_ZP; ++z) q[SEA_HALO + z] = own[z * (LH * LW) + TM_TY * c * LW];
#pragma unroll
            for (int z = 0; z < TM_ZP; ++z) {
                const float* row = own + z * (LH * LW) + TM_TY * c * LW;
                const float ctr = q[SEA_HALO + z];
                float s = w.w[0] * ctr;
                float u = ctr, d = ctr;
#pragma unroll
                for (int k = 1; k <= SEA_HALO; ++k) {
                    u = wshl1(u);
                    d = wshr1(d);
                    s += w.w[k] *
                         ((u + d) + (row[k * LW] + row[-k * LW]) + (q[SEA_HALO + z + k] + q[SEA_HALO + z - k]));
                }
                ap[c][z] = s;
                dacc += (double)ctr * (double)s;
                here(ap[c][z]);
                here(dacc);
            }
        }
        tm.begin(dacc);
        float cv[TM_C][TM_ZP];
#pragma unroll
        for (int c = 0; c < TM_C; ++c) {
            const int o = fresh(off(c, 0));
#pragma unroll
            for (int z = 0; z < TM_ZP; ++z) cv[c][z] = cc.ld(o + z * PL);
        }
        double pAp;
        if (!tm.end(pAp)) return false;
        const float al = (float)(rho / pAp);
        asm volatile("" : "+v"(tid));
        // r -= alpha A p, <r, r>; c += alpha p
        double racc = 0.0;
#pragma unroll
        for (int c = 0; c < TM_C; ++c) {
            const int no = fresh(nown);
            const float m = msk(c);
#pragma unroll
            for (int z = 0; z < TM_ZP; ++z) {
                const float rn = (z < no ? m : 0.0f) * (r[c][z] - al * ap[c][z]);
                r[c][z] = rn;
                racc += (double)rn * (double)rn;
                here(r[c][z]);
                here(racc);
            }
        }
        tm.begin(racc);
#pragma unroll
        for (int c = 0; c < TM_C; ++c) {
            const int o = fresh(off(c, 0));
#pragma unroll
            for (int z = 0; z < TM_ZP; ++z) cc.st(o + z * PL, cv[c][z] + al * own[z * (LH * LW) + TM_TY * c * LW]);
        }
        double rn2;
        if (!tm.end(rn2)) return false;
        ++it;
        if (lead) hist_put(a, pid, it, rn2, bb);
        const bool nan = !(rn2 == rn2);
        if (!nan && rn2 > tol2 * bb && rn2 > Delta<float>::v2 * rupd && it < a.max_iter) {
            beta = (float)(rn2 / rho);
            rho = rn2;
            continue;
        }
        // reliable update in FP64: r64 -= A c, x += c
        if (!refresh(r2)) return false;
        if (!(r2 == r2)) { conv = -1; break; }
        if (r2 <= tol2 * bb) { conv = 1; break; }
        if (it >= a.max_iter) break;
        // continue the same Krylov process from the replaced residual
        double r2t;
        if (!reset(false, r2t)) return false;
        beta = (float)(r2t / rho);
        rho = r2t;
        rupd = r2;
    }
    end = TeamEnd{it, conv, bb > 0.0 ? sqrt(r2 / bb) : 0.0};
    return true;
}

// Clears the control blocks and marks the pairs that teams may take: none of them
// is solved yet.
__global__ __launch_bounds__(256) void k_team_start(ExxArgs a, int* __restrict__ ctl, int n_ctl) {
    const int t0 = blockIdx.x * 256 + threadIdx.x, nt = gridDim.x * 256;
    if (t0 == 0) a.queue_ctr[16] = 0;
    for (int t = t0; t < n_ctl; t += nt) ctl[t] = 0;
    for (int t = t0; t < a.n_pairs; t += nt)
        if (cg_team_takes(a.pairs[t])) {
            a.stats[t].iters = 0;
            a.stats[t].converged = CG_TEAM_LEFT;
            a.stats[t].rel_res = __builtin_nan("");
        }
}

// Class of workgroup k: k mod 8, the XCD it runs on; eight that arrive one after
// the other there are a team.
__global__ __launch_bounds__(TM_NT) void k_cg_team(ExxArgs a, char* ctl, int n_teams, long long limit) {
    extern __shared__ unsigned char smem[];
    float* pl = reinterpret_cast<float*>(smem);
    __shared__ double red[TM_NT / 64];
    __shared__ double tot;
    __shared__ int fail, place_sh;
    char* tail = ctl + (size_t)n_teams * CG_TEAM_CTL;
    int* queue = reinterpret_cast<int*>(tail);
    const int cls = blockIdx.x % RZ_XCD;
    if (threadIdx.x == 0) {
        TeamWord word{reinterpret_cast<unsigned*>(tail + 64 * (1 + cls)), queue, a.n_pairs, wall_clock64(), limit};
        place_sh = team_join(word, TM_G, (n_teams - cls + RZ_XCD - 1) / RZ_XCD * TM_G);
        fail = 0;
    }
    __syncthreads();
    const int place = place_sh;
    if (place < 0) return;
    const int team = place / TM_G * RZ_XCD + cls;
    Team tm{reinterpret_cast<TeamCtl*>(ctl + (size_t)team * CG_TEAM_CTL), place % TM_G};
    tm.red = red;
    tm.tot = &tot;
    tm.fail = &fail;
    const bool lead = tm.g == 0 && threadIdx.x == 0;
    for (int i = threadIdx.x; i < TM_ZP * LW * LH; i += TM_NT) pl[i] = 0.0f;
    // the team's slot: c, the exported p (floats), r64, 64 planes each (CG_TEAM_SLOT)
    constexpr int planes = TM_G * TM_ZP * PL;
    float* fs = reinterpret_cast<float*>(a.slots + (size_t)team * 4 * a.slot_stride);
    const TeamIO cc(fs, planes, threadIdx.x), ph(fs + planes, planes, threadIdx.x);
    double* r64 = a.slots + (size_t)team * 4 * a.slot_stride + planes;
    for (int turn = 0;; turn ^= 1) {
        if (lead) {   // the next of the pairs that are for teams, largest domains first
            int qi, pid = -1;
            while ((qi = atomicAdd(queue, 1)) < a.n_pairs) {
                pid = a.order ? a.order[qi] : qi;
                if (cg_team_takes(a.pairs[pid])) break;
            }
            st_dev(&tm.ctl->pid[turn], qi < a.n_pairs ? pid : -1);
        }
        if (!tm.sync()) break;
        const int pid = __builtin_amdgcn_readfirstlane(ld_dev(&tm.ctl->pid[turn]));
        if (pid < 0) break;
        // solved when all of the team say so: a member whose last wait ran out does
        // not come to this meeting, and its planes may be unfinished
        TeamEnd end;
        const bool ok = team_solve(a, pid, tm, pl, cc, ph, r64, end) && tm.sync();
        if (lead) {
            a.stats[pid].converged = ok ? end.converged : -1;
            if (ok) {
                a.stats[pid].iters = end.iters;
                a.stats[pid].rel_res = end.rel_res;
            }
        }
        if (!ok) break;
    }
}

// Pair energy e_ij = dV sum rho x and the final flags, one workgroup per pair.
// With a.epart (after the scatter) a pair whose W box of orbital i holds its
// domain has its energy from the scatter's partials, summed here in
// slot order; the others (and every pair without a.epart) sum rho x over
// the domain here.
constexpr int FIN_BS = 512;

__global__ __launch_bounds__(FIN_BS) void k_cg_finish(ExxArgs a) {
    __shared__ double red[FIN_BS / 64 + 1];
    const int pid = blockIdx.x;
    const DevCell C = a.cells[a.pair_cell[pid]];   // copied: fields stay in registers
    const sea_pair P = a.pairs[pid];
    const int nx = P.n[0], ny = P.n[1], nz = P.n[2];
    const int n = nx * ny * nz;
    const double* x = a.v + (size_t)pid * a.stride;
    const size_t oi = (size_t)P.i * C.Ng, oj = (size_t)P.j * C.Ng;
    double e = 0.0;
    if (a.epart && ep_takes(P.lo, P.n, a.dbox + 12 * (size_t)pid)) {
        const int ns = ep_slots(P, C.N);
        const double* ep = a.epart + (size_t)pid * a.ep_stride;
        for (int k = threadIdx.x; k < ns; k += FIN_BS) e += ep[k];
    } else {
        BoxWalk wk((int)threadIdx.x, FIN_BS, nx, ny);
        // FIN_U points per thread at a time, their loads issued together; one
        // copy per orbital precision, widened at the product.  The sum runs in
        // the same order as one point at a time.
        constexpr int FIN_U = 4;
        auto run = [&](auto f32) {
            using PT = typename std::conditional<decltype(f32)::value, float, double>::type;
            typedef __attribute__((address_space(1))) const PT gPT;
            const gPT* ph = (const gPT*)C.phi;
            for (int id0 = threadIdx.x; id0 < n; id0 += FIN_U * FIN_BS) {
                PT fi[FIN_U], fj[FIN_U];
                double xv[FIN_U];
#pragma unroll
                for (int k = 0; k < FIN_U; ++k) {
                    // past n the walk leaves the box along z, still a grid point
                    // after wrapping; x is then read at the box's last point
                    const size_t g = ((size_t)wrap_near(P.lo[2] + wk.z, C.N[2]) * C.N[1] + wrap_near(P.lo[1] + wk.y, C.N[1])) *
                                         C.N[0] +
                                     wrap_near(P.lo[0] + wk.x, C.N[0]);
                    fi[k] = ph[oi + g];
                    fj[k] = ph[oj + g];
                    xv[k] = x[min(id0 + k * FIN_BS, n - 1)];
                    wk.next();
                }
#pragma unroll
                for (int k = 0; k < FIN_U; ++k)
                    if (id0 + k * FIN_BS < n) e += (double)fi[k] * (double)fj[k] * xv[k];
            }
        };
        if (C.phi_f32) run(std::true_type());
        else run(std::false_type());
    }
    e = block_sum<FIN_BS>(e, red);
    if (threadIdx.x == 0) {
        DevStat st = a.stats[pid];
        if (st.converged >= 0) st.converged = (st.rel_res <= a.rel_tol) ? 1 : 0;
        if (!(st.rel_res == st.rel_res) || !(e == e)) st.converged = -1;
        st.e_ij = C.dV * e;
        st.s_abs = a.mom[(size_t)pid * SEA_NACC + SEA_NMOM];
        st.q = a.mom[(size_t)pid * SEA_NACC + SEA_NMOM + 1];
        a.stats[pid] = st;
    }
}

}  // namespace

bool cg_zm_fits(const sea_pair* pairs, int n_pairs, const double* h) {
    if (h && (h[0] != h[1] || h[0] != h[2])) return false;
    for (int k = 0; k < n_pairs; ++k)
        if (pairs[k].n[0] > 64 || pairs[k].n[1] > 64) return false;
    return true;
}

size_t cg_team_lds_bytes() { return (size_t)TM_ZP * LW * LH * sizeof(float); }
int cg_teams(int n_cu) { return n_cu / TM_G; }
int cg_team_beside(int n_cu, int n_eligible) {
    const int teams = std::min(cg_teams(n_cu), n_eligible), per_xcd = (teams + RZ_XCD - 1) / RZ_XCD * TM_G;
    return std::max(0, n_cu / RZ_XCD - per_xcd) * RZ_XCD;
}

size_t cg_zm_lds_bytes(int state_f32) { return (size_t)2 * LW * LH * (state_f32 ? sizeof(float) : sizeof(double)); }

// b - A x0 for a start guess x0 (FP64), one workgroup per pair.
__global__ __launch_bounds__(FIN_BS) void k_start_residual(ExxArgs a) {
    const int pid = blockIdx.x;
    const DevCell& C = a.cells[a.pair_cell[pid]];
    const sea_pair P = a.pairs[pid];
    const int nx = P.n[0], ny = P.n[1], nz = P.n[2];
    const int n = nx * ny * nz, nxy = nx * ny;
    const double ih2 = 1.0 / (C.h[0] * C.h[0]);
    const double* b = a.b + (size_t)pid * a.stride;
    const double* x = a.v + (size_t)pid * a.stride;
    double* br = a.bres + (size_t)pid * a.stride;
    for (int id = threadIdx.x; id < n; id += FIN_BS) {
        const int xx = id % nx, yy = (id / nx) % ny, zz = id / nxy;
        br[id] = b[id] - apply_A_global(x, id, xx, yy, zz, nx, ny, nz, ih2);
    }
}

// b - A x in FP64 for every pair of a cubic grid with nx, ny <= 64, by the
// row-tile march below.  Two launches: NORMS writes |b|^2 and |b - A x|^2 of the owned rows into
// a.rnorm[pair][tile][2] and nothing else; WRITE stores b - A x into bres
// for the pairs whose start does not meet the CG's exit test (from those
// norms; the others return at once), so a start that is already converged
// costs one read of x and b.
// Workgroups are numbered so that the row tiles of one pair run together
// on one XCD (workgroup k goes to XCD k mod 8): the rows a tile fetches
// again for its neighbours' window are then served by the same L2.
constexpr int RZ_NT = 1024;
constexpr int RZ_ROWS = 16;   // rows owned per workgroup: one per wavefront
constexpr int RZ_WR = RZ_ROWS + 2 * SEA_HALO;   // rows of the window
#ifndef SEA_RZ_PRE
#define SEA_RZ_PRE 2
#endif
#ifndef SEA_RZ_DEPTH
#define SEA_RZ_DEPTH 2
#endif
#ifndef SEA_CG64_DEPTH
#define SEA_CG64_DEPTH 1
#endif
constexpr int RZ_PRE = SEA_RZ_PRE;           // steps ahead that the owned point's data is loaded
constexpr int RZ_DEPTH = SEA_RZ_DEPTH;       // steps ahead that the residual sweep fetches x
constexpr int CG64_DEPTH = SEA_CG64_DEPTH;   // the same for the CG sweeps
static_assert(RZ_TILES * RZ_ROWS >= 64, "row tiles cover 64 rows");
static_assert(RZ_NT / 64 == RZ_ROWS, "a wavefront per owned row");

__device__ __forceinline__ void rz_block(int& pid, int& tile) {
    const int k = blockIdx.x, m = k / RZ_XCD;
    pid = (m / RZ_TILES) * RZ_XCD + k % RZ_XCD;
    tile = m % RZ_TILES;
}

// Row-tile z-march of A applied to a field f (FP64).  A workgroup owns
// RZ_ROWS rows (y) of one pair, a wavefront per row and a lane per x, and
// marches z over a window of RZ_WR rows (SEA_HALO more on each side, which
// the neighbouring workgroups own).  Only the owned rows keep the 13-plane
// register queue and form the stencil; wavefronts ty < 2 SEA_HALO also load
// one halo row's current plane into LDS for the y taps (window row ty below
// the tile, ty + RZ_ROWS above it; with fewer owned rows than halo rows a
// wavefront takes two).  fetch(yw, z) issues the loads of window
// row yw at plane z, DEPTH steps before they are used (measured: the
// residual sweep, with one plane of output loads, runs faster at DEPTH 2;
// the CG sweeps, with two, at DEPTH 1), make(yw, z, F) turns them into f,
// pre(z) loads the owned point's data of output plane z (z < nz), PRE steps
// before out(z, A f, f, PV) consumes it (issued with the step's other loads,
// so that its latency is not paid at the step's end).  Two LDS planes of
// RZ_WR x 64 doubles.
template <int DEPTH, int PRE, typename F, typename PV, typename FetchF, typename MakeF, typename PreF, typename OutF>
__device__ __forceinline__ void rtmarch(int nz, double* lds, const SW<double>& w, FetchF&& fetch, MakeF&& make,
                                        PreF&& pre, OutF&& out) {
    static_assert(DEPTH >= 1 && DEPTH <= 4, "prefetch depth");
    static_assert(PRE >= 0 && PRE <= 4, "output data prefetch depth");
    constexpr int HR = 2 * SEA_HALO;                           // halo rows of the window
    constexpr int HPW = (HR + RZ_ROWS - 1) / RZ_ROWS;           // halo rows per wavefront (at most)
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const int yo = ty + SEA_HALO;                               // owned row in the window
    // halo row h = ty + RZ_ROWS e (h < HR) sits at window row h below the
    // tile and h + RZ_ROWS above it
    auto hrow = [&](int e) { const int h = ty + RZ_ROWS * e; return h < SEA_HALO ? h : h + RZ_ROWS; };
    auto has_h = [&](int e) { return ty + RZ_ROWS * e < HR; };
    double q[13];
#pragma unroll
    for (int k = 0; k < 6; ++k) q[k] = 0.0;
#pragma unroll
    for (int s = 0; s < 7; ++s) q[6 + s] = make(yo, s, fetch(yo, min(s, nz)));
    // the owned row's plane z + 7 is fetched at step z + 1 - DEPTH (DEPTH 1:
    // in the step that uses it, at its end) and the halo rows' plane z at
    // step z - DEPTH
    F oq[DEPTH > 1 ? DEPTH - 1 : 1];
#pragma unroll
    for (int i = 0; i + 1 < DEPTH; ++i) oq[i] = fetch(yo, min(7 + i, nz));
    F hq[HPW][DEPTH];
#pragma unroll
    for (int e = 0; e < HPW; ++e)
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) hq[e][i] = has_h(e) ? fetch(hrow(e), min(i, nz)) : F{};
    PV pq[PRE > 0 ? PRE : 1];
#pragma unroll
    for (int i = 0; i < PRE; ++i) pq[i] = pre(min(i, nz - 1));
    for (int z = 0; z < nz; ++z) {
        F nxt;
        if constexpr (DEPTH == 1) {
            nxt = fetch(yo, min(z + 7, nz));
        } else {
            nxt = oq[0];
#pragma unroll
            for (int i = 0; i + 2 < DEPTH; ++i) oq[i] = oq[i + 1];
            oq[DEPTH - 2] = fetch(yo, min(z + 6 + DEPTH, nz));
        }
        F hc[HPW];
#pragma unroll
        for (int e = 0; e < HPW; ++e) {
            hc[e] = hq[e][0];
            if (has_h(e)) {
#pragma unroll
                for (int i = 0; i + 1 < DEPTH; ++i) hq[e][i] = hq[e][i + 1];
                hq[e][DEPTH - 1] = fetch(hrow(e), min(z + DEPTH, nz));
            }
        }
        PV pv;
        if constexpr (PRE == 0) {
            pv = pre(z);
        } else {
            pv = pq[0];
#pragma unroll
            for (int i = 0; i + 1 < PRE; ++i) pq[i] = pq[i + 1];
            pq[PRE - 1] = pre(min(z + PRE, nz - 1));   // (past the last plane: the last again, unused)
        }
        double* pl = lds + (z & 1) * (LW * RZ_WR);
        pl[yo * LW + tx] = q[6];
#pragma unroll
        for (int e = 0; e < HPW; ++e)
            if (has_h(e)) pl[hrow(e) * LW + tx] = make(hrow(e), z, hc[e]);
        lds_sync();
        __builtin_amdgcn_sched_barrier(0);
        const double* row = pl + yo * LW + tx;
        double sacc = w.w[0] * q[6];
        double u = q[6], d = q[6];
#pragma unroll
        for (int k = 1; k <= SEA_HALO; ++k) {
            u = wshl1(u);
            d = wshr1(d);
            sacc += w.w[k] * ((u + d) + (row[k * LW] + row[-k * LW]) + (q[6 + k] + q[6 - k]));
        }
        out(z, sacc, q[6], pv);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int k = 0; k < 12; ++k) q[k] = q[k + 1];
        q[12] = make(yo, z + 7, nxt);
    }
}

// One row tile of one pair: b - A x of its rows into bres (WRITE) or the
// tile's sums of |b|^2 and |b - A x|^2 into rnorm.
template <bool WRITE>
__device__ __forceinline__ void residual_tile(const ExxArgs& a, int pid, int tile, double* lds, double* red) {
    const sea_pair P = a.pairs[pid];
    const int nx = P.n[0], ny = P.n[1], nz = P.n[2];
    const int y0 = tile * RZ_ROWS;
    if (y0 >= ny) {
        if (!WRITE && threadIdx.x == 0) {
            a.rnorm[((size_t)pid * RZ_TILES + tile) * 2] = 0.0;
            a.rnorm[((size_t)pid * RZ_TILES + tile) * 2 + 1] = 0.0;
        }
        return;
    }
    const DevCell& C = a.cells[a.pair_cell[pid]];
    const SW<double> w = make_sw<double>(1.0 / (C.h[0] * C.h[0]));
    const double* __restrict__ x = a.v + (size_t)pid * a.stride;
    const double* __restrict__ b = a.b + (size_t)pid * a.stride;
    double* __restrict__ r = a.bres + (size_t)pid * a.stride;
    const int tx = threadIdx.x & 63, yown = y0 + (threadIdx.x >> 6);
    const bool own = yown < ny && tx < nx;
    double bb = 0.0, rr = 0.0;
    rtmarch<RZ_DEPTH, RZ_PRE, double, double>(
        nz, lds, w,
        [&](int yw, int z) -> double {   // window row yw is grid row y0 - SEA_HALO + yw
            const int y = y0 - SEA_HALO + yw;
            return (tx < nx && y >= 0 && y < ny && z < nz) ? x[(z * ny + y) * nx + tx] : 0.0;
        },
        [&](int, int, double v) -> double { return v; },
        [&](int z) -> double { return own ? b[(z * ny + yown) * nx + tx] : 0.0; },
        [&](int z, double s, double, double bv) {
            if (own) {
                const double rv = bv - s;
                if (WRITE) r[(z * ny + yown) * nx + tx] = rv;
                bb += bv * bv;
                rr += rv * rv;
            }
        });
    if (WRITE) return;
    bb = block_sum<RZ_NT>(bb, red);
    rr = block_sum<RZ_NT>(rr, red);
    if (threadIdx.x == 0) {
        a.rnorm[((size_t)pid * RZ_TILES + tile) * 2] = bb;
        a.rnorm[((size_t)pid * RZ_TILES + tile) * 2 + 1] = rr;
    }
}

template <bool WRITE>
__global__ __launch_bounds__(RZ_NT) void k_residual_zm(ExxArgs a) {
    extern __shared__ unsigned char smem[];
    __shared__ double red[RZ_NT / 64 + 1];
    int pid, tile;
    rz_block(pid, tile);
    if (pid >= a.n_pairs) return;
    if (WRITE) {
        double b2, q2;
        if (start_meets_target(a, pid, Delta<float>::target * Delta<float>::target * a.rel_tol * a.rel_tol, b2, q2)) return;
    }
    residual_tile<WRITE>(a, pid, tile, reinterpret_cast<double*>(smem), red);
}

// The same for the pairs of a refinement list (their row tiles dealt to a
// grid that fits the chip, so that an empty list costs a few microseconds).
template <bool WRITE>
__global__ __launch_bounds__(RZ_NT) void k_residual_list(ExxArgs a, const int* list, const int* count) {
    extern __shared__ unsigned char smem[];
    __shared__ double red[RZ_NT / 64 + 1];
    const int items = count[0] * RZ_TILES;
    for (int q = blockIdx.x; q < items; q += gridDim.x) {
        residual_tile<WRITE>(a, list[q / RZ_TILES], q % RZ_TILES, reinterpret_cast<double*>(smem), red);
        __syncthreads();   // the planes in LDS are reused
    }
}

// Whether each pair's start (it = 0), or its `it`-th correction, meets the
// target, from the norms of the true residual; the pairs that do not go on
// the next list while corrections are left.
constexpr double REFINE_TARGET = 0.9;   // x rel_tol
__global__ __launch_bounds__(64) void k_refine_flags(ExxArgs a, int* lists, int* counts, int it, int last) {
    const int k = blockIdx.x * 64 + threadIdx.x;
    if (k >= (it ? counts[it - 1] : a.n_pairs)) return;
    const int pid = it ? lists[(size_t)(it - 1) * a.n_pairs + k] : k;
    double b2, q2;
    const bool meets = start_meets_target(a, pid, REFINE_TARGET * REFINE_TARGET * a.rel_tol * a.rel_tol, b2, q2);
    const bool nan = !(b2 == b2) || !(q2 == q2);
    a.stats[pid].iters = it;
    a.stats[pid].converged = nan ? -1 : (meets ? 1 : 0);
    a.stats[pid].rel_res = b2 > 0.0 ? sqrt(q2 / b2) : 0.0;
    hist_put(a, pid, it, q2, b2);
    if (!meets && !nan && !last) lists[(size_t)it * a.n_pairs + atomicAdd(counts + it, 1)] = pid;
}

// ---------------------------------------------------------------------------
// FP64-state CG by row tiles (the plain FP64 form of Eq. 9).  Its 13-plane
// FP64 register queue does not fit a whole pair in one workgroup, so the
// state of every pair (x in v, r and p in their own arrays) stays in HBM
// and every CG sweep is one launch over all pairs and their row tiles (the
// residual sweep's 16 owned rows, 28-row window and XCD mapping).  The
// scalars of a pair come from per-tile partial sums, summed by every tile in
// the same fixed order, so all tiles of a pair take the same decisions:
//   sweep A (iteration k): rho_k = |r|^2; stop if rho_k <= tol^2 |b|^2, at
//     max_iter or on a non-finite value; else beta = rho_k / rho_{k-1}
//     (0 at k = 0), p = r + beta p on the window (the halo rows recomputed,
//     the owned rows written to the other of two p arrays), <p, A p>;
//   sweep B: alpha = rho_k / <p, A p>, x += alpha p, r -= alpha A p, |r|^2.
// The |r|^2 partials alternate between two slots by iteration parity, so a
// sweep never overwrites a partial another tile of its pair still reads.
// The stop test runs on the recursive residual at 0.9 x rel_tol; the true
// FP64 residual b - A x is formed afterwards for the reported rel_res.
constexpr double CG64_TARGET = 0.9;
// partial slots per row tile: |r|^2 by parity (0, 1), <p, A p> (2), |b|^2 (3)
constexpr int CG64_SLOTS = 4;
static_assert(RZ_TILES * CG64_SLOTS <= CG64_PART, "a pair's partial sums");

__device__ __forceinline__ double cg64_sum(const ExxArgs& a, int pid, int slot) {
    double s = 0.0;
    for (int t = 0; t < RZ_TILES; ++t) s += a.cg_part[(size_t)pid * CG64_PART + t * CG64_SLOTS + slot];
    return s;
}

// Sweep A's decisions of iteration k: whether pair pid goes on, and beta.
// `lead` is the one thread of the pair that records them.
__device__ __forceinline__ bool cg64_goes_on(const ExxArgs& a, int pid, int k, double rho, double bb, bool lead) {
    const double tol2 = CG64_TARGET * CG64_TARGET * a.rel_tol * a.rel_tol;
    const bool nan = !(rho == rho) || !(bb == bb);
    if (lead) hist_put(a, pid, k, rho, bb);
    if (nan || rho <= tol2 * bb || k >= a.max_iter) {
        if (lead) {
            a.stats[pid].iters = k;
            a.stats[pid].converged = nan ? -1 : (rho <= tol2 * bb ? 1 : 0);
            a.stats[pid].rel_res = bb > 0.0 ? sqrt(rho / bb) : 0.0;
            a.cg_done[pid] = 1;
        }
        return false;
    }
    if (lead) {
        atomicAdd(a.cg_active + k, 1);
        a.cg_rho[(size_t)pid * 2 + (k & 1)] = rho;
    }
    return true;
}

__global__ __launch_bounds__(RZ_NT) void k_cg64_init(ExxArgs a) {
    extern __shared__ unsigned char smem[];
    double* lds = reinterpret_cast<double*>(smem);
    __shared__ double red[RZ_NT / 64 + 1];
    int pid, tile;
    rz_block(pid, tile);
    if (pid >= a.n_pairs) return;
    const sea_pair P = a.pairs[pid];
    const int nx = P.n[0], ny = P.n[1], nz = P.n[2];
    const int y0 = tile * RZ_ROWS;
    if (cg64_small(P)) return;
    double* part = a.cg_part + (size_t)pid * CG64_PART + tile * CG64_SLOTS;
    if (tile == 0 && threadIdx.x == 0) a.cg_done[pid] = 0;
    if (y0 >= ny) {
        if (threadIdx.x == 0)
            for (int q = 0; q < CG64_SLOTS; ++q) part[q] = 0.0;
        return;
    }
    const DevCell& C = a.cells[a.pair_cell[pid]];
    const SW<double> w = make_sw<double>(1.0 / (C.h[0] * C.h[0]));
    double* __restrict__ x = a.v + (size_t)pid * a.stride;
    const double* __restrict__ b = a.b + (size_t)pid * a.stride;
    double* __restrict__ r = a.cg_r + (size_t)pid * a.stride;
    double* __restrict__ p = a.cg_p + (size_t)pid * a.stride;   // parity 0: read by sweep A of iteration 0
    const int tx = threadIdx.x & 63, yown = y0 + (threadIdx.x >> 6);
    const bool own = yown < ny && tx < nx;
    const bool x0 = a.x_nonzero;
    double bb = 0.0, rr = 0.0;
    rtmarch<CG64_DEPTH, RZ_PRE, double, double>(
        nz, lds, w,
        [&](int yw, int z) -> double {
            const int y = y0 - SEA_HALO + yw;
            return (x0 && tx < nx && y >= 0 && y < ny && z < nz) ? x[(z * ny + y) * nx + tx] : 0.0;
        },
        [&](int, int, double v) -> double { return v; },
        [&](int z) -> double { return own ? b[(z * ny + yown) * nx + tx] : 0.0; },
        [&](int z, double s, double, double bv) {
            if (own) {
                const int id = (z * ny + yown) * nx + tx;
                const double rv = bv - s;
                r[id] = rv;
                p[id] = rv;
                if (!x0) x[id] = 0.0;
                bb += bv * bv;
                rr += rv * rv;
            }
        });
    bb = block_sum<RZ_NT>(bb, red);
    rr = block_sum<RZ_NT>(rr, red);
    if (threadIdx.x == 0) {
        for (int q = 0; q < CG64_SLOTS; ++q) part[q] = 0.0;
        part[0] = rr;
        part[3] = bb;
    }
}

template <int SWEEP>
__global__ __launch_bounds__(RZ_NT) void k_cg64_sweep(ExxArgs a) {
    extern __shared__ unsigned char smem[];
    double* lds = reinterpret_cast<double*>(smem);
    __shared__ double red[RZ_NT / 64 + 1];
    int pid, tile;
    rz_block(pid, tile);
    if (pid >= a.n_pairs || a.cg_done[pid]) return;
    const int k = a.cg_it;
    const sea_pair P = a.pairs[pid];
    if (cg64_small(P)) return;
    const double rho = cg64_sum(a, pid, k & 1);
    if (SWEEP == 0 && !cg64_goes_on(a, pid, k, rho, cg64_sum(a, pid, 3), tile == 0 && threadIdx.x == 0)) return;
    const int nx = P.n[0], ny = P.n[1], nz = P.n[2];
    const int y0 = tile * RZ_ROWS;
    double* part = a.cg_part + (size_t)pid * CG64_PART + tile * CG64_SLOTS;
    if (y0 >= ny) {
        if (threadIdx.x == 0) part[SWEEP == 0 ? 2 : ((k + 1) & 1)] = 0.0;
        return;
    }
    const DevCell& C = a.cells[a.pair_cell[pid]];
    const SW<double> w = make_sw<double>(1.0 / (C.h[0] * C.h[0]));
    double* __restrict__ x = a.v + (size_t)pid * a.stride;
    double* __restrict__ r = a.cg_r + (size_t)pid * a.stride;
    // p by iteration parity: sweep A of iteration k reads p_k from array
    // k & 1 (every tile reads its window's halo rows there, owned by other
    // tiles) and writes p_{k+1} = r + beta p_k into the other array, which
    // sweep B then reads
    const double* __restrict__ p_in = a.cg_p + ((size_t)(k & 1) * a.n_pairs + pid) * a.stride;
    double* __restrict__ p = a.cg_p + ((size_t)((k + 1) & 1) * a.n_pairs + pid) * a.stride;
    const int tx = threadIdx.x & 63, yown = y0 + (threadIdx.x >> 6);
    const bool own = yown < ny && tx < nx;
    auto inwin = [&](int yw, int z) {   // window row yw is grid row y0 - SEA_HALO + yw
        const int y = y0 - SEA_HALO + yw;
        return tx < nx && y >= 0 && y < ny && z < nz;
    };
    auto widx = [&](int yw, int z) { return (z * ny + y0 - SEA_HALO + yw) * nx + tx; };   // < 64^3: 32-bit
    auto oidx = [&](int z) { return (z * ny + yown) * nx + tx; };
    double acc = 0.0;
    if constexpr (SWEEP == 0) {
        // p = r + beta p over the window (the halo rows recomputed here, the
        // owned rows written), <p, A p> over the owned rows
        const double beta = k > 0 ? rho / a.cg_rho[(size_t)pid * 2 + ((k - 1) & 1)] : 0.0;
        rtmarch<CG64_DEPTH, 0, F2<double>, Empty>(
            nz, lds, w,
            [&](int yw, int z) -> F2<double> {
                if (!inwin(yw, z)) return F2<double>{0.0, 0.0};
                const int id = widx(yw, z);
                return F2<double>{r[id], p_in[id]};
            },
            [&](int, int, F2<double> f) -> double { return f.a + beta * f.b; },
            [&](int) { return Empty{}; },
            [&](int z, double s, double ctr, Empty) {
                if (own) {
                    p[oidx(z)] = ctr;
                    acc += ctr * s;
                }
            });
        acc = block_sum<RZ_NT>(acc, red);
        if (threadIdx.x == 0) part[2] = acc;
    } else {
        // x += alpha p, r -= alpha A p, |r|^2 over the owned rows
        const double alpha = rho / cg64_sum(a, pid, 2);
        rtmarch<CG64_DEPTH, RZ_PRE, double, F2<double>>(
            nz, lds, w,
            [&](int yw, int z) -> double { return inwin(yw, z) ? p[widx(yw, z)] : 0.0; },
            [&](int, int, double v) -> double { return v; },
            [&](int z) -> F2<double> {
                if (!own) return F2<double>{0.0, 0.0};
                const int id = oidx(z);
                return F2<double>{x[id], r[id]};
            },
            [&](int z, double s, double ctr, F2<double> xr) {
                if (own) {
                    const int id = oidx(z);
                    x[id] = xr.a + alpha * ctr;
                    const double rn = xr.b - alpha * s;
                    r[id] = rn;
                    acc += rn * rn;
                }
            });
        acc = block_sum<RZ_NT>(acc, red);
        if (threadIdx.x == 0) part[(k + 1) & 1] = acc;
    }
}

// The same CG on small domains (cg64_small).  There a plane-by-plane march is
// a chain of memory latencies (a 29^3 domain: 36 of them a sweep, on two
// workgroups a pair), so the domain is cut along z too: a workgroup owns
// RZ_ROWS rows of CS_ZC planes, loads what it needs (each owned column's
// planes with six more on either side, the planes' halo rows into LDS) at
// once and passes one barrier.  A p is stored, which makes sweep B a plain
// pass over the points without the stencil; the arrays of the domains this
// serves stay in the caches, where two more words a point cost less than the
// stencil again.  Partial sums per workgroup, added up by every wavefront in
// the same order.  Measured at 29^3, 77 pairs: sweep A 63 -> 21.7 us, B 76 ->
// 14.5 us (90 MB at 6.2 TB/s; they exceed the L2s).
constexpr int CS_ZC = 8;
constexpr int CS_NT = 256, CS_PTS = 8;   // sweep B: points per thread
constexpr int CS_SLOTS = 64;             // partials of one sum: <p, A p>, |r|^2 by parity, |b|^2
static_assert(4 * CS_SLOTS <= CG64_PART, "a small pair's partial sums");
static_assert((64 / RZ_ROWS) * (CG64_SMALL_NZ / CS_ZC) <= CS_SLOTS && CG64_SMALL_PTS <= CS_SLOTS * CS_NT * CS_PTS,
              "partials of the largest small domain");
__host__ __device__ inline int cs_tiles(const sea_pair& P) { return (P.n[1] + RZ_ROWS - 1) / RZ_ROWS; }
__host__ __device__ inline int cs_chunks(const sea_pair& P) { return (P.n[2] + CS_ZC - 1) / CS_ZC; }
__host__ __device__ inline int cs_blocks(const sea_pair& P) {
    return (P.n[0] * P.n[1] * P.n[2] + CS_NT * CS_PTS - 1) / (CS_NT * CS_PTS);
}
// Partial sums of one kind, one to a lane, loaded along with everything else a
// workgroup needs (which of them count follows from the domain).
__device__ __forceinline__ double cs_part(const ExxArgs& a, int pid, int kind) {
    return a.cg_part[(size_t)pid * CG64_PART + kind * CS_SLOTS + (threadIdx.x & (CS_SLOTS - 1))];
}
__device__ __forceinline__ double cs_sum(double part, int count) {
    double t = (int)(threadIdx.x & 63) < count ? part : 0.0;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) t += __shfl_xor(t, off, 64);
    return t;
}
// how many partials |r|^2 has before iteration k: the init's, then sweep B's
__device__ __forceinline__ int cs_nrho(const sea_pair& P, int k) {
    return k == 0 ? cs_tiles(P) * cs_chunks(P) : cs_blocks(P);
}
// workgroup -> (pair, its w-th of `per` workgroups), a pair's on one XCD
__device__ __forceinline__ void cs_block(int per, int& pid, int& w) {
    const int k = blockIdx.x, m = k / RZ_XCD;
    pid = (m / per) * RZ_XCD + k % RZ_XCD;
    w = m % per;
}

// INIT: r = b - A x (x = 0 without a start guess), p = r, |r|^2, |b|^2;
// else sweep A: p = r + beta p into the other p array, A p, <p, A p>.
// R = 2: rows of up to 29 points (CS_PACK) lie two to a wavefront, six idle
// lanes apart, which are the zeros that the x shifts bring in.
constexpr int CS_PACK = (64 - SEA_HALO) / 2;
template <bool INIT, int R>
__global__ __launch_bounds__(64 * RZ_ROWS / R, 4) void k_cg64_small_a(ExxArgs a, int tiles, int chunks) {
    constexpr int NTH = 64 * RZ_ROWS / R, CW = 64 / R;
    __shared__ double pl[CS_ZC][RZ_WR][CW];
    __shared__ double red[NTH / 64 + 1];
    int pid, wg;
    cs_block(tiles * chunks, pid, wg);
    if (pid >= a.n_pairs) return;
    const sea_pair P = a.pairs[pid];
    const int nx = P.n[0], ny = P.n[1], nz = P.n[2];
    const int tile = wg % tiles, chunk = wg / tiles;
    const int y0 = tile * RZ_ROWS, z0 = chunk * CS_ZC;
    if (!cg64_small(P) || (nx <= CS_PACK) != (R == 2) || y0 >= ny || z0 >= nz) return;
    const int k = a.cg_it;
    const int lane = threadIdx.x & 63;
    const int sub = R == 2 && lane >= nx + SEA_HALO;
    const int tx = lane - sub * (nx + SEA_HALO), wv = R * (threadIdx.x >> 6) + sub;   // x, row slot
    double* __restrict__ x = a.v + (size_t)pid * a.stride;
    const double* __restrict__ b = a.b + (size_t)pid * a.stride;
    double* __restrict__ r = a.cg_r + (size_t)pid * a.stride;
    const double* __restrict__ p_in = a.cg_p + ((size_t)(k & 1) * a.n_pairs + pid) * a.stride;
    double* __restrict__ p = a.cg_p + ((size_t)(INIT ? 0 : (k + 1) & 1) * a.n_pairs + pid) * a.stride;
    double* __restrict__ ap = a.cg_ap + (size_t)pid * a.stride;
    const int yown = y0 + wv, np = nx * ny;
    const bool own = yown < ny && tx < nx;
    const bool x0 = a.x_nonzero;
    // point (y, z) of the field: zero outside the domain, whose reads go to its first point
    auto in = [&](int y, int z) { return tx < nx && y >= 0 && y < ny && z >= 0 && z < nz; };
    auto load = [&](int y, int z) -> F2<double> {
        const int id = in(y, z) ? z * np + y * nx + tx : 0;
        return INIT ? F2<double>{x[id], 0.0} : F2<double>{r[id], p_in[id]};
    };
    // halo row-planes dealt to the row slots
    constexpr int HR = 2 * SEA_HALO, HE = HR * CS_ZC / RZ_ROWS;
    static_assert(HE * RZ_ROWS == HR * CS_ZC, "halo rows of a chunk");
    auto hrow = [&](int e) { const int h = (wv + RZ_ROWS * e) % HR; return h < SEA_HALO ? h : h + RZ_ROWS; };
    auto hz = [&](int e) { return (wv + RZ_ROWS * e) / HR; };
    const double prho = INIT ? 0.0 : cs_part(a, pid, 1 + (k & 1)), pbb = INIT ? 0.0 : cs_part(a, pid, 3);
    const bool lead = wg == 0 && threadIdx.x == 0;
    double beta = 0.0;
    if (INIT) {
        if (lead) a.cg_done[pid] = 0;
    } else {
        const double prev = a.cg_rho[(size_t)pid * 2 + ((k - 1) & 1)];
        if (a.cg_done[pid]) return;
        const double rho = cs_sum(prho, cs_nrho(P, k));
        if (!cg64_goes_on(a, pid, k, rho, cs_sum(pbb, cs_tiles(P) * cs_chunks(P)), lead)) return;
        if (k > 0) beta = rho / prev;
    }
    const DevCell& C = a.cells[a.pair_cell[pid]];
    SW<double> w = make_sw<double>(1.0 / (C.h[0] * C.h[0]));
#pragma unroll
    for (int i = 0; i < 7; ++i) w.w[i] = uniform(w.w[i]);
    auto field = [&](F2<double> f, int y, int z) -> double {
        if (INIT) return in(y, z) && x0 ? f.a : 0.0;
        return in(y, z) ? f.a + beta * f.b : 0.0;
    };
    double q[CS_ZC + 2 * SEA_HALO];
#pragma unroll
    for (int i = 0; i < CS_ZC + 2 * SEA_HALO; ++i)
        q[i] = field(load(yown, z0 - SEA_HALO + i), yown, z0 - SEA_HALO + i);
    const int cx = R == 2 ? (tx < nx ? tx : CW - 1) : tx;   // LDS column (idle lanes: the unused last, all zeros)
#pragma unroll
    for (int e = 0; e < HE; ++e) pl[hz(e)][hrow(e)][cx] =
        field(load(y0 - SEA_HALO + hrow(e), z0 + hz(e)), y0 - SEA_HALO + hrow(e), z0 + hz(e));
#pragma unroll
    for (int i = 0; i < CS_ZC; ++i) pl[i][wv + SEA_HALO][cx] = q[i + SEA_HALO];
    __syncthreads();
    double acc = 0.0, bacc = 0.0;
#pragma unroll
    for (int i = 0; i < CS_ZC; ++i) {
        const double ctr = q[i + SEA_HALO];
        const double* row = &pl[i][wv + SEA_HALO][cx];
        double s = w.w[0] * ctr;
        double u = ctr, d = ctr;
#pragma unroll
        for (int t = 1; t <= SEA_HALO; ++t) {
            u = wshl1(u);
            d = wshr1(d);
            s += w.w[t] * ((u + d) + (row[t * CW] + row[-t * CW]) + (q[i + SEA_HALO + t] + q[i + SEA_HALO - t]));
        }
        if (own && z0 + i < nz) {
            const int id = (z0 + i) * np + yown * nx + tx;
            if (INIT) {
                const double bv = b[id], rv = bv - s;
                r[id] = rv;
                p[id] = rv;
                if (!x0) x[id] = 0.0;
                acc += rv * rv;
                bacc += bv * bv;
            } else {
                p[id] = ctr;
                ap[id] = s;
                acc += ctr * s;
            }
        }
    }
    acc = block_sum<NTH>(acc, red);
    if (INIT) bacc = block_sum<NTH>(bacc, red);
    if (threadIdx.x == 0) {
        double* out = a.cg_part + (size_t)pid * CG64_PART + tile * cs_chunks(P) + chunk;
        out[(INIT ? 1 : 0) * CS_SLOTS] = acc;
        if (INIT) out[3 * CS_SLOTS] = bacc;
    }
}

// sweep B: x += alpha p, r -= alpha A p, |r|^2
__global__ __launch_bounds__(CS_NT) void k_cg64_small_b(ExxArgs a, int blocks) {
    __shared__ double red[CS_NT / 64 + 1];
    int pid, wg;
    cs_block(blocks, pid, wg);
    if (pid >= a.n_pairs) return;
    const sea_pair P = a.pairs[pid];
    if (!cg64_small(P) || wg >= cs_blocks(P)) return;
    const int n = P.n[0] * P.n[1] * P.n[2], k = a.cg_it;
    const double prho = cs_part(a, pid, 1 + (k & 1)), ppap = cs_part(a, pid, 0);
    double* __restrict__ x = a.v + (size_t)pid * a.stride;
    double* __restrict__ r = a.cg_r + (size_t)pid * a.stride;
    const double* __restrict__ p = a.cg_p + ((size_t)((k + 1) & 1) * a.n_pairs + pid) * a.stride;
    const double* __restrict__ ap = a.cg_ap + (size_t)pid * a.stride;
    const int id0 = wg * CS_NT * CS_PTS + threadIdx.x;
    double xv[CS_PTS], rv[CS_PTS], pv[CS_PTS], av[CS_PTS];
#pragma unroll
    for (int e = 0; e < CS_PTS; ++e) {
        const int id = min(id0 + e * CS_NT, n - 1);
        xv[e] = x[id];
        rv[e] = r[id];
        pv[e] = p[id];
        av[e] = ap[id];
    }
    if (a.cg_done[pid]) return;
    const double alpha = cs_sum(prho, cs_nrho(P, k)) / cs_sum(ppap, cs_tiles(P) * cs_chunks(P));
    double acc = 0.0;
#pragma unroll
    for (int e = 0; e < CS_PTS; ++e) {
        const int id = id0 + e * CS_NT;
        if (id < n) {
            x[id] = xv[e] + alpha * pv[e];
            const double rn = rv[e] - alpha * av[e];
            r[id] = rn;
            acc += rn * rn;
        }
    }
    acc = block_sum<CS_NT>(acc, red);
    if (threadIdx.x == 0) a.cg_part[(size_t)pid * CG64_PART + (1 + ((k + 1) & 1)) * CS_SLOTS + wg] = acc;
}

// The reported residual: the true FP64 one from the residual sweep's norms.
__global__ __launch_bounds__(64) void k_cg64_exit(ExxArgs a) {
    const int pid = blockIdx.x * 64 + threadIdx.x;
    if (pid >= a.n_pairs) return;
    double b2 = 0.0, q2 = 0.0;
    for (int t = 0; t < RZ_TILES; ++t) {
        b2 += a.rnorm[((size_t)pid * RZ_TILES + t) * 2];
        q2 += a.rnorm[((size_t)pid * RZ_TILES + t) * 2 + 1];
    }
    DevStat st = a.stats[pid];
    st.rel_res = b2 > 0.0 ? sqrt(q2 / b2) : 0.0;
    if (!(q2 == q2)) st.converged = -1;
    a.stats[pid] = st;
}

__global__ __launch_bounds__(256) void k_fill_int(int* p, size_t n) {
    for (size_t k = blockIdx.x * (size_t)256 + threadIdx.x; k < n; k += (size_t)gridDim.x * 256) p[k] = 0;
}

size_t residual_zm_lds_bytes() { return (size_t)2 * LW * RZ_WR * sizeof(double); }

hipError_t launch_residual_zm(const ExxArgs& a, hipStream_t s, bool write) {
    if (a.n_pairs <= 0) return hipSuccess;
    const int lds = (int)residual_zm_lds_bytes();
    const unsigned nb = (unsigned)((a.n_pairs + RZ_XCD - 1) / RZ_XCD) * RZ_XCD * RZ_TILES;
    hipError_t e = hipFuncSetAttribute((const void*)k_residual_zm<false>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void*)k_residual_zm<true>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_residual_zm<false>, dim3(nb), dim3(RZ_NT), lds, s, a);
    if (write) hipLaunchKernelGGL(k_residual_zm<true>, dim3(nb), dim3(RZ_NT), lds, s, a);
    return hipGetLastError();
}

static unsigned rz_blocks(int n_pairs) { return (unsigned)((n_pairs + RZ_XCD - 1) / RZ_XCD) * RZ_XCD * RZ_TILES; }

hipError_t launch_cg64_init(const ExxArgs& a, hipStream_t s) {
    if (a.n_pairs <= 0) return hipSuccess;
    const int lds = (int)residual_zm_lds_bytes();
    hipError_t e = hipFuncSetAttribute((const void*)k_cg64_init, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_cg64_init, dim3(rz_blocks(a.n_pairs)), dim3(RZ_NT), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_cg64_sweep(const ExxArgs& a, int sweep, hipStream_t s) {
    if (a.n_pairs <= 0) return hipSuccess;
    const int lds = (int)residual_zm_lds_bytes();
    const void* fn = sweep == 0 ? (const void*)k_cg64_sweep<0> : (const void*)k_cg64_sweep<1>;
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    if (sweep == 0) hipLaunchKernelGGL(k_cg64_sweep<0>, dim3(rz_blocks(a.n_pairs)), dim3(RZ_NT), lds, s, a);
    else hipLaunchKernelGGL(k_cg64_sweep<1>, dim3(rz_blocks(a.n_pairs)), dim3(RZ_NT), lds, s, a);
    return hipGetLastError();
}

namespace {
unsigned cs_grid(int n_pairs, int per) { return (unsigned)((n_pairs + RZ_XCD - 1) / RZ_XCD * RZ_XCD * per); }
}  // namespace

Cg64Small cg64_small_extents(const sea_pair* pairs, int n_pairs) {
    Cg64Small e{};
    for (int k = 0; k < n_pairs; ++k) {
        if (!cg64_small(pairs[k])) continue;
        ++e.n;
        if (pairs[k].n[0] <= CS_PACK) ++e.packed;
        e.tiles = std::max(e.tiles, cs_tiles(pairs[k]));
        e.chunks = std::max(e.chunks, cs_chunks(pairs[k]));
        e.blocks = std::max(e.blocks, cs_blocks(pairs[k]));
    }
    return e;
}

hipError_t launch_cg64_small(const ExxArgs& a, const Cg64Small& e, int sweep, hipStream_t s) {
    if (sweep == 1) {
        hipLaunchKernelGGL(k_cg64_small_b, dim3(cs_grid(a.n_pairs, e.blocks)), dim3(CS_NT), 0, s, a, e.blocks);
        return hipGetLastError();
    }
    const dim3 grid(cs_grid(a.n_pairs, e.tiles * e.chunks)), one(64 * RZ_ROWS), two(32 * RZ_ROWS);
    if (e.packed) {
        if (sweep < 0) hipLaunchKernelGGL((k_cg64_small_a<true, 2>), grid, two, 0, s, a, e.tiles, e.chunks);
        else hipLaunchKernelGGL((k_cg64_small_a<false, 2>), grid, two, 0, s, a, e.tiles, e.chunks);
    }
    if (e.packed < e.n) {
        if (sweep < 0) hipLaunchKernelGGL((k_cg64_small_a<true, 1>), grid, one, 0, s, a, e.tiles, e.chunks);
        else hipLaunchKernelGGL((k_cg64_small_a<false, 1>), grid, one, 0, s, a, e.tiles, e.chunks);
    }
    return hipGetLastError();
}

hipError_t launch_residual_list(const ExxArgs& a, const int* list, const int* count, bool write, int n_cu,
                                hipStream_t s) {
    if (a.n_pairs <= 0) return hipSuccess;
    const int lds = (int)residual_zm_lds_bytes();
    const void* fn = write ? (const void*)k_residual_list<true> : (const void*)k_residual_list<false>;
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    const long items = (long)a.n_pairs * RZ_TILES;
    const dim3 grid((unsigned)(items < n_cu ? items : n_cu));   // one workgroup of 1024 threads per CU
    if (write) hipLaunchKernelGGL(k_residual_list<true>, grid, dim3(RZ_NT), lds, s, a, list, count);
    else hipLaunchKernelGGL(k_residual_list<false>, grid, dim3(RZ_NT), lds, s, a, list, count);
    return hipGetLastError();
}

hipError_t launch_refine_flags(const ExxArgs& a, int* lists, int* counts, int it, bool last, hipStream_t s) {
    if (a.n_pairs <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_refine_flags, dim3((a.n_pairs + 63) / 64), dim3(64), 0, s, a, lists, counts, it, last ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_cg64_exit(const ExxArgs& a, hipStream_t s) {
    if (a.n_pairs <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_cg64_exit, dim3((a.n_pairs + 63) / 64), dim3(64), 0, s, a);
    return hipGetLastError();
}

__global__ void k_fill_nan(double* __restrict__ p, size_t n) {
    const double q = __builtin_nan("");
    for (size_t k = blockIdx.x * (size_t)256 + threadIdx.x; k < n; k += (size_t)gridDim.x * 256) p[k] = q;
}

hipError_t launch_fill_nan(double* p, size_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    const unsigned nb = (unsigned)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
    hipLaunchKernelGGL(k_fill_nan, dim3(nb), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_fill_int(int* p, size_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    const unsigned nb = (unsigned)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
    hipLaunchKernelGGL(k_fill_int, dim3(nb), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_start_residual(const ExxArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(k_start_residual, dim3(a.n_pairs), dim3(FIN_BS), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_cg_finish(const ExxArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(k_cg_finish, dim3(a.n_pairs), dim3(FIN_BS), 0, s, a);
    return hipGetLastError();
}

// Compiled z-march variants (FP32 state); the autotuner picks one per
// workload.  nt: workgroup size (rows of the 64 x 64 plane per thread =
// 4096 / nt; smaller workgroups need more queue registers than the 128 a
// lane may hold at this size and spill in the plane loop); pf: prefetch c
// and r of the output plane before the barrier; d: planes of p in flight
// ahead of the register queue; buf: state arrays through buffer
// instructions (32-bit offsets) instead of 64-bit global addresses; xc:
// paired iterate updates (c read and written every second iteration).
namespace {
using CgKernel = void (*)(ExxArgs);
struct CgVariant {
    const char* name;
    CgKernel fn;
    int nt;
};
const CgVariant kCgVariants[] = {
    {"nt1024-pf-d1", k_cg_zm<float, 1024, 4, true, 1, false, false>, 1024},
    {"nt1024-pf-d2", k_cg_zm<float, 1024, 4, true, 2, false, false>, 1024},
    {"nt1024-d1", k_cg_zm<float, 1024, 4, false, 1, false, false>, 1024},
    {"nt1024-d2", k_cg_zm<float, 1024, 4, false, 2, false, false>, 1024},
    {"buf-pf-d1", k_cg_zm<float, 1024, 4, true, 1, true, false>, 1024},
    {"buf-pf-d2", k_cg_zm<float, 1024, 4, true, 2, true, false>, 1024},
    {"buf-d2", k_cg_zm<float, 1024, 4, false, 2, true, false>, 1024},
    {"buf-pf-d1-xc", k_cg_zm<float, 1024, 4, true, 1, true, true>, 1024},
    {"buf-pf-d2-xc", k_cg_zm<float, 1024, 4, true, 2, true, true>, 1024},
    {"nt1024-pf-d1-xc", k_cg_zm<float, 1024, 4, true, 1, false, true>, 1024},
};
constexpr int kNumCgVariants = sizeof(kCgVariants) / sizeof(kCgVariants[0]);
}  // namespace

int cg_variant_count() { return kNumCgVariants; }

const char* cg_variant_name(int v) { return (v >= 0 && v < kNumCgVariants) ? kCgVariants[v].name : nullptr; }

hipError_t launch_cg_zm(const ExxArgs& a, int variant, hipStream_t s) {
    if (variant < 0 || variant >= kNumCgVariants) return hipErrorInvalidValue;
    const CgVariant& v = kCgVariants[variant];
    const int lds = (int)cg_zm_lds_bytes(1);
    hipError_t e = hipFuncSetAttribute((const void*)v.fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(v.fn, dim3(a.n_slots), dim3(v.nt), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_cg_team(const ExxArgs& a, int n_eligible, char* ctl, int n_cu, hipStream_t s) {
    const int lds = (int)cg_team_lds_bytes();
    const int teams = std::min(std::min(cg_teams(n_cu), n_eligible), a.n_slots);
    hipError_t e = hipFuncSetAttribute((const void*)k_cg_team, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    int dev = 0, khz = 0;   // of the wall clock
    if (e == hipSuccess) e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev);
    if (e != hipSuccess) return e;
    const int n_ctl = (int)((teams * CG_TEAM_CTL + CG_TEAM_TAIL) / sizeof(int));
    hipLaunchKernelGGL(k_team_start, dim3(64), dim3(256), 0, s, a, (int*)ctl, n_ctl);
    hipLaunchKernelGGL(k_cg_team, dim3((teams + RZ_XCD - 1) / RZ_XCD * RZ_XCD * TM_G), dim3(TM_NT), lds, s, a, ctl,
                       teams, (long long)khz * TM_JOIN_MS);
    return hipGetLastError();
}
