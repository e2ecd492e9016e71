// SCDM column selection (Sec. II.A, Eq. 1): the pivots of a column-pivoted QR
// of Phi^T (n_occ x Ng), in FP64.
//
// Pivot k is the column of Phi^T whose part orthogonal to the columns already
// chosen is longest.  With q_0..q_{k-1} the orthonormal directions of the
// chosen columns, that squared length is nrm_j = |a_j|^2 - sum_l (q_l . a_j)^2.
// Keeping every nrm_j current would read all of Phi^T once per pivot; instead
// pivots are chosen in rounds:
//
//   * at the start of a round every nrm_j is exact; its largest column is the
//     next pivot (no question of staleness);
//   * the columns whose nrm_j lies within a few octaves of that maximum (at
//     most SC_TMAX of them, picked by a histogram of the norms' bit patterns)
//     become candidates: their n_occ-vectors are copied out and their norms
//     are kept current pivot by pivot;
//   * a later pivot of the round is the best candidate as long as its norm
//     strictly exceeds tau, the largest round-start norm of any
//     non-candidate (norms only shrink, so no outside column can beat it);
//     otherwise the round ends, all nrm_j take the round's q's in one pass
//     over Phi^T, and the next round starts.
//
// The result is the greedy choice itself (up to rounding), with one pass
// over Phi^T per round instead of per pivot.  The new direction q_k is the
// pivot column orthogonalized against q_0..q_{k-1} by classical Gram-Schmidt
// applied twice: against the directions of earlier rounds for all candidates
// at once when the round starts (matrix products), against those of the round
// when the pivot is taken.
#include "k_ace.h"
#include "k_scdm.h"

namespace {

constexpr int SC_BS = 256;       // block of the grid-wide kernels
constexpr int SC_PICK = 1024;    // block of the pick kernel
constexpr int SC_NB = 4096;      // histogram bins: 64 per octave of nrm_j / max

struct __align__(16) ScdmState {
    int k;              // pivots chosen so far
    int k0;             // first pivot of the current round
    int stop;           // the current round has ended
    int fail;           // 1-based step whose residual vanished (rank), 0 = none
    int ncand;          // candidates of the current round
    int bstar;          // last histogram bin taken into the candidate set (-1: none)
    int gslot;          // and its place among the candidates
    long long gidx;     // column of the largest nrm_j at the round start
    double gmax;        // that nrm_j
    unsigned long long tau_bits;   // largest nrm_j outside the candidates (bits)
    double nrm0;        // largest initial column norm^2
};

__device__ __forceinline__ int bin_of(double v, double gmax) {
    // nonnegative doubles order like their bit patterns; 2^46 in the pattern
    // is 1/64 of an octave
    const unsigned long long d =
        (unsigned long long)__double_as_longlong(gmax) - (unsigned long long)__double_as_longlong(v);
    const unsigned long long b = d >> 46;
    return b >= (unsigned long long)SC_NB ? SC_NB - 1 : (int)b;
}

// (value, index) maximum with the smaller index on equal values
__device__ __forceinline__ bool better(double v, long long j, double bv, long long bj) {
    return v > bv || (v == bv && j < bj);
}

__device__ __forceinline__ void wave_argmax(double& v, long long& j) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const double ov = __shfl_down(v, off, 64);
        const long long oj = __shfl_down(j, off, 64);
        if (better(ov, oj, v, j)) {
            v = ov;
            j = oj;
        }
    }
}

template <int BS>
__device__ void block_argmax(double& v, long long& j, double* sv, long long* sj) {
    wave_argmax(v, j);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) {
        sv[w] = v;
        sj[w] = j;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int t = 1; t < BS / 64; ++t)
            if (better(sv[t], sj[t], v, j)) {
                v = sv[t];
                j = sj[t];
            }
    }
}

template <int BS>
__device__ double block_sum(double v, double* red) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    __syncthreads();
    if (lane == 0) red[w] = v;
    __syncthreads();
    double t = 0.0;
    for (int u = 0; u < BS / 64; ++u) t += red[u];
    return t;   // every thread
}

template <typename T>
__device__ __forceinline__ double ld(const T* p, size_t o) {
    return (double)p[o];
}

// nrm_j = |a_j|^2.  Per block: the largest nrm_j and its column.
template <typename T>
__global__ __launch_bounds__(SC_BS) void k_scdm_norms(const T* __restrict__ phi, long Ng, int n,
                                                     double* __restrict__ nrm, double* __restrict__ pv,
                                                     long long* __restrict__ pj) {
    __shared__ double sv[SC_BS / 64];
    __shared__ long long sj[SC_BS / 64];
    const long j = (long)blockIdx.x * SC_BS + threadIdx.x;
    const bool live = j < Ng;
    const long jj = live ? j : 0;
    double v = 0.0;
    int i = 0;
    for (; i + 8 <= n; i += 8) {
        double a[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) a[u] = ld(phi, (size_t)(i + u) * Ng + jj);
#pragma unroll
        for (int u = 0; u < 8; ++u) v += a[u] * a[u];
    }
    for (; i < n; ++i) {
        const double a = ld(phi, (size_t)i * Ng + jj);
        v += a * a;
    }
    if (live) nrm[j] = v;
    else v = -1.0;
    long long bj = live ? j : (long long)Ng;
    block_argmax<SC_BS>(v, bj, sv, sj);
    if (threadIdx.x == 0) {
        pv[blockIdx.x] = v;
        pj[blockIdx.x] = bj;
    }
}

// nrm_j -= sum_{l<b} (q_l . a_j)^2 for the b <= 32 directions Qr (rows of n
// doubles); chosen pivots (nrm_j < 0) stay negative.  Per block: the largest
// nrm_j and its column.
//
// One read of Phi^T is the floor (64 molecules: 3.5 GB); with the 32 products
// of a value on the vector ALUs their LDS broadcasts took longer (1.02 ms; now
// 0.69 ms, 5.1 TB/s).  On the FP64 matrix cores a wavefront forms 32 directions
// x 32 columns: the directions from LDS (a chunk of UP_IC orbitals, rows 65
// 16-byte units apart), the columns straight from memory, a pair of columns to
// a lane, the next 32 orbitals' loads in flight over this 32's products.  In
// lane group g = lane / 16 step s of an 8-orbital block takes orbital 2 g + s
// on both sides.
typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int UP_NT = 512, UP_IC = 128, UP_PITCH = UP_IC + 2;
static_assert(UP_NT / 64 * 32 == SC_BS, "columns of a block");
template <typename T>
__global__ __launch_bounds__(UP_NT) void k_scdm_update(const T* __restrict__ phi, long Ng, int n,
                                                      const double* __restrict__ Qr, int b,
                                                      double* __restrict__ nrm, double* __restrict__ pv,
                                                      long long* __restrict__ pj) {
    __shared__ __attribute__((aligned(16))) double qs[SC_RB][UP_PITCH];
    __shared__ double sv[UP_NT / 64];
    __shared__ long long sj[UP_NT / 64];
    struct Pair {
        T v[2];
    };
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
    const long jc = (long)blockIdx.x * SC_BS + (threadIdx.x >> 6) * 32 + 2 * r;   // this lane's pair of columns
    const bool whole = (long)(blockIdx.x + 1) * SC_BS <= Ng;
    const long ja = min(jc, Ng - 1), jb = min(jc + 1, Ng - 1);
    auto load = [&](int i) -> Pair {   // past the last orbital: that one again (its direction is zero there)
        const T* row = phi + (size_t)min(i, n - 1) * Ng;
        Pair c;
        if (whole) __builtin_memcpy(&c, row + jc, sizeof(c));
        else c = Pair{{row[ja], row[jb]}};
        return c;
    };
    f64x4 acc[2][2];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q) acc[p][q] = f64x4{0, 0, 0, 0};
    constexpr int G = 4;   // 8-orbital blocks loaded together
    Pair nxt[2 * G];
    auto load_group = [&](int i) {
#pragma unroll
        for (int h = 0; h < G; ++h)
#pragma unroll
            for (int s = 0; s < 2; ++s) nxt[2 * h + s] = load(i + 8 * h + 2 * g + s);
    };
    load_group(0);
    for (int i0 = 0; i0 < n; i0 += UP_IC) {
        const int ic = min(UP_IC, n - i0);
        __syncthreads();
        for (int t = threadIdx.x; t < SC_RB * UP_IC; t += UP_NT) {
            const int l = t / UP_IC, ii = t % UP_IC;
            qs[l][ii] = (l < b && ii < ic) ? Qr[(size_t)l * n + i0 + ii] : 0.0;
        }
        __syncthreads();
        for (int ii = 0; ii < ic; ii += 8 * G) {
            Pair c[2 * G];
#pragma unroll
            for (int u = 0; u < 2 * G; ++u) c[u] = nxt[u];
            if (i0 + ii + 8 * G < n) load_group(i0 + ii + 8 * G);
#pragma unroll
            for (int h = 0; h < G; ++h) {
                f64x2 a[2];
#pragma unroll
                for (int p = 0; p < 2; ++p)
                    a[p] = *reinterpret_cast<const f64x2*>(&qs[16 * p + r][ii + 8 * h + 2 * g]);
#pragma unroll
                for (int s = 0; s < 2; ++s)
#pragma unroll
                    for (int p = 0; p < 2; ++p)
#pragma unroll
                        for (int q = 0; q < 2; ++q)
                            acc[p][q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[p][s], (double)c[2 * h + s].v[q],
                                                                            acc[p][q], 0, 0, 0);
            }
        }
    }
    // a result column's 32 directions lie in the four lane groups
    double d[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        d[q] = 0.0;
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int u = 0; u < 4; ++u) d[q] += acc[p][q][u] * acc[p][q][u];
        d[q] += __shfl_xor(d[q], 16, 64);
        d[q] += __shfl_xor(d[q], 32, 64);
    }
    const long j = jc + g;   // lane groups 0 and 1 finish the two columns
    const bool live = g < 2 && j < Ng;
    double v = -1.0;
    if (live) {
        v = nrm[j];
        if (v >= 0.0) {
            v -= g == 0 ? d[0] : d[1];
            if (!(v >= 0.0)) v = -0.5;   // numerically inside the span
        }
        nrm[j] = v;
    }
    long long bj = live ? j : (long long)Ng;
    block_argmax<UP_NT>(v, bj, sv, sj);
    if (threadIdx.x == 0) {
        pv[blockIdx.x] = v;
        pj[blockIdx.x] = bj;
    }
}

// Round start: the largest nrm_j over the update partials; counters cleared.
__global__ __launch_bounds__(SC_PICK) void k_scdm_round_start(const double* __restrict__ pv,
                                                            const long long* __restrict__ pj, int np,
                                                            ScdmState* __restrict__ st,
                                                            unsigned* __restrict__ hist, int first) {
    __shared__ double sv[SC_PICK / 64];
    __shared__ long long sj[SC_PICK / 64];
    double v = -2.0;
    long long j = 0x7fffffffffffffffll;
    for (int t = threadIdx.x; t < np; t += SC_PICK)
        if (better(pv[t], pj[t], v, j)) {
            v = pv[t];
            j = pj[t];
        }
    block_argmax<SC_PICK>(v, j, sv, sj);
    for (int t = threadIdx.x; t < SC_NB; t += SC_PICK) hist[t] = 0u;
    if (threadIdx.x == 0) {
        if (first) {
            st->k = 0;
            st->fail = 0;
            st->nrm0 = v;
        }
        st->k0 = st->k;
        st->gmax = v;
        st->gidx = j;
        st->ncand = 0;
        st->tau_bits = 0ull;
        // no positive norm left: the remaining columns lie in the span
        st->stop = (v > 1e-26 * st->nrm0) ? 0 : 1;
        if (st->stop && !st->fail) st->fail = st->k + 1;
    }
}

// Histogram of the positive norms by bin_of.
__global__ __launch_bounds__(SC_BS) void k_scdm_hist(const double* __restrict__ nrm, long Ng,
                                                   const ScdmState* __restrict__ st, unsigned* __restrict__ hist) {
    __shared__ unsigned h[SC_NB];
    for (int t = threadIdx.x; t < SC_NB; t += SC_BS) h[t] = 0u;
    __syncthreads();
    const double gmax = st->gmax;
    const bool run = !st->stop;
    if (run)
        for (long j = (long)blockIdx.x * SC_BS + threadIdx.x; j < Ng; j += (long)gridDim.x * SC_BS) {
            const double v = nrm[j];
            if (v > 0.0) atomicAdd(&h[bin_of(v, gmax)], 1u);
        }
    __syncthreads();
    if (run)
        for (int t = threadIdx.x; t < SC_NB; t += SC_BS)
            if (h[t]) atomicAdd(&hist[t], h[t]);
}

// bstar = the last bin whose cumulative count stays within SC_TMAX.
__global__ __launch_bounds__(SC_PICK) void k_scdm_select(const unsigned* __restrict__ hist,
                                                       ScdmState* __restrict__ st) {
    constexpr int PER = SC_NB / SC_PICK;
    __shared__ unsigned scan[SC_PICK];
    __shared__ int best[SC_PICK / 64];
    unsigned loc[PER];
    unsigned s = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        loc[u] = hist[threadIdx.x * PER + u];
        s += loc[u];
    }
    scan[threadIdx.x] = s;
    __syncthreads();
    for (int off = 1; off < SC_PICK; off <<= 1) {
        const unsigned add = threadIdx.x >= (unsigned)off ? scan[threadIdx.x - off] : 0u;
        __syncthreads();
        scan[threadIdx.x] += add;
        __syncthreads();
    }
    unsigned cum = scan[threadIdx.x] - s;   // exclusive prefix
    int b = -1;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        cum += loc[u];
        if (cum <= (unsigned)SC_TMAX) b = threadIdx.x * PER + u;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) b = max(b, __shfl_down(b, off, 64));
    if ((threadIdx.x & 63) == 0) best[threadIdx.x >> 6] = b;
    __syncthreads();
    if (threadIdx.x == 0) {
        int m = -1;
        for (int w = 0; w < SC_PICK / 64; ++w) m = max(m, best[w]);
        if (!st->stop) st->bstar = m;
    }
}

// Candidates: positive norms in bins <= bstar, plus the round's first pivot.
// tau = the largest positive norm of the rest.
__global__ __launch_bounds__(SC_BS) void k_scdm_gather(const double* __restrict__ nrm, long Ng,
                                                     ScdmState* __restrict__ st, int* __restrict__ cidx,
                                                     double* __restrict__ cval) {
    if (st->stop) return;
    const double gmax = st->gmax;
    const int bstar = st->bstar;
    const long long gidx = st->gidx;
    const int lane = threadIdx.x & 63;
    unsigned long long tb = 0ull;
    for (long base = (long)blockIdx.x * SC_BS; base < Ng; base += (long)gridDim.x * SC_BS) {
        const long j = base + threadIdx.x;
        const double v = j < Ng ? nrm[j] : -1.0;
        bool cand = false;
        if (v > 0.0) {
            cand = bin_of(v, gmax) <= bstar || j == gidx;
            if (!cand) tb = max(tb, (unsigned long long)__double_as_longlong(v));
        }
        const unsigned long long m = __ballot(cand);
        if (m) {
            int pos0 = 0;
            if (lane == 0) pos0 = atomicAdd(&st->ncand, __popcll(m));
            pos0 = __shfl(pos0, 0, 64);
            if (cand) {
                const int pos = pos0 + __popcll(m & ((1ull << lane) - 1ull));
                if (pos < SC_TMAX + 1) {
                    cidx[pos] = (int)j;
                    cval[pos] = v;
                    if (j == gidx) st->gslot = pos;
                }
            }
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const unsigned long long o = __shfl_down(tb, off, 64);
        tb = o > tb ? o : tb;
    }
    __shared__ unsigned long long tw[SC_BS / 64];
    if (lane == 0) tw[threadIdx.x >> 6] = tb;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int u = 1; u < SC_BS / 64; ++u) tb = tw[u] > tb ? tw[u] : tb;
        if (tb) atomicMax(&st->tau_bits, tb);
    }
}

// cvec[t][i] = Phi^T(i, cidx[t]) for the candidates.
template <typename T>
__global__ __launch_bounds__(SC_BS) void k_scdm_cand_vec(const T* __restrict__ phi, long Ng, int n,
                                                       const ScdmState* __restrict__ st,
                                                       const int* __restrict__ cidx, double* __restrict__ cvec) {
    if (st->stop) return;
    const int t = blockIdx.y;
    if (t >= min(st->ncand, SC_TMAX + 1)) return;
    const int i = blockIdx.x * SC_BS + threadIdx.x;
    if (i < n) cvec[(size_t)t * n + i] = ld(phi, (size_t)i * Ng + cidx[t]);
}

// a += b
__global__ __launch_bounds__(SC_BS) void k_scdm_add(double* __restrict__ a, const double* __restrict__ b, size_t len) {
    const size_t t = (size_t)blockIdx.x * SC_BS + threadIdx.x;
    if (t < len) a[t] += b[t];
}

// One pivot.  The round's first is the largest exact norm; later ones the best
// candidate if it beats tau, else the round ends.  The pivot's candidate
// vector (orthogonal to the directions before this round) is orthogonalized
// against the round's own (classical Gram-Schmidt, twice) and normalized into
// row k of Q; then the candidates take the new direction, a wavefront per
// candidate, and each block leaves its best remaining one for the next step.
//
// Every block forms the new direction for itself, in the same way: a pivot
// costs one launch and no pass over all of Q through one CU (256 orbitals: 27
// us for the pivot and 8 us for the candidates before; 14 us now).  Block 0
// records it.  What it writes here, other blocks read in a later launch only,
// but for st->stop, which no block needs where another has set it.
struct ScdmBest {   // per block: value, column, candidate slot
    double* v;
    long long* j;
    int* slot;
};
constexpr int SC_STEP = 256;   // blocks of a step
__global__ __launch_bounds__(SC_PICK) void k_scdm_step(int n, int step, ScdmState* __restrict__ st,
                                                     const int* __restrict__ cidx, double* __restrict__ cval,
                                                     const double* __restrict__ cvec, ScdmBest in, ScdmBest out,
                                                     double* __restrict__ Q, int* __restrict__ piv,
                                                     double* __restrict__ rdiag, double* __restrict__ nrm) {
    constexpr int W = SC_PICK / 64;
    __shared__ double r[SC_NMAX];
    __shared__ double d[SC_RB];
    __shared__ double sv[W];
    __shared__ long long sj[W];
    __shared__ int slot_sh, go_sh;
    const bool rec = blockIdx.x == 0 && threadIdx.x == 0;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int k0 = st->k0, k = k0 + step;
    if (k >= n) {
        if (rec) st->stop = 1;
        return;
    }
    // One thread reads st->stop for its block: block 0 of this launch may set it
    // meanwhile, and all of a block have to see the same (a block that sees the old
    // value comes to the same end by itself)
    if (step == 0) {
        if (threadIdx.x == 0) {
            slot_sh = st->gslot;
            go_sh = !st->stop;
        }
    } else {
        double v = -2.0;
        long long j = 0x7fffffffffffffffll;
        int slot = 0;
        if (threadIdx.x < SC_STEP) {
            v = in.v[threadIdx.x];
            j = in.j[threadIdx.x];
            slot = in.slot[threadIdx.x];
        }
        double bv = v;
        long long bj = j;
        block_argmax<SC_PICK>(bv, bj, sv, sj);
        if (threadIdx.x == 0) {
            const double tau = __longlong_as_double((long long)st->tau_bits);
            go_sh = !st->stop && bv > tau && bv > 0.0;
            sj[0] = bj;
            if (!go_sh && rec) st->stop = 1;
        }
        __syncthreads();
        if (threadIdx.x < SC_STEP && j == sj[0]) slot_sh = slot;   // a column is one block's
    }
    __syncthreads();
    if (!go_sh) return;
    const int slot = slot_sh;
    for (int i = threadIdx.x; i < n; i += SC_PICK) r[i] = cvec[(size_t)slot * n + i];
    __syncthreads();
    const double* Q1 = Q + (size_t)k0 * n;
    for (int pass = 0; pass < 2 && step > 0; ++pass) {
        for (int l = w; l < step; l += W) {
            const double* q = Q1 + (size_t)l * n;
            double s = 0.0;
            for (int i = lane; i < n; i += 64) s += q[i] * r[i];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
            if (lane == 0) d[l] = s;
        }
        __syncthreads();
        for (int i = threadIdx.x; i < n; i += SC_PICK) {
            double s = 0.0;
#pragma unroll 8
            for (int l = 0; l < step; ++l) s += d[l] * Q1[(size_t)l * n + i];
            r[i] -= s;
        }
        __syncthreads();
    }
    double ss = 0.0;
    for (int i = threadIdx.x; i < n; i += SC_PICK) ss += r[i] * r[i];
    ss = block_sum<SC_PICK>(ss, sv);
    if (!(ss > 1e-26 * st->nrm0)) {
        if (rec) {
            st->fail = k + 1;
            st->stop = 1;
        }
        return;
    }
    const double rn = sqrt(ss), inv = 1.0 / rn;
    const int c = cidx[slot];
    for (int i = threadIdx.x; i < n; i += SC_PICK) {
        r[i] *= inv;
        if (blockIdx.x == 0) Q[(size_t)k * n + i] = r[i];
    }
    if (rec) {
        piv[k] = c;
        rdiag[k] = rn;
        nrm[c] = -1.0;
        st->k = k + 1;
    }
    __syncthreads();
    const int nc = min(st->ncand, SC_TMAX + 1);
    double bv = -2.0;
    long long bj = 0x7fffffffffffffffll;
    int bs = 0;
    for (int t = blockIdx.x * W + w; t < nc; t += SC_STEP * W) {
        double v = t == slot ? -1.0 : cval[t];   // chosen as a pivot
        const int j = cidx[t];
        if (v >= 0.0) {
            const double* a = cvec + (size_t)t * n;
            double s = 0.0;
            for (int i = lane; i < n; i += 64) s += a[i] * r[i];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
            v -= s * s;
            if (!(v >= 0.0)) v = -0.5;
        }
        if (lane == 0) cval[t] = v;
        if (better(v, j, bv, bj)) {
            bv = v;
            bj = j;
            bs = t;
        }
    }
    const double v0 = bv;
    const long long j0 = bj;
    block_argmax<SC_PICK>(bv, bj, sv, sj);
    if (threadIdx.x == 0) {
        out.v[blockIdx.x] = bv;
        out.j[blockIdx.x] = bj;
        sv[0] = bv;
        sj[0] = bj;
    }
    __syncthreads();
    if (lane == 0 && j0 == sj[0] && v0 == sv[0] && v0 > -2.0) out.slot[blockIdx.x] = bs;
}

// G[a][i] = Phi^T(i, piv[a])
template <typename T>
__global__ __launch_bounds__(SC_BS) void k_scdm_pivot_rows(const T* __restrict__ phi, long Ng, int n,
                                                         const int* __restrict__ piv, double* __restrict__ G) {
    const int a = blockIdx.y;
    const int i = blockIdx.x * SC_BS + threadIdx.x;
    if (i < n) G[(size_t)a * n + i] = ld(phi, (size_t)i * Ng + piv[a]);
}

// Newton-Schulz steps for the polar factor (see scdm_polar_*): one workgroup.
constexpr int NS_BS = 1024;

// Y = G / |G|_F
__global__ __launch_bounds__(NS_BS) void k_ns_scale(const double* __restrict__ G, int n, double* __restrict__ Y) {
    __shared__ double red[NS_BS / 64];
    const long nn = (long)n * n;
    double s = 0.0;
    for (long t = threadIdx.x; t < nn; t += NS_BS) s += G[t] * G[t];
    s = block_sum<NS_BS>(s, red);
    const double inv = 1.0 / sqrt(s);
    for (long t = threadIdx.x; t < nn; t += NS_BS) Y[t] = G[t] * inv;
}

// S <- 1.5 I - 0.5 S, err[block] = the block's part of |S - I|_F^2 of the incoming S
__global__ __launch_bounds__(SC_BS) void k_ns_mid(double* __restrict__ S, int n, double* __restrict__ err) {
    __shared__ double red[SC_BS / 64];
    const long nn = (long)n * n;
    double e = 0.0;
    for (long t = (long)blockIdx.x * SC_BS + threadIdx.x; t < nn; t += (long)SC_NS_ERR * SC_BS) {
        const bool diag = (t / n) == (t % n);
        const double v = S[t];
        const double d = diag ? v - 1.0 : v;
        e += d * d;
        S[t] = (diag ? 1.5 : 0.0) - 0.5 * v;
    }
    e = block_sum<SC_BS>(e, red);
    if (threadIdx.x == 0) err[blockIdx.x] = e;
}

}  // namespace

hipError_t scdm_ns_scale(const double* G, int n, double* Y, hipStream_t s) {
    hipLaunchKernelGGL(k_ns_scale, dim3(1), dim3(NS_BS), 0, s, G, n, Y);
    return hipGetLastError();
}

hipError_t scdm_ns_mid(double* S, int n, double* err, hipStream_t s) {
    hipLaunchKernelGGL(k_ns_mid, dim3(SC_NS_ERR), dim3(SC_BS), 0, s, S, n, err);
    return hipGetLastError();
}

ScdmLayout scdm_layout(long Ng, int n) {
    ScdmLayout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off = (off + bytes + 255) & ~(size_t)255;
        return o;
    };
    const long nub = (Ng + SC_BS - 1) / SC_BS;
    L.n_upd_blocks = nub;
    L.state = take(sizeof(ScdmState));
    L.nrm = take((size_t)Ng * sizeof(double));
    L.upv = take((size_t)nub * sizeof(double));
    L.upj = take((size_t)nub * sizeof(long long));
    L.hist = take(SC_NB * sizeof(unsigned));
    L.cidx = take((SC_TMAX + 1) * sizeof(int));
    L.cval = take((SC_TMAX + 1) * sizeof(double));
    L.cvec = take((size_t)(SC_TMAX + 1) * n * sizeof(double));
    L.cdot = take((size_t)(SC_TMAX + 1) * n * sizeof(double));
    L.cprj = take((size_t)(SC_TMAX + 1) * n * sizeof(double));
    L.dv = take((size_t)2 * SC_STEP * sizeof(double));
    L.dj = take((size_t)2 * SC_STEP * sizeof(long long));
    L.ds = take((size_t)2 * SC_STEP * sizeof(int));
    L.Q = take((size_t)n * n * sizeof(double));
    L.piv = take((size_t)n * sizeof(int));
    L.rdiag = take((size_t)n * sizeof(double));
    L.total = off;
    return L;
}

size_t scdm_state_bytes() { return sizeof(ScdmState); }

hipError_t scdm_init(const void* phi, int f32, long Ng, int n, char* ws, const ScdmLayout& L, hipStream_t s) {
    double* nrm = (double*)(ws + L.nrm);
    double* upv = (double*)(ws + L.upv);
    long long* upj = (long long*)(ws + L.upj);
    const unsigned nb = (unsigned)L.n_upd_blocks;
    if (f32)
        hipLaunchKernelGGL((k_scdm_norms<float>), dim3(nb), dim3(SC_BS), 0, s, (const float*)phi, Ng, n, nrm, upv, upj);
    else
        hipLaunchKernelGGL((k_scdm_norms<double>), dim3(nb), dim3(SC_BS), 0, s, (const double*)phi, Ng, n, nrm, upv,
                           upj);
    return hipGetLastError();
}

hipError_t scdm_update(const void* phi, int f32, long Ng, int n, int k0, int b, char* ws, const ScdmLayout& L,
                       hipStream_t s) {
    double* nrm = (double*)(ws + L.nrm);
    double* upv = (double*)(ws + L.upv);
    long long* upj = (long long*)(ws + L.upj);
    const double* Qr = (const double*)(ws + L.Q) + (size_t)k0 * n;
    const unsigned nb = (unsigned)L.n_upd_blocks;
    if (b < 0 || b > SC_RB) return hipErrorInvalidValue;
    if (f32)
        hipLaunchKernelGGL((k_scdm_update<float>), dim3(nb), dim3(UP_NT), 0, s, (const float*)phi, Ng, n, Qr, b, nrm,
                           upv, upj);
    else
        hipLaunchKernelGGL((k_scdm_update<double>), dim3(nb), dim3(UP_NT), 0, s, (const double*)phi, Ng, n, Qr, b, nrm,
                           upv, upj);
    return hipGetLastError();
}

hipError_t scdm_round(const void* phi, int f32, long Ng, int n, int k0, char* ws, const ScdmLayout& L,
                      hipStream_t s) {
    ScdmState* st = (ScdmState*)(ws + L.state);
    double* nrm = (double*)(ws + L.nrm);
    unsigned* hist = (unsigned*)(ws + L.hist);
    int* cidx = (int*)(ws + L.cidx);
    double* cval = (double*)(ws + L.cval);
    double* cvec = (double*)(ws + L.cvec);
    double* Q = (double*)(ws + L.Q);
    int* piv = (int*)(ws + L.piv);
    double* rdiag = (double*)(ws + L.rdiag);
    hipLaunchKernelGGL(k_scdm_round_start, dim3(1), dim3(SC_PICK), 0, s, (const double*)(ws + L.upv),
                       (const long long*)(ws + L.upj), (int)L.n_upd_blocks, st, hist, k0 == 0);
    const long gb = (Ng + SC_BS - 1) / SC_BS;
    const unsigned g = (unsigned)(gb < 2048 ? gb : 2048);
    hipLaunchKernelGGL(k_scdm_hist, dim3(g), dim3(SC_BS), 0, s, (const double*)nrm, Ng, (const ScdmState*)st, hist);
    hipLaunchKernelGGL(k_scdm_select, dim3(1), dim3(SC_PICK), 0, s, (const unsigned*)hist, st);
    hipLaunchKernelGGL(k_scdm_gather, dim3(g), dim3(SC_BS), 0, s, (const double*)nrm, Ng, st, cidx, cval);
    const dim3 cg((n + SC_BS - 1) / SC_BS, SC_TMAX + 1);
    if (f32)
        hipLaunchKernelGGL((k_scdm_cand_vec<float>), cg, dim3(SC_BS), 0, s, (const float*)phi, Ng, n,
                           (const ScdmState*)st, (const int*)cidx, cvec);
    else
        hipLaunchKernelGGL((k_scdm_cand_vec<double>), cg, dim3(SC_BS), 0, s, (const double*)phi, Ng, n,
                           (const ScdmState*)st, (const int*)cidx, cvec);
    // the candidates' parts orthogonal to the directions so far: a -= Q^T (Q a), twice
    for (int pass = 0; pass < 2 && k0 > 0; ++pass) {
        double* dot = (double*)(ws + L.cdot);
        double* prj = (double*)(ws + L.cprj);   // (also the first product's partials: one slice of it)
        hipError_t e = ace_mm_nt<ACE_F64, double, double>(cvec, Q, SC_TMAX + 1, k0, n, 1.0, prj, dot, s, 1);
        if (e == hipSuccess)
            e = ace_mm_nn<ACE_F64, double, double>(dot, k0, 1, Q, SC_TMAX + 1, k0, n, -1.0, prj, s);
        if (e != hipSuccess) return e;
        const size_t len = (size_t)(SC_TMAX + 1) * n;
        hipLaunchKernelGGL(k_scdm_add, dim3((unsigned)((len + SC_BS - 1) / SC_BS)), dim3(SC_BS), 0, s, cvec,
                           (const double*)prj, len);
    }
    ScdmBest best[2];
    for (int q = 0; q < 2; ++q)
        best[q] = ScdmBest{(double*)(ws + L.dv) + q * SC_STEP, (long long*)(ws + L.dj) + q * SC_STEP,
                           (int*)(ws + L.ds) + q * SC_STEP};
    for (int step = 0; step < SC_RB; ++step)
        hipLaunchKernelGGL(k_scdm_step, dim3(SC_STEP), dim3(SC_PICK), 0, s, n, step, st, (const int*)cidx, cval,
                           (const double*)cvec, best[(step + 1) & 1], best[step & 1], Q, piv, rdiag, nrm);
    return hipGetLastError();
}

hipError_t scdm_pivot_rows(const void* phi, int f32, long Ng, int n, const int* piv, double* G, hipStream_t s) {
    const dim3 g((n + SC_BS - 1) / SC_BS, n);
    if (f32)
        hipLaunchKernelGGL((k_scdm_pivot_rows<float>), g, dim3(SC_BS), 0, s, (const float*)phi, Ng, n, piv, G);
    else
        hipLaunchKernelGGL((k_scdm_pivot_rows<double>), g, dim3(SC_BS), 0, s, (const double*)phi, Ng, n, piv, G);
    return hipGetLastError();
}

// Host view of the state fields the round loop needs.
hipError_t scdm_read_state(const char* ws, const ScdmLayout& L, int* k, int* fail, hipStream_t s) {
    ScdmState h;
    hipError_t e = hipMemcpyAsync(&h, ws + L.state, sizeof(h), hipMemcpyDeviceToHost, s);
    if (e != hipSuccess) return e;
    e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    *k = h.k;
    *fail = h.fail;
    return hipSuccess;
}
