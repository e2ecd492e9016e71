// Owner-computes scatter of the exx action for gfx950 (Eq. 13-14): W_o(g)
// is the sum over the pairs of orbital o, in pair order, of v_ij(g) times
// the other orbital, with v_ij the pair potential inside the pair's domain
// and its multipole expansion (Eq. 10) outside it; no atomics, so W is
// bitwise reproducible.  On the way it forms the pair energies of Eq. 8:
// the workgroup of orbital i = min(i, j) multiplies each contribution
// v_ij phi_j at a domain point by phi_i there and sums them per (pair,
// tile), so e_ij = dV sum rho_ij v_ij needs one more orbital load per tile
// point instead of a pass of its own over every pair domain.
#include <algorithm>
#include <type_traits>

#include "exx_device.h"
#include "sea_internal.h"

namespace {

// owner-computes scatter: W_o(g) = sum over o's pairs (pair order) of
//    v_pair(g - lo) phi_other(g), every domain duplicate of g included.

constexpr int SC_BS = 256;
constexpr int SC_MAXE = 128;   // list entries per chunk
constexpr int SC_NM = 84;      // monomial coefficients of a pair's multipole sum

// (orbital, tile) of this workgroup, by the order of the workgroups (the
// schedule; the autotuner's variants).  0: the tiles of one orbital in
// turn; 1: the orbitals of one tile in turn; 2: as 1 within each XCD
// (workgroup k runs on XCD k mod 8), which owns every eighth tile, so that
// the owners of a tile share that XCD's L2 for the partner orbitals and pair
// potentials they read there.  Measured on the 64-molecule cell: 4.80, 6.22
// and 4.56 ms per launch; 0 and 2 are compiled.
constexpr int SC_XCD = 8;

template <int ORDER>
__device__ __forceinline__ void sc_block(int n_tiles, int n_occ, int& o, int& t) {
    const int k = blockIdx.x;
    if constexpr (ORDER == 0) {
        t = k % n_tiles;
        o = k / n_tiles;
    } else if constexpr (ORDER == 1) {
        o = k % n_occ;
        t = k / n_occ;
    } else {
        const int x = k % SC_XCD, m = k / SC_XCD;
        o = m % n_occ;
        t = (m / n_occ) * SC_XCD + x;
    }
}
__host__ inline long sc_grid(int order, int n_tiles, int n_occ) {
    return order == 2 ? (long)((n_tiles + SC_XCD - 1) / SC_XCD) * SC_XCD * n_occ : (long)n_tiles * n_occ;
}

__device__ __forceinline__ bool axis_hits(int t0, int T, int lo, int n, int N) {
    if (n >= N) return true;
    const int s = wrap_idx(t0 - lo, N);
    return s < n || s + T > N;
}

// W gathered per (orbital, tile): every pair of the orbital whose W box
// touches the tile adds v * phi_partner at the tile's points, in pair order.
// The box is the pair's W box for this orbital's side (lo[3], n[3] in the
// pair domain's unwrapped frame); inside the pair's domain v is the solution,
// outside it the multipole potential of the pair (Eq. 10).
// The cell's record comes by value, so its pointers are kernel arguments:
// uniform, and known to the compiler to address global memory.
// BOX: what the cell's W boxes ask for.  0: every W box is its pair's domain
// and holds a grid point once; 1: some is wider than the cell (points met once
// per image of the cell); 2: some reaches beyond its pair's domain as well
// (multipole values there).  Each kernel carries no more than its own paths
// (nor their registers).  Images are passes of the same column loads: point by
// point with the images innermost, as the kernel did before, the 8-molecule
// cell (63-point domains in a 60-point cell) took 1.28 ms and a domain sum of
// 0.35 ms for its pair energies; now 0.56 ms together.  Multipole values come
// from the column's line coefficients, folded once for its SC_TZ points and
// evaluated side by side (84 terms a point, one point after another, before:
// the epsilon boxes of the 64-molecule cell 2.54 ms, now 2.07 ms with the
// launch that finds their tiles).
// PT: the orbitals' precision.
struct ScShared {
    int list[SC_MAXE];
    // per listed entry: pair, partner orbital, W box (lo, n), domain (lo, n),
    // energy slot (-1: this workgroup adds nothing to e_ij)
    int meta[SC_MAXE][15];
    // per entry of the orbital's list: the wavefronts' parts of its energy
    // partial, its slot and pair (the list has at most SC_EP_MAXE entries
    // when a.epart is set)
    double ep_w[SC_EP_MAXE][SC_BS / 64];
    int ep_slot_of[SC_EP_MAXE], ep_pid_of[SC_EP_MAXE];
    // this orbital at the tile's points (energy partials)
    double po_s[SC_TZ][SC_BS];
    int cnt, n_e;
};
// BOX 2 alone: the multipole coefficients of SC_CFN entries at a time (read
// from memory where they are used, they held each entry up by a chain of
// scalar loads)
constexpr int SC_CFN = 12;
struct ScCoeffs {
    double cf[SC_CFN][SC_NM];
};
struct ScNone {};

__device__ __forceinline__ int sc_tiles(const DevCell& C) {
    return ((C.N[0] + SC_TX - 1) / SC_TX) * ((C.N[1] + SC_TY - 1) / SC_TY) * ((C.N[2] + SC_TZ - 1) / SC_TZ);
}

template <int BOX, typename PT>
__device__ __forceinline__ void scatter_tile(const ExxArgs& a, const DevCell& C, const int* __restrict__ off_all,
                                             const ScEntry* __restrict__ ent, int o, int t, ScShared& S,
                                             typename std::conditional<BOX == 2, ScCoeffs, ScNone>::type& CF) {
    auto& list = S.list;
    auto& meta = S.meta;
    auto& ep_w = S.ep_w;
    auto& ep_slot_of = S.ep_slot_of;
    auto& ep_pid_of = S.ep_pid_of;
    auto& po_s = S.po_s;
    int &cnt = S.cnt, &n_e = S.n_e;
    const int* off = off_all + C.csr_base;
    double* __restrict__ W = C.W;
    const int tiles_x = (C.N[0] + SC_TX - 1) / SC_TX;
    const int tiles_y = (C.N[1] + SC_TY - 1) / SC_TY;
    const int tx0 = (t % tiles_x) * SC_TX;
    const int ty0 = ((t / tiles_x) % tiles_y) * SC_TY;
    const int tz0 = (t / (tiles_x * tiles_y)) * SC_TZ;
    const int tiles[3] = {tiles_x, tiles_y, (C.N[2] + SC_TZ - 1) / SC_TZ};
    const int tc[3] = {t % tiles_x, (t / tiles_x) % tiles_y, t / (tiles_x * tiles_y)};
    const int e0 = off[o], e1 = off[o + 1];
    // energy partials only for lists that fit the per-entry LDS arrays (the
    // host leaves a.epart unset otherwise)
    const bool take_e = a.epart && e1 - e0 <= SC_EP_MAXE;
    if (threadIdx.x == 0) cnt = 0;
    if (take_e)
        for (int q = threadIdx.x; q < e1 - e0; q += SC_BS) ep_slot_of[q] = -1;
    __syncthreads();
    double acc[SC_TX * SC_TY * SC_TZ / SC_BS];
#pragma unroll
    for (int k = 0; k < SC_TX * SC_TY * SC_TZ / SC_BS; ++k) acc[k] = 0.0;
    for (int c0 = e0; c0 < e1; c0 += SC_MAXE) {
        const int c1 = min(e1, c0 + SC_MAXE);
        // ordered compaction by wavefront 0: lane k tests entry c0 + 64 s + k,
        // hits keep their order through the ballot's prefix counts
        if (threadIdx.x < 64) {
            const int lane = threadIdx.x;
            int m = 0, ne = 0;
            for (int b0 = c0; b0 < c1; b0 += 64) {
                const int e = b0 + lane;
                bool hit = false;
                int slot = -1;
                ScEntry R{};
                if (e < c1) {
                    R = ent[e];
                    hit = axis_hits(tx0, SC_TX, R.D[0], R.D[3], C.N[0]) && axis_hits(ty0, SC_TY, R.D[1], R.D[4], C.N[1]) &&
                          axis_hits(tz0, SC_TZ, R.D[2], R.D[5], C.N[2]);
                    // the pair's energy partial of this tile: i side, a W box
                    // that holds the domain, a tile the domain meets
                    if (hit && R.iside && take_e && ep_takes(R.lo, R.n, R.D) &&
                        axis_hits(tx0, SC_TX, R.lo[0], R.n[0], C.N[0]) &&
                        axis_hits(ty0, SC_TY, R.lo[1], R.n[1], C.N[1]) &&
                        axis_hits(tz0, SC_TZ, R.lo[2], R.n[2], C.N[2]))
                        slot = ep_slot(R.lo, R.n, C.N, tc, tiles);
                }
                const unsigned long long mask = __ballot(hit);
                const unsigned long long below = lane ? (mask << (64 - lane)) : 0ull;
                if (hit) {
                    const int q = m + __popcll(below);
                    list[q] = e;
                    meta[q][0] = R.pid;
                    meta[q][1] = R.other;
#pragma unroll
                    for (int d = 0; d < 6; ++d) meta[q][2 + d] = R.D[d];
#pragma unroll
                    for (int d = 0; d < 3; ++d) {
                        meta[q][8 + d] = R.lo[d];
                        meta[q][11 + d] = R.n[d];
                    }
                    meta[q][14] = slot;
                    if (slot >= 0) {
                        ep_slot_of[e - e0] = slot;
                        ep_pid_of[e - e0] = R.pid;
                    }
                }
                m += __popcll(mask);
                ne += __popcll(__ballot(slot >= 0));
            }
            if (lane == 0) {
                cnt = m;
                n_e = ne;
            }
        }
        __syncthreads();
        const int m = cnt;
        // this thread's column (gx, gy) and planes tz0 + k, found in each box
        // from per-pair offsets by compare-and-subtract instead of modulo
        static_assert(SC_TX * SC_TY == SC_BS, "one (x, y) column per thread");
        const int cx = threadIdx.x % SC_TX, cy = threadIdx.x / SC_TX;
        const int gx = tx0 + cx, gy = ty0 + cy;
        const bool colin = gx < C.N[0] && gy < C.N[1];
        {
            const PT* __restrict__ ph = (const PT*)C.phi;
            // this orbital at the column's points (in LDS), for the energy partials
            if (n_e) {
                const size_t gcol = (size_t)o * C.Ng + (size_t)gy * C.N[0] + gx;
                const size_t gplane = (size_t)C.N[0] * C.N[1];
#pragma unroll
                for (int k = 0; k < SC_TZ; ++k)
                    po_s[k][threadIdx.x] = colin ? (double)ph[gcol + (size_t)min(tz0 + k, C.N[2] - 1) * gplane] : 0.0;
            }
            for (int q = 0; q < m; ++q) {
                if constexpr (BOX == 2) {
                    if (q % SC_CFN == 0) {   // uniform
                        __syncthreads();
                        for (int i = threadIdx.x; i < SC_CFN * SC_NM; i += SC_BS) {
                            const int qe = q + i / SC_NM;
                            if (qe < m) CF.cf[i / SC_NM][i % SC_NM] = a.mpoly[(size_t)meta[qe][0] * SC_NM + i % SC_NM];
                        }
                        __syncthreads();
                    }
                }
                // the entry's values are the same in every lane: read them into
                // scalar registers, so the per-plane addresses below are a scalar
                // base plus one per-lane offset shared by all planes
                int e[14];
#pragma unroll
                for (int d = 0; d < 14; ++d) e[d] = __builtin_amdgcn_readfirstlane(meta[q][d]);
                const int eslot = __builtin_amdgcn_readfirstlane(meta[q][14]);
                const int pid = e[0], oth = e[1];
                const int* D = &e[2];
                const int* plo = &e[8];
                const int* pn = &e[11];
                // box coordinates of the tile corner (uniform), then of this column:
                // gx < N keeps lx below 2N, so one subtraction wraps it
                int lx = wrap_idx(tx0 - D[0], C.N[0]) + cx;
                int ly = wrap_idx(ty0 - D[1], C.N[1]) + cy;
                lx -= (lx >= C.N[0]) ? C.N[0] : 0;
                ly -= (ly >= C.N[1]) ? C.N[1] : 0;
                double ep = 0.0;
                // a box wider than the cell meets a grid point once per image of
                // the cell that it reaches into (one image otherwise)
                const int lx0 = lx, ly0 = ly;
                const int imx = BOX ? (D[3] + C.N[0] - 1) / C.N[0] : 1, imy = BOX ? (D[4] + C.N[1] - 1) / C.N[1] : 1,
                          imz = BOX ? (D[5] + C.N[2] - 1) / C.N[2] : 1;
                for (int im = 0; im < imx * imy * imz; ++im) {
                    if (BOX) {
                        lx = lx0 + im % imx * C.N[0];
                        ly = ly0 + im / imx % imy * C.N[1];
                    }
                    if (!(colin && lx < D[3] && ly < D[4])) continue;
                    const int lzi = BOX ? im / (imx * imy) * C.N[2] : 0;
                    const int lz0 = wrap_idx(tz0 - D[2], C.N[2]);
                    if (BOX && (lz0 + SC_TZ > C.N[2] ? 0 : lz0) + lzi >= D[5]) continue;   // no plane of this image
                    const int sx = D[0] + lx - plo[0], sy = D[1] + ly - plo[1];
                    const bool in_xy = sx >= 0 && sx < pn[0] && sy >= 0 && sy < pn[1];
                    const double* v = a.v + (size_t)pid * a.stride;
                    const unsigned vcol = in_xy ? (unsigned)(sy * pn[0] + sx) : 0u;
                    const size_t vplane = (size_t)pn[0] * pn[1], gplane = (size_t)C.N[0] * C.N[1];
                    const unsigned gcol = (unsigned)(gy * C.N[0] + gx);
                    const size_t phoff = (size_t)oth * C.Ng;
                    // all loads of the column's points first (independent, in flight
                    // together), then the multipole values of points outside the domain
                    double vv[SC_TZ];
                    PT pv[SC_TZ];   // converted at the product: no wait inside the load sequence
                    bool ins[SC_TZ];
                    unsigned me = 0;   // points outside the domain (BOX 2)
#pragma unroll
                    for (int k = 0; k < SC_TZ; ++k) {
                        const int gz = tz0 + k;
                        int lz = lz0 + k;
                        lz -= (lz >= C.N[2]) ? C.N[2] : 0;
                        lz += lzi;
                        const bool valid = gz < C.N[2] && lz < D[5];
                        const int sz = D[2] + lz - plo[2];
                        const bool zin = valid && sz >= 0 && sz < pn[2];
                        const bool inside = zin && in_xy;
                        ins[k] = inside;
                        if (BOX == 2 && valid && !inside) me |= 1u << k;
                        if constexpr (std::is_same<PT, float>::value) {
                            // unconditional (a clamped plane is in bounds), so the
                            // widening is not pulled into a branch with its own wait
                            const size_t go = phoff + (size_t)min(gz, C.N[2] - 1) * gplane;
                            pv[k] = ph[go + gcol];
                            pv[k] = valid ? pv[k] : 0.0f;
                        } else {
                            const size_t go = phoff + (size_t)(valid ? gz : 0) * gplane;
                            pv[k] = valid ? ph[go + gcol] : 0.0;
                        }
                        const double* vz = v + (size_t)(zin ? sz : 0) * vplane;
                        vv[k] = inside ? vz[vcol] : 0.0;
                    }
                    if constexpr (BOX == 2) {
                        if (me) {   // the multipole value outside the domain (W boxes beyond it)
                            // the column's line coefficients once; then every
                            // point, without a branch between them
                            const double* org = a.pairs[pid].origin;
                            const double d[3] = {(D[0] + lx) * C.h[0] - org[0], (D[1] + ly) * C.h[1] - org[1], 0.0};
                            double ql[SEA_LMAX + 1][SEA_LMAX + 1];
                            me_line_coeffs<2>(CF.cf[q % SC_CFN], d, ql);
                            const double rt2 = d[0] * d[0] + d[1] * d[1];
#pragma unroll
                            for (int k = 0; k < SC_TZ; ++k) {
                                int lz = lz0 + k;
                                lz -= (lz >= C.N[2]) ? C.N[2] : 0;
                                const double z = (D[2] + lz + lzi) * C.h[2] - org[2];
                                // (at the origin itself, inside a domain, the value is not used)
                                const double mv = me_line_potential(ql, z, rt2);
                                vv[k] = (me >> k & 1u) ? mv : vv[k];
                            }
                        }
                    }
#pragma unroll
                    for (int k = 0; k < SC_TZ; ++k) {
                        const double c = vv[k] * (double)pv[k];
                        acc[k] += c;
                        if (ins[k]) ep += po_s[k][threadIdx.x] * c;
                    }
                }
                if (eslot >= 0) {   // uniform: every lane of the workgroup is here
#pragma unroll
                    for (int off = 32; off > 0; off >>= 1) ep += __shfl_xor(ep, off, 64);
                    if ((threadIdx.x & 63) == 0) ep_w[list[q] - e0][threadIdx.x >> 6] = ep;
                }
            }
        }
        __syncthreads();
    }
    // the energy partials: the wavefronts' parts of each entry summed in a
    // fixed order
    if (take_e)
    for (int q = threadIdx.x; q < e1 - e0; q += SC_BS) {
        if (ep_slot_of[q] >= 0) {
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < SC_BS / 64; ++w) t += ep_w[q][w];
            a.epart[(size_t)ep_pid_of[q] * a.ep_stride + ep_slot_of[q]] = t;
        }
    }
#pragma unroll
    for (int k = 0; k < SC_TX * SC_TY * SC_TZ / SC_BS; ++k) {
        const int lid = threadIdx.x + k * SC_BS;
        const int gx = tx0 + lid % SC_TX, gy = ty0 + (lid / SC_TX) % SC_TY, gz = tz0 + lid / (SC_TX * SC_TY);
        if (gx >= C.N[0] || gy >= C.N[1] || gz >= C.N[2]) continue;
        W[(size_t)o * C.Ng + ((size_t)gz * C.N[1] + gy) * C.N[0] + gx] = acc[k];
    }
}

template <int BOX, typename PT, int ORDER>
__global__ __launch_bounds__(SC_BS, BOX ? 4 : 5) void k_scatter(ExxArgs a, const DevCell C,
                                                                const int* __restrict__ off_all,
                                                                const ScEntry* __restrict__ ent) {
    __shared__ ScShared S;
    ScNone none;
    const int n_tiles = sc_tiles(C);
    int o, t;
    sc_block<ORDER>(n_tiles, C.n_occ, o, t);
    if (t >= n_tiles) return;
    scatter_tile<BOX, PT>(a, C, off_all, ent, o, t, S, none);
}

// BOX 2 in two launches.  Most tiles of most orbitals meet no box there (the
// epsilon boxes of the 64-molecule cell: 37 of 230 thousand do), and a workgroup
// of the kernel above, whose multipole path takes the registers of a third of
// a CU, spends its time finding that out.  This one, at full occupancy, writes
// the zeros of the tiles no box meets and lists the others.
template <int ORDER>
__global__ __launch_bounds__(SC_BS) void k_scatter_scan(const DevCell C, const int* __restrict__ off_all,
                                                        const ScEntry* __restrict__ ent, int* __restrict__ work) {
    __shared__ int any;
    const int n_tiles = sc_tiles(C);
    int o, t;
    sc_block<ORDER>(n_tiles, C.n_occ, o, t);
    if (t >= n_tiles) return;
    const int tiles_x = (C.N[0] + SC_TX - 1) / SC_TX, tiles_y = (C.N[1] + SC_TY - 1) / SC_TY;
    const int tx0 = t % tiles_x * SC_TX, ty0 = t / tiles_x % tiles_y * SC_TY, tz0 = t / (tiles_x * tiles_y) * SC_TZ;
    const int* off = off_all + C.csr_base;
    const int e0 = off[o], e1 = off[o + 1];
    if (threadIdx.x == 0) any = 0;
    __syncthreads();
    bool hit = false;
    for (int e = e0 + threadIdx.x; e < e1; e += SC_BS) {
        const int* D = ent[e].D;
        hit = hit || (axis_hits(tx0, SC_TX, D[0], D[3], C.N[0]) && axis_hits(ty0, SC_TY, D[1], D[4], C.N[1]) &&
                      axis_hits(tz0, SC_TZ, D[2], D[5], C.N[2]));
    }
    if (hit) any = 1;
    __syncthreads();
    if (any) {
        if (threadIdx.x == 0) work[1 + atomicAdd(work, 1)] = t * C.n_occ + o;
        return;
    }
#pragma unroll
    for (int k = 0; k < SC_TZ; ++k) {
        const int gx = tx0 + (int)threadIdx.x % SC_TX, gy = ty0 + (int)threadIdx.x / SC_TX, gz = tz0 + k;
        if (gx < C.N[0] && gy < C.N[1] && gz < C.N[2])
            C.W[(size_t)o * C.Ng + ((size_t)gz * C.N[1] + gy) * C.N[0] + gx] = 0.0;
    }
}

template <typename PT>
__global__ __launch_bounds__(SC_BS, 3) void k_scatter_listed(ExxArgs a, const DevCell C, const int* __restrict__ off_all,
                                                             const ScEntry* __restrict__ ent,
                                                             const int* __restrict__ work) {
    __shared__ ScShared S;
    __shared__ ScCoeffs CF;
    const int n = work[0];
    for (int i = blockIdx.x; i < n; i += gridDim.x) {
        const int k = work[1 + i];
        scatter_tile<2, PT>(a, C, off_all, ent, k % C.n_occ, k / C.n_occ, S, CF);
        __syncthreads();   // the arrays in LDS are reused
    }
}

__global__ __launch_bounds__(256) void k_epart_clear(double* __restrict__ p, size_t n) {
    for (size_t k = blockIdx.x * (size_t)256 + threadIdx.x; k < n; k += (size_t)gridDim.x * 256) p[k] = 0.0;
}

}  // namespace

hipError_t launch_epart_clear(const ExxArgs& a, hipStream_t s) {
    const size_t n = (size_t)a.n_pairs * a.ep_stride;
    if (!a.epart || n == 0) return hipSuccess;
    const unsigned nb = (unsigned)std::min<size_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(k_epart_clear, dim3(nb), dim3(256), 0, s, a.epart, n);
    return hipGetLastError();
}

namespace {
using ScatterKernel = void (*)(ExxArgs, const DevCell, const int*, const ScEntry*);
using ScanKernel = void (*)(const DevCell, const int*, const ScEntry*, int*);
struct ScatterVariant {
    const char* name;
    int order;
    ScatterKernel k[2][2];   // [W boxes][FP32 orbitals]
    ScanKernel scan;
};
template <int ORDER>
ScatterVariant scatter_variant(const char* name) {
    return {name,
            ORDER,
            {{k_scatter<0, double, ORDER>, k_scatter<0, float, ORDER>},
             {k_scatter<1, double, ORDER>, k_scatter<1, float, ORDER>}},
            k_scatter_scan<ORDER>};
}
const ScatterVariant kScatterVariants[] = {
    scatter_variant<2>("scatter-xcd-owners"),
    scatter_variant<0>("scatter-orbital-tiles"),
};
constexpr int kNumScatter = sizeof(kScatterVariants) / sizeof(kScatterVariants[0]);
long sc_cell_tiles(const DevCell& c) {
    return (long)((c.N[0] + SC_TX - 1) / SC_TX) * ((c.N[1] + SC_TY - 1) / SC_TY) * ((c.N[2] + SC_TZ - 1) / SC_TZ);
}
}  // namespace

int scatter_variant_count() { return kNumScatter; }
const char* scatter_variant_name(int v) { return v >= 0 && v < kNumScatter ? kScatterVariants[v].name : nullptr; }

size_t scatter_work_ints(const DevCell& c) { return c.wbox == 2 ? 1 + (size_t)sc_cell_tiles(c) * c.n_occ : 0; }

hipError_t launch_scatter(const ExxArgs& a, const DevCell& cell, const int* csr_off, const ScEntry* csr_ent, int* work,
                          int variant, int n_cu, hipStream_t s) {
    if (variant < 0 || variant >= kNumScatter) return hipErrorInvalidValue;
    const ScatterVariant& V = kScatterVariants[variant];
    const long tiles = sc_cell_tiles(cell), nb = sc_grid(V.order, (int)tiles, cell.n_occ);
    if (nb > 0x7fffffffL) return hipErrorInvalidValue;
    if (cell.wbox < 2) {
        hipLaunchKernelGGL(V.k[cell.wbox][cell.phi_f32 ? 1 : 0], dim3((unsigned)nb), dim3(SC_BS), 0, s, a, cell, csr_off,
                           csr_ent);
        return hipGetLastError();
    }
    hipError_t e = launch_fill_int(work, 1, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(V.scan, dim3((unsigned)nb), dim3(SC_BS), 0, s, cell, csr_off, csr_ent, work);
    const long items = tiles * cell.n_occ, most = 12L * n_cu;   // a few rounds of three workgroups per CU
    const dim3 grid((unsigned)(items < most ? items : most));
    if (cell.phi_f32)
        hipLaunchKernelGGL(k_scatter_listed<float>, grid, dim3(SC_BS), 0, s, a, cell, csr_off, csr_ent, work);
    else
        hipLaunchKernelGGL(k_scatter_listed<double>, grid, dim3(SC_BS), 0, s, a, cell, csr_off, csr_ent, work);
    return hipGetLastError();
}
