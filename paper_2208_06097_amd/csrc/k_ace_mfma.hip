// ACE products on the matrix cores (Eq. 18-19): the two shapes of the ACE
// build and apply, for FP64, FP32 and BF16 operands.
//
//   NT (long K):  C = alpha A B^T, A: m x K, B: n x K, K = grid points.
//                 Split over K; every workgroup writes an FP64 partial
//                 m x n block of its K slice and a second kernel sums the
//                 slices in FP64 (M = dV Phi^T W, dV psi xi^T, dV Phi^T xi).
//   NN (small K): C = alpha A B, A: m x K (FP64, small), B: K x ncol,
//                 ncol = grid points (xi = L^-1 W, K psi = -C xi).
//                 Persistent workgroups walk the column tiles with the
//                 stages of the next tile in flight over the end of this one.
//
// Operand kinds: FP64 -> v_mfma_f64_16x16x4f64 (FP64 accumulation);
// FP32 -> v_mfma_f32_16x16x4f32 and BF16 -> v_mfma_f32_16x16x32_bf16, both
// with FP32 accumulation inside a workgroup's K range.  Inputs of another
// type are rounded to the operand kind while they are staged in LDS.
//
// Tiling: 256 threads, four wavefronts in a 2 x 2 grid of 16P x 16Q tiles
// each.  An operand row's share of a K stage is eight 16-byte chunks (KT = 16
// FP64, 32 FP32, 64 BF16 values; NN's BF16 stage: four chunks, 32 values) at
// a pitch of nine (five): chunks of consecutive rows then start in different
// banks.  A thread moves whole chunks: one wide load (rows of an odd grid are
// aligned to their element only, which global loads take), one 16-byte LDS
// write, and 16-byte LDS reads whose values feed consecutive matrix
// instructions.  For that, lane group g = lane / 16 takes k = CE g + s in step
// s (CE values per chunk); A and B agree, so only the order of the sum
// differs from the natural one.  Two LDS buffers: the next stage is written
// between the halves of this one's matrix work, and one barrier per stage
// remains.
// Block heights follow the matrix (32 to 128 rows): small products are bound by
// reading their operands and large ones by the matrix cores.  Measured, against
// 128 x 128 blocks throughout with element-wise staging between two barriers:
// FP64 32 x 32 x 216000 320 -> 22 us (5.0 TB/s), 256 x 256 x 1728000 4.19 ->
// 3.45 ms (66 TFLOP/s); FP32 NN 256 x 256 x 1728000 2.66 -> 2.21 ms, its
// triangular form 2.80 -> 1.86 ms; BF16 NN 200 x 152 x 1030301 0.63 -> 0.43 ms.
// Operand lanes: A row = lane % 16, B column = lane % 16, k block = lane / 16.
// Result lanes: column = lane % 16; the row of item v is 4 (lane / 16) + v
// for the FP32-accumulating instructions and lane / 16 + 4 v for the FP64
// one (measured on gfx950).
#include <algorithm>
#include <type_traits>

#include "k_ace.h"
#include "sea_internal.h"

namespace {

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));

constexpr int NT = 256;
constexpr int BN = 128;   // columns of an NN tile
// Workgroups are handed to the 8 XCDs (each with its own L2) in turn.  The
// workgroups that read the same operand tiles (NT: the output tiles of one
// K slice; NN: the row blocks of one column tile of the grid-point operand)
// are given consecutive places in one XCD's sequence, so that they run there
// together and the second read of a tile comes from that L2.
constexpr int ACE_XCD = 8;
__host__ __device__ inline long xcd_grid(long groups, int per_group) {
    return (groups + ACE_XCD - 1) / ACE_XCD * ACE_XCD * per_group;
}
// workgroup k -> (group, member): group g's members on XCD g % ACE_XCD
__device__ __forceinline__ void xcd_block(int per_group, long& group, int& member) {
    const long k = blockIdx.x, x = k % ACE_XCD, mseq = k / ACE_XCD;
    member = (int)(mseq % per_group);
    group = (mseq / per_group) * ACE_XCD + x;
}

__device__ __forceinline__ float bf_to_f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ uint16_t f_to_bf(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0;
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// value of a stored element as float/double
template <typename T>
__device__ __forceinline__ double as_d(T v) { return (double)v; }
template <>
__device__ __forceinline__ double as_d<uint16_t>(uint16_t v) { return (double)bf_to_f(v); }
template <typename T>
__device__ __forceinline__ float as_f(T v) { return (float)v; }
template <>
__device__ __forceinline__ float as_f<uint16_t>(uint16_t v) { return bf_to_f(v); }

// N consecutive values, loaded or stored as one access at element alignment
template <typename T, int N>
struct Chunk {
    T v[N];
};
template <int N, typename T>
__device__ __forceinline__ Chunk<T, N> load_chunk(const T* p) {
    Chunk<T, N> c;
    __builtin_memcpy(&c, p, sizeof(c));
    return c;
}

// per-kind operand element, chunk and matrix step
template <int KIND>
struct Kind;
template <>
struct Kind<ACE_F64> {
    using E = double;
    using Vec = f64x2;
    using Acc = f64x4;
    static constexpr int CE = 2, STEPS = 2;   // values and matrix steps of a chunk
    // output item v of lane-group g holds tile row g + 4 v (FP64 layout)
    __device__ static int row(int g, int v) { return g + 4 * v; }
    template <typename T>
    __device__ static E cvt(T v) { return as_d(v); }
    __device__ static Acc mma(Vec a, Vec b, int s, Acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], b[s], c, 0, 0, 0);
    }
};
template <>
struct Kind<ACE_F32> {
    using E = float;
    using Vec = f32x4;
    using Acc = f32x4;
    static constexpr int CE = 4, STEPS = 4;
    // output item v of lane-group g holds tile row 4 g + v
    __device__ static int row(int g, int v) { return 4 * g + v; }
    template <typename T>
    __device__ static E cvt(T v) { return as_f(v); }
    __device__ static Acc mma(Vec a, Vec b, int s, Acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], b[s], c, 0, 0, 0);
    }
};
template <>
struct Kind<ACE_BF16> {
    using E = uint16_t;
    using Vec = u16x8;
    using Acc = f32x4;
    static constexpr int CE = 8, STEPS = 1;
    __device__ static int row(int g, int v) { return 4 * g + v; }
    template <typename T>
    __device__ static E cvt(T v) {
        if constexpr (std::is_same<T, uint16_t>::value) return v;  // already BF16 bits
        else return f_to_bf(as_f(v));
    }
    __device__ static Acc mma(Vec a, Vec b, int, Acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                       0, 0, 0);
    }
};

// A chunk of T as the 16 bytes of the operand kind
template <int KIND, typename T>
__device__ __forceinline__ typename Kind<KIND>::Vec to_vec(const Chunk<T, Kind<KIND>::CE>& c) {
    typename Kind<KIND>::Vec v;
#pragma unroll
    for (int i = 0; i < Kind<KIND>::CE; ++i) v[i] = Kind<KIND>::cvt(c.v[i]);
    return v;
}

// Workgroups per CU asked of the compiler: what the LDS of the two buffers
// (9 KB per 32 rows) holds, up to four.  An FP64 block of 128 x 128 has 128
// accumulator registers a lane and fits twice.
constexpr int nt_minb(int P, int Q) { return P + Q <= 4 ? 4 : P + Q <= 5 ? 3 : 2; }
// Stages in flight in registers beside the two in LDS.  Large BF16 blocks wait for
// their loads (59% of the wavefronts' time with one); a large FP64 or FP32 block
// has no registers left for a second and small blocks gain nothing.
constexpr int nt_ahead(int kind, int P, int Q) { return kind == ACE_BF16 && P * Q > 4 ? 2 : 1; }

template <int KIND, typename TA, typename TB, int P, int Q>
__global__ __launch_bounds__(NT, nt_minb(P, Q)) void k_nt_mfma(const TA* __restrict__ A, const TB* __restrict__ B,
                                                               int m, int n, long K, long kslice, int splits,
                                                               double* __restrict__ part) {
    using Kd = Kind<KIND>;
    using E = typename Kd::E;
    using Vec = typename Kd::Vec;
    constexpr int CE = Kd::CE, KT = 8 * CE, PITCH = 9 * CE;
    constexpr int TM = 32 * P, TN = 32 * Q;
    __shared__ __attribute__((aligned(16))) E As[2][TM * PITCH];
    __shared__ __attribute__((aligned(16))) E Bs[2][TN * PITCH];
    // group: K slice; member: output tile
    const int tn = (n + TN - 1) / TN, tm = (m + TM - 1) / TM;
    long slice;
    int tile;
    if (splits < ACE_XCD) {   // (too few slices to give each XCD some: the tiles go round)
        slice = blockIdx.x / (tn * tm);
        tile = blockIdx.x % (tn * tm);
    } else {
        xcd_block(tn * tm, slice, tile);
    }
    if (slice >= splits) return;   // padding of the last XCD round (an empty slice still writes its zeros)
    const long kb = slice * kslice;
    const int j0 = (tile % tn) * TN, i0 = (tile / tn) * TM;
    const long ke = min(K, kb + kslice);
    typename Kd::Acc acc[P][Q];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int q = 0; q < Q; ++q) acc[p][q] = typename Kd::Acc{0, 0, 0, 0};
    // Chunk e of thread t: row t / 8 + 32 e, k CE (t % 8).  Rows past the
    // matrix repeat its last one: what they give is not stored.
    const int cr = threadIdx.x >> 3, ck = CE * (threadIdx.x & 7);
    const TA* pa[P];
    const TB* pb[Q];
#pragma unroll
    for (int e = 0; e < P; ++e) pa[e] = A + (size_t)min(i0 + cr + 32 * e, m - 1) * K + ck;
#pragma unroll
    for (int e = 0; e < Q; ++e) pb[e] = B + (size_t)min(j0 + cr + 32 * e, n - 1) * K + ck;
    constexpr int AH = nt_ahead(KIND, P, Q);
    Chunk<TA, CE> ra[AH][P];
    Chunk<TB, CE> rb[AH][Q];
    auto load_whole = [&](long k0, int slot = 0) {
#pragma unroll
        for (int e = 0; e < P; ++e) ra[slot][e] = load_chunk<CE>(pa[e] + k0);
#pragma unroll
        for (int e = 0; e < Q; ++e) rb[slot][e] = load_chunk<CE>(pb[e] + k0);
    };
    auto load = [&](int slot, long k0) {
        if (k0 + KT <= ke) {
            load_whole(k0, slot);
        } else {
            const int kl = (int)(ke - k0) - ck;   // values of this thread's chunk inside
#pragma unroll
            for (int e = 0; e < P; ++e)
#pragma unroll
                for (int i = 0; i < CE; ++i) ra[slot][e].v[i] = i < kl ? pa[e][k0 + i] : TA(0);
#pragma unroll
            for (int e = 0; e < Q; ++e)
#pragma unroll
                for (int i = 0; i < CE; ++i) rb[slot][e].v[i] = i < kl ? pb[e][k0 + i] : TB(0);
        }
    };
    auto stage = [&](int slot, int buf) {
#pragma unroll
        for (int e = 0; e < P; ++e)
            *reinterpret_cast<Vec*>(&As[buf][(cr + 32 * e) * PITCH + ck]) = to_vec<KIND, TA>(ra[slot][e]);
#pragma unroll
        for (int e = 0; e < Q; ++e)
            *reinterpret_cast<Vec*>(&Bs[buf][(cr + 32 * e) * PITCH + ck]) = to_vec<KIND, TB>(rb[slot][e]);
    };
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int r = lane & 15, g = lane >> 4;
    auto mma = [&](int buf, int h) {
        Vec a[P], b[Q];
#pragma unroll
        for (int p = 0; p < P; ++p)
            a[p] = *reinterpret_cast<const Vec*>(&As[buf][((wm * P + p) * 16 + r) * PITCH + (4 * h + g) * CE]);
#pragma unroll
        for (int q = 0; q < Q; ++q)
            b[q] = *reinterpret_cast<const Vec*>(&Bs[buf][((wn * Q + q) * 16 + r) * PITCH + (4 * h + g) * CE]);
#pragma unroll
        for (int s = 0; s < Kd::STEPS; ++s)
#pragma unroll
            for (int p = 0; p < P; ++p)
#pragma unroll
                for (int q = 0; q < Q; ++q) acc[p][q] = Kd::mma(a[p], b[q], s, acc[p][q]);
    };
    if constexpr (AH == 1) {
        if (kb < ke) {
            load(0, kb);
            stage(0, 0);
            if (kb + KT < ke) load(0, kb + KT);
            lds_sync();
            int buf = 0;
            long k0 = kb;
            // whole stages with two more behind them: no branches, and the LDS
            // writes and loads dealt out between the matrix instructions (in one
            // run they hold up the next operands' reads: FP64 256 x 256 x 1728000
            // 3.87 -> 3.45 ms, 66 TFLOP/s)
            for (; k0 + 3 * KT <= ke; k0 += KT) {
                mma(buf, 0);
                stage(0, buf ^ 1);
                load_whole(k0 + 2 * KT);
                mma(buf, 1);
                constexpr int MM = P * Q * Kd::STEPS;   // of one half
                __builtin_amdgcn_sched_group_barrier(0x100, P + Q, 0);   // first half's operands
#pragma unroll
                for (int e = 0; e < P + Q; ++e) {
                    __builtin_amdgcn_sched_group_barrier(0x008, MM / (P + Q), 0);
                    __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
                }
                __builtin_amdgcn_sched_group_barrier(0x100, P + Q, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 2 * MM, 0);
                lds_sync();   // the loads in flight cross it
                buf ^= 1;
            }
            for (; k0 < ke; k0 += KT) {
                mma(buf, 0);
                if (k0 + KT < ke) stage(0, buf ^ 1);
                if (k0 + 2 * KT < ke) load(0, k0 + 2 * KT);
                mma(buf, 1);
                lds_sync();
                buf ^= 1;
            }
        }
    } else if (kb < ke) {
        load(0, kb);
        stage(0, 0);
#pragma unroll
        for (int u = 0; u < AH; ++u)
            if (kb + (u + 1) * KT < ke) load(u, kb + (u + 1) * KT);
        lds_sync();
        // stage i: slot (i - 1) % AH holds stage i once stage i - 1 is multiplied
        int buf = 0;
        for (long k0 = kb; k0 < ke; k0 += AH * KT) {
#pragma unroll
            for (int u = 0; u < AH; ++u) {
                const long k = k0 + u * KT;
                if (u > 0 && k >= ke) break;
                mma(buf, 0);
                if (k + KT < ke) stage(u, buf ^ 1);
                if (k + (AH + 1) * KT < ke) load(u, k + (AH + 1) * KT);
                mma(buf, 1);
                lds_sync();   // the loads in flight cross it
                buf ^= 1;
            }
        }
    }
    double* Pt = part + (size_t)slice * m * n;
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = i0 + (wm * P + p) * 16 + Kd::row(g, v);
                const int j = j0 + (wn * Q + q) * 16 + r;
                if (i < m && j < n) Pt[(size_t)i * n + j] = (double)acc[p][q][v];
            }
}

// C = alpha (sum of the slices): 32 elements per workgroup, 8 threads each
// taking every eighth slice (256 slices of 256 x 256, 134 MB: 91 -> 33 us
// against one thread per element, whose loads wait on each other's sums).
constexpr int SS_E = 32, SS_G = 8;
__global__ __launch_bounds__(SS_E* SS_G) void k_slice_sum(const double* __restrict__ part, int splits, int mn,
                                                          double alpha, double* __restrict__ C) {
    __shared__ double red[SS_G][SS_E];
    const int e = threadIdx.x % SS_E, g = threadIdx.x / SS_E;
    const int t = blockIdx.x * SS_E + e;
    double s = 0.0;
    if (t < mn) {
#pragma unroll 8
        for (int q = g; q < splits; q += SS_G) s += part[(size_t)q * mn + t];
    }
    red[g][e] = s;
    __syncthreads();
    if (g || t >= mn) return;
    for (int i = 1; i < SS_G; ++i) s += red[i][e];
    C[t] = alpha * s;
}

template <typename T>
__device__ __forceinline__ T store_as(double v);
template <>
__device__ __forceinline__ double store_as<double>(double v) { return v; }
template <>
__device__ __forceinline__ float store_as<float>(double v) { return (float)v; }
template <>
__device__ __forceinline__ uint16_t store_as<uint16_t>(double v) { return f_to_bf((float)v); }

// Persistent: `slots` workgroups per (XCD, row block), all resident at once.
// Workgroup k runs on XCD x = k % 8; with q = k / 8 it takes row block
// q % (row blocks) and slot s = q / (row blocks), and walks the column tiles
// jt = (s + i slots) 8 + x, i = 0, 1, ..., so that the row blocks of one
// column tile run together on one XCD (the second read of the tile comes
// from that L2).  Stages are counted through the tiles: the pipeline does
// not drain between them (K is short here: the orbital count).
//
// FP64 and FP32 columns stay as they lie in memory: B staged [k][column],
// read as runs of consecutive columns, so that a lane's results are runs too
// (4 FP32, 2 FP64) and leave as 16-byte stores.  BF16 needs 8 consecutive k of
// a column: a thread loads 4 x 4 (k x column) and writes each column's four
// values; column c of a 64-wide half lies at row (c % 4) 16 + c / 4, so that
// tile q holds the columns 4 r + q as well.
//
// RES: the workgroup's rows of A stay in LDS for all its tiles (converted
// once) where that leaves two workgroups per CU; else they are staged with B.
// LOWER: A(i, k) = 0 for k > i, and a row block stops at its last row's k;
// a workgroup then takes the next row block with each tile, so that all do
// the same work.
//
// FP32 256 x 256 x 1728000 2.66 -> 1.95 ms, FP64 4.46 -> 4.1 ms with the staging
// dealt out inside the tiles.
template <int KIND>
struct NN {
    using Kd = Kind<KIND>;
    static constexpr int CH = KIND == ACE_BF16 ? 4 : 8;       // chunks of a row's stage
    static constexpr int KT = CH * Kd::CE, PITCH = (CH + 1) * Kd::CE;
    static constexpr int B_ELEMS = KIND == ACE_BF16 ? BN * PITCH : KT * BN;
    static constexpr int ROWS = NT / CH;                      // A rows of one pass of the threads
};
constexpr int nn_minb(int P) { return P <= 2 ? 3 : 2; }
// Stages of B in flight in registers: BF16 operands with the coefficients resident
// are bound by them (FP64 and FP32 gain nothing).
template <int KIND, typename TB>
constexpr int nn_ahead(bool res) { return res && KIND == ACE_BF16 && sizeof(TB) == 2 ? 4 : 1; }

template <int KIND, typename TB, typename TC, int P, bool RES, bool LOWER>
__global__ __launch_bounds__(NT, nn_minb(P)) void k_nn_mfma(const double* __restrict__ A, long sai, long sak,
                                                            const TB* __restrict__ B, int m, int K, long ncol,
                                                            double alpha, TC* __restrict__ C, int slots) {
    using Kd = Kind<KIND>;
    using S = NN<KIND>;
    using E = typename Kd::E;
    using Vec = typename Kd::Vec;
    constexpr int CE = Kd::CE, KT = S::KT, PITCH = S::PITCH;
    constexpr int TM = 32 * P, PA = (TM + S::ROWS - 1) / S::ROWS;
    constexpr int AST = TM * PITCH;   // one stage of A in LDS
    extern __shared__ __attribute__((aligned(16))) char nn_smem[];
    E* const Bs = reinterpret_cast<E*>(nn_smem);            // [2][B_ELEMS]
    E* const As = Bs + 2 * S::B_ELEMS;                     // RES: every stage; else [2]
    const int per = (m + TM - 1) / TM;
    const int x = blockIdx.x % ACE_XCD, mseq = blockIdx.x / ACE_XCD;
    const long ntile = (ncol + BN - 1) / BN, jstep = (long)slots * ACE_XCD;
    const int nst_all = K > 0 ? (K + KT - 1) / KT : 1;   // K = 0: one stage of zeros
    struct It {
        long jt;
        int st, ib;
    };
    auto stages = [&](int ib) { return LOWER ? min(nst_all, ((ib + 1) * TM + KT - 1) / KT) : nst_all; };
    auto next = [&](It it) {
        if (it.st + 1 < stages(it.ib)) return It{it.jt, it.st + 1, it.ib};
        return It{it.jt + jstep, 0, LOWER ? (it.ib + 1 < per ? it.ib + 1 : 0) : it.ib};
    };
    It cur{(long)(mseq / per) * ACE_XCD + x, 0, mseq % per};
    if (cur.jt >= ntile) return;
    typename Kd::Acc acc[P][4];
#pragma unroll
    for (int p = 0; p < P; ++p)
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[p][q] = typename Kd::Acc{0, 0, 0, 0};

    // A: chunk e of thread t: row t / CH + ROWS e, k CE (t % CH); rows past m
    // repeat the last one, k past K are zeros
    const int ar = threadIdx.x / S::CH, ak = CE * (threadIdx.x % S::CH);
    Chunk<double, CE> ra[PA];
    auto a_at = [&](int ib, int st, int e) {
        return A + (long)min(ib * TM + ar + S::ROWS * e, m - 1) * sai + (long)(st * KT + ak) * sak;
    };
    auto load_a_whole = [&](int ib, int st) {
#pragma unroll
        for (int e = 0; e < PA; ++e) ra[e] = load_chunk<CE>(a_at(ib, st, e));
    };
    auto load_a = [&](int ib, int st) {
        if (sak == 1 && (st + 1) * KT <= K) {
            load_a_whole(ib, st);
        } else {
            const int k0 = st * KT + ak;
#pragma unroll
            for (int e = 0; e < PA; ++e) {
                const double* a = a_at(ib, st, e);
#pragma unroll
                for (int i = 0; i < CE; ++i) ra[e].v[i] = k0 + i < K ? a[i * sak] : 0.0;
            }
        }
    };
    auto stage_a = [&](E* dst) {
#pragma unroll
        for (int e = 0; e < PA; ++e)
            if (TM % S::ROWS == 0 || ar + S::ROWS * e < TM)
                *reinterpret_cast<Vec*>(&dst[(ar + S::ROWS * e) * PITCH + ak]) = to_vec<KIND, double>(ra[e]);
    };
    // B: RB pieces of CB columns per thread
    constexpr int CB = KIND == ACE_F64 ? 2 : 4;
    constexpr int RB = 4;
    // FP64, FP32: piece e is row t / (BN / CB) + e NT / (BN / CB); BF16: rows 4 (t / 32) + e
    const int bc = CB * (threadIdx.x % (BN / CB));
    const int br = KIND == ACE_BF16 ? 4 * (threadIdx.x / (BN / CB)) : threadIdx.x / (BN / CB);
    constexpr int BSTEP = KIND == ACE_BF16 ? 1 : NT / (BN / CB);
    static_assert(KIND == ACE_BF16 ? 4 * NT / (BN / CB) == KT : RB * BSTEP == KT, "B stage");
    constexpr int AH = nn_ahead<KIND, TB>(RES);
    Chunk<TB, CB> rb[AH][RB];
    auto load_b_whole = [&](int slot, long jt, int st) {
        const TB* b = B + (size_t)(st * KT + br) * ncol + jt * BN + bc;
#pragma unroll
        for (int e = 0; e < RB; ++e) rb[slot][e] = load_chunk<CB>(b + (size_t)(e * BSTEP) * ncol);
    };
    auto load_b = [&](int slot, long jt, int st) {
        const long j0 = jt * BN + bc;
        const int k0 = st * KT + br;
        if ((st + 1) * KT <= K && (jt + 1) * BN <= ncol) {
            load_b_whole(slot, jt, st);
        } else {
#pragma unroll
            for (int e = 0; e < RB; ++e)
#pragma unroll
                for (int i = 0; i < CB; ++i)
                    rb[slot][e].v[i] = (k0 + e * BSTEP < K && j0 + i < ncol)
                                           ? B[(size_t)(k0 + e * BSTEP) * ncol + j0 + i]
                                           : TB(0);
        }
    };
    auto stage_b = [&](int slot, int buf) {
        E* dst = Bs + buf * S::B_ELEMS;
        if constexpr (KIND == ACE_BF16) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                Chunk<E, 4> w;
#pragma unroll
                for (int e = 0; e < 4; ++e) w.v[e] = Kd::cvt(rb[slot][e].v[i]);
                const int row = (bc & 64) + i * 16 + ((bc & 63) >> 2);
                __builtin_memcpy(__builtin_assume_aligned(&dst[row * PITCH + br], 8), &w, 8);
            }
        } else {
#pragma unroll
            for (int e = 0; e < RB; ++e) {
                Vec v;
#pragma unroll
                for (int i = 0; i < CB; ++i) v[i] = Kd::cvt(rb[slot][e].v[i]);
                *reinterpret_cast<Vec*>(&dst[(br + e * BSTEP) * BN + bc]) = v;
            }
        }
    };
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int r = lane & 15, g = lane >> 4;
    // column of tile q held by this lane, within the wave's 64
    auto col = [&](int q) { return KIND == ACE_F64 ? 32 * (q >> 1) + 2 * r + (q & 1) : 4 * r + q; };
    auto mma = [&](const E* a_st, int buf, int h) {
        const E* b_st = Bs + buf * S::B_ELEMS;
        Vec a[P];
#pragma unroll
        for (int p = 0; p < P; ++p)
            a[p] = *reinterpret_cast<const Vec*>(&a_st[((wm * P + p) * 16 + r) * PITCH + (4 * h + g) * CE]);
        if constexpr (KIND == ACE_BF16) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const Vec b = *reinterpret_cast<const Vec*>(&b_st[(wn * 64 + q * 16 + r) * PITCH + g * CE]);
#pragma unroll
                for (int p = 0; p < P; ++p) acc[p][q] = Kd::mma(a[p], b, 0, acc[p][q]);
            }
        } else {
#pragma unroll
            for (int s = 0; s < Kd::STEPS; ++s) {
                const E* brow = &b_st[((4 * h + g) * CE + s) * BN + wn * 64];
                E b[4];
                if constexpr (KIND == ACE_F64) {
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        const Vec w = *reinterpret_cast<const Vec*>(&brow[32 * u + 2 * r]);
                        b[2 * u] = w[0];
                        b[2 * u + 1] = w[1];
                    }
                } else {
                    const Vec w = *reinterpret_cast<const Vec*>(&brow[4 * r]);
#pragma unroll
                    for (int q = 0; q < 4; ++q) b[q] = w[q];
                }
#pragma unroll
                for (int p = 0; p < P; ++p)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        Vec bv{};
                        bv[s] = b[q];
                        acc[p][q] = Kd::mma(a[p], bv, s, acc[p][q]);
                    }
            }
        }
    };
    auto store = [&](It it) {
        const int ib = it.ib * TM + wm * 16 * P;
        const long jb = it.jt * BN + wn * 64;
        const bool inside = jb + 64 <= ncol;
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = ib + p * 16 + Kd::row(g, v);
                if (i < m) {
                    TC* Cr = C + (size_t)i * ncol + jb;
#pragma unroll
                    for (int q0 = 0; q0 < 4; q0 += CB) {
                        Chunk<TC, CB> c;
#pragma unroll
                        for (int u = 0; u < CB; ++u) c.v[u] = store_as<TC>(alpha * (double)acc[p][q0 + u][v]);
                        if (inside) {
                            __builtin_memcpy(Cr + col(q0), &c, sizeof(c));
                        } else {
#pragma unroll
                            for (int u = 0; u < CB; ++u)
                                if (jb + col(q0 + u) < ncol) Cr[col(q0 + u)] = c.v[u];
                        }
                    }
                }
            }
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[p][q] = typename Kd::Acc{0, 0, 0, 0};
    };

    if constexpr (RES)
        for (int st = 0; st < nst_all; ++st) {
            load_a(cur.ib, st);
            stage_a(As + st * AST);
        }
    auto load = [&](int slot, It it) {
        if (!RES) load_a(it.ib, it.st);
        load_b(slot, it.jt, it.st);
    };
    auto stage = [&](int slot, int buf) {
        if (!RES) stage_a(As + buf * AST);
        stage_b(slot, buf);
    };
    load(0, cur);
    stage(0, 0);
    It n1 = next(cur);
    if constexpr (AH == 1) {
        if (n1.jt < ntile) load(0, n1);
        lds_sync();
        int buf = 0;
        for (;;) {
            // whole stages inside a column tile with two more behind them: no
            // branches, and the LDS writes and loads dealt out between the matrix
            // instructions (as in the NT product)
            if constexpr (!RES && S::CH == 8) {
                const bool tile_whole = sak == 1 && (cur.jt + 1) * BN <= ncol;
                while (tile_whole && cur.st + 2 < stages(cur.ib) && (cur.st + 3) * KT <= K) {
                    const E* a_st = As + buf * AST;
                    mma(a_st, buf, 0);
                    stage(0, buf ^ 1);
                    load_a_whole(cur.ib, cur.st + 2);
                    load_b_whole(0, cur.jt, cur.st + 2);
                    mma(a_st, buf, 1);
                    constexpr int MM = P * 4 * Kd::STEPS, NW = PA + RB;   // of one half; LDS writes
                    constexpr int LD = KIND == ACE_F32 ? 2 : 1;           // loads per write
                    __builtin_amdgcn_sched_group_barrier(0x100, P + 4, 0);   // first half's operands
#pragma unroll
                    for (int e = 0; e < NW; ++e) {
                        __builtin_amdgcn_sched_group_barrier(0x008, MM / NW, 0);
                        __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x020, LD, 0);
                    }
                    __builtin_amdgcn_sched_group_barrier(0x100, P + 4, 0);
                    __builtin_amdgcn_sched_group_barrier(0x008, 2 * MM, 0);
                    lds_sync();   // the loads in flight cross it
                    ++cur.st;
                    buf ^= 1;
                }
                n1 = next(cur);
            }
            const It n2 = next(n1);
            const E* a_st = As + (RES ? cur.st : buf) * AST;
            if (S::CH == 8) mma(a_st, buf, 0);
            if (n1.jt < ntile) {
                stage(0, buf ^ 1);
                if (n2.jt < ntile) load(0, n2);
            }
            mma(a_st, buf, S::CH == 8 ? 1 : 0);
            if (n1.st == 0) store(cur);
            if (n1.jt >= ntile) return;
            lds_sync();   // the loads in flight cross it
            cur = n1;
            n1 = n2;
            buf ^= 1;
        }
    }
    It ahead = n1;   // the next stage to load
#pragma unroll
    for (int u = 0; u < AH; ++u) {
        if (ahead.jt < ntile) load(u, ahead);
        ahead = next(ahead);
    }
    lds_sync();
    for (int buf = 0;;) {
#pragma unroll
        for (int u = 0; u < AH; ++u) {   // slot u holds n1
            const E* a_st = As + (RES ? cur.st : buf) * AST;
            if (S::CH == 8) mma(a_st, buf, 0);
            if (n1.jt < ntile) stage(u, buf ^ 1);
            if (ahead.jt < ntile) load(u, ahead);
            mma(a_st, buf, S::CH == 8 ? 1 : 0);
            if (n1.st == 0) store(cur);
            if (n1.jt >= ntile) return;
            lds_sync();   // the loads in flight cross it
            cur = n1;
            n1 = next(n1);
            ahead = next(ahead);
            buf ^= 1;
        }
    }
}

// Rows (and columns) of 32 in an NT block: as few blocks of at most 128 as hold
// the side, as thin as that many allow.  Products over a short K are not split
// along it and take smaller blocks until there is one for each CU, or the
// smallest (256 x 256 x 256: 64 workgroups, not 4, 45 -> 11 us).
constexpr long NT_SHORT_K = 2048;
int nt_side(int x) {
    const int nb = (x + 127) / 128;
    return std::max(1, (x + 32 * nb - 1) / (32 * nb));
}
void nt_block(long K, int m, int n, int& P, int& Q) {
    P = nt_side(m);
    Q = nt_side(n);
    auto blocks = [&] { return (long)((m + 32 * P - 1) / (32 * P)) * ((n + 32 * Q - 1) / (32 * Q)); };
    if (K <= NT_SHORT_K)
        while (blocks() < 256 && (P > 1 || Q > 1)) {
            P = std::max(1, P / 2);
            Q = std::max(1, Q / 2);
        }
}

template <int KIND, typename TA, typename TB, int P, int Q>
void nt_launch(unsigned nb, hipStream_t s, const TA* A, const TB* B, int m, int n, long K, long kslice, int splits,
               double* part) {
    hipLaunchKernelGGL((k_nt_mfma<KIND, TA, TB, P, Q>), dim3(nb), dim3(NT), 0, s, A, B, m, n, K, kslice, splits, part);
}
template <int KIND, typename TA, typename TB, int P>
void nt_launch_p(int Q, unsigned nb, hipStream_t s, const TA* A, const TB* B, int m, int n, long K, long kslice,
                 int splits, double* part) {
    switch (Q) {
        case 1: return nt_launch<KIND, TA, TB, P, 1>(nb, s, A, B, m, n, K, kslice, splits, part);
        case 2: return nt_launch<KIND, TA, TB, P, 2>(nb, s, A, B, m, n, K, kslice, splits, part);
        case 3: return nt_launch<KIND, TA, TB, P, 3>(nb, s, A, B, m, n, K, kslice, splits, part);
        default: return nt_launch<KIND, TA, TB, P, 4>(nb, s, A, B, m, n, K, kslice, splits, part);
    }
}

// LDS of an NN workgroup; resident A up to half a CU's 160 KB
constexpr size_t NN_LDS_HALF = 80 * 1024;
template <int KIND>
size_t nn_lds(int P, int a_stages) {
    using S = NN<KIND>;
    return sizeof(typename Kind<KIND>::E) * ((size_t)2 * S::B_ELEMS + (size_t)a_stages * 32 * P * S::PITCH);
}

template <int KIND, typename TB, typename TC, int P, bool RES, bool LOWER>
hipError_t nn_launch(const double* A, long sai, long sak, const TB* B, int m, int K, long ncol, double alpha, TC* C,
                     size_t lds, hipStream_t s) {
    // resident workgroups per CU by registers and the CU count, queried once
    // per process (a thread-safe static initialization)
    struct Fill {
        hipError_t err;
        int occ, n_cu;
    };
    static const Fill fill = [] {
        int dev = 0, o = 0, c = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e == hipSuccess) e = hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev);
        if (e == hipSuccess)
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&o, k_nn_mfma<KIND, TB, TC, P, RES, LOWER>, NT, 0);
        if (e == hipSuccess && (o < 1 || c < 1)) e = hipErrorInvalidValue;
        return Fill{e, o, c};
    }();
    if (fill.err != hipSuccess) return fill.err;
    const int occ = std::max(1, std::min(fill.occ, (int)(2 * NN_LDS_HALF / lds)));
    const int per = (m + 32 * P - 1) / (32 * P);
    const long ntile = (ncol + BN - 1) / BN;
    // as many slots as stay resident (at least one), no more than the tiles need
    long slots = (long)fill.n_cu * occ / ((long)ACE_XCD * per);
    slots = std::max(1L, std::min(slots, (ntile + ACE_XCD - 1) / ACE_XCD));
    const long nb = slots * ACE_XCD * per;
    if (nb > 0x7fffffffL) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_nn_mfma<KIND, TB, TC, P, RES, LOWER>), dim3((unsigned)nb), dim3(NT), lds, s, A, sai, sak, B,
                       m, K, ncol, alpha, C, (int)slots);
    return hipGetLastError();
}
template <int KIND, typename TB, typename TC, int P>
hipError_t nn_launch_p(const double* A, long sai, long sak, const TB* B, int m, int K, long ncol, double alpha, TC* C,
                       bool lower, hipStream_t s) {
    const int nst = K > 0 ? (K + NN<KIND>::KT - 1) / NN<KIND>::KT : 1;
    const size_t res = nn_lds<KIND>(P, nst);
    if (res <= NN_LDS_HALF)
        return nn_launch<KIND, TB, TC, P, true, false>(A, sai, sak, B, m, K, ncol, alpha, C, res, s);
    const size_t lds = nn_lds<KIND>(P, 2);
    // L^-1 multiplies W, which is FP64
    constexpr bool W64 = std::is_same<TB, double>::value;
    if (W64 && lower && m > 32 * P)
        return nn_launch<KIND, TB, TC, P, false, W64>(A, sai, sak, B, m, K, ncol, alpha, C, lds, s);
    return nn_launch<KIND, TB, TC, P, false, false>(A, sai, sak, B, m, K, ncol, alpha, C, lds, s);
}

}  // namespace

// Blocks wanted: two rounds of two workgroups per CU for the large tiles, four
// for the small ones, which are bound by loads in flight; a slice is at least
// four block sides long, so that writing the partials stays small beside
// reading the operands.
int ace_mfma_splits(long K, int m, int n, int max_splits) {
    int P, Q;
    nt_block(K, m, n, P, Q);
    const int tm = 32 * P, tn = 32 * Q;
    const long tiles = (long)((m + tm - 1) / tm) * ((n + tn - 1) / tn);
    const long want = tm * tn <= 64 * 64 ? 2048 : 1024;
    long s = (want + tiles - 1) / tiles;
    const long min_slice = std::max(256, 4 * std::max(tm, tn));
    const long maxs = K <= NT_SHORT_K ? 1 : (K + min_slice - 1) / min_slice;
    if (s > maxs) s = maxs;
    if (max_splits > 0 && s > max_splits) s = max_splits;
    if (s < 1) s = 1;
    return (int)s;
}

template <int KIND, typename TA, typename TB>
hipError_t ace_mm_nt(const TA* A, const TB* B, int m, int n, long K, double alpha, double* part, double* C,
                     hipStream_t s, int max_splits) {
    if (128 * K >= 0x7fffffffL) return hipErrorInvalidValue;
    const int splits = ace_mfma_splits(K, m, n, max_splits);
    int P, Q;
    nt_block(K, m, n, P, Q);
    constexpr int KT = 8 * Kind<KIND>::CE;
    long kslice = (K + splits - 1) / splits;
    kslice = (kslice + KT - 1) / KT * KT;
    const int tiles = ((n + 32 * Q - 1) / (32 * Q)) * ((m + 32 * P - 1) / (32 * P));
    const long nb = splits < ACE_XCD ? (long)splits * tiles : xcd_grid(splits, tiles);
    if (nb > 0x7fffffffL) return hipErrorInvalidValue;
    switch (P) {
        case 1: nt_launch_p<KIND, TA, TB, 1>(Q, (unsigned)nb, s, A, B, m, n, K, kslice, splits, part); break;
        case 2: nt_launch_p<KIND, TA, TB, 2>(Q, (unsigned)nb, s, A, B, m, n, K, kslice, splits, part); break;
        case 3: nt_launch_p<KIND, TA, TB, 3>(Q, (unsigned)nb, s, A, B, m, n, K, kslice, splits, part); break;
        default: nt_launch_p<KIND, TA, TB, 4>(Q, (unsigned)nb, s, A, B, m, n, K, kslice, splits, part); break;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int mn = m * n;
    hipLaunchKernelGGL(k_slice_sum, dim3((mn + SS_E - 1) / SS_E), dim3(SS_E * SS_G), 0, s, part, splits, mn, alpha, C);
    return hipGetLastError();
}

template <int KIND, typename TB, typename TC>
hipError_t ace_mm_nn(const double* A, long sai, long sak, const TB* B, int m, int K, long ncol, double alpha, TC* C,
                     hipStream_t s, bool lower) {
    if (m <= 0 || ncol <= 0) return hipSuccess;
    if (sai < 0 || sak < 0 || 8 * sai + 32 * sak >= 0x7fffffffL || 2 * ncol + BN >= 0x7fffffffL)
        return hipErrorInvalidValue;
    // blocks as in the NT product; the smallest where the columns are few (256 x
    // 256 x 256: 16 workgroups, not 4)
    const int nb = (m + 127) / 128;
    switch (ncol <= NT_SHORT_K && m <= NT_SHORT_K ? 1 : (m + 32 * nb - 1) / (32 * nb)) {
        case 1: return nn_launch_p<KIND, TB, TC, 1>(A, sai, sak, B, m, K, ncol, alpha, C, lower, s);
        case 2: return nn_launch_p<KIND, TB, TC, 2>(A, sai, sak, B, m, K, ncol, alpha, C, lower, s);
        case 3: return nn_launch_p<KIND, TB, TC, 3>(A, sai, sak, B, m, K, ncol, alpha, C, lower, s);
        default: return nn_launch_p<KIND, TB, TC, 4>(A, sai, sak, B, m, K, ncol, alpha, C, lower, s);
    }
}

#define NT_INST(KIND, TA, TB) \
    template hipError_t ace_mm_nt<KIND, TA, TB>(const TA*, const TB*, int, int, long, double, double*, double*, \
                                                hipStream_t, int);
#define NN_INST(KIND, TB, TC)                                                                                      \
    template hipError_t ace_mm_nn<KIND, TB, TC>(const double*, long, long, const TB*, int, int, long, double, TC*, \
                                                hipStream_t, bool);
// M and the energy (FP64 operands; xi converted exactly), dV psi xi^T per ace_dtype
NT_INST(ACE_F64, double, double)
NT_INST(ACE_F64, double, float)
NT_INST(ACE_F64, double, uint16_t)
NT_INST(ACE_F32, float, float)
NT_INST(ACE_BF16, uint16_t, uint16_t)
// xi = L^-1 W and K psi = -C xi per ace_dtype
NN_INST(ACE_F64, double, double)
NN_INST(ACE_F32, double, float)
NN_INST(ACE_F32, float, float)
NN_INST(ACE_BF16, double, uint16_t)
NN_INST(ACE_BF16, uint16_t, float)
