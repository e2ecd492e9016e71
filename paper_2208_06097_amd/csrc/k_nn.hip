// Learned CG warm start: a 3-D U-Net that maps the pair density (resampled
// to a D^3 grid, D = 32 in production) to the correction of the multipole
// guess, plus its backward pass and Adam, all as hand-written kernels.
//
// Network (16 channels; levels D, D/2, D/4, D/8; every 3x3x3 convolution
// but the head followed by ReLU; zero padding 1):
//   e0a(1->16) e0b -> s0, avgpool2, e1a e1b -> s1, avgpool2, e2a e2b -> s2,
//   avgpool2, e3a e3b, up2, [up, s2] d2a(32->16) d2b, up2, [up, s1] d1a d1b,
//   up2, [up, s0] d0a d0b, head(16->1).
//
// Activations: FP32, layout [B][C][D][D][D].  Parameters: one flat FP32
// master array (per layer: weights [O][C][27], then bias [O]); a BF16 copy
// of it is what the convolutions read when BF16 weights are selected.
// Accumulation is FP32 everywhere.
#include <hip/hip_bf16.h>

#include "nn_internal.h"
#include "sea_internal.h"

namespace {

__device__ __forceinline__ float bf16_bits_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// round-to-nearest-even FP32 -> BF16 bits (finite inputs)
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Tiles of a D^3 level: a workgroup takes tx x ty x tz voxels (at most 256)
// of one batch entry and holds them in LDS with one halo voxel on each side.
constexpr int TC_BS = 256;
constexpr int TC_VOX = 256;    // voxels per tile, at most
constexpr int TC_HALO = 816;   // voxels with halo, at most (34 x 6 x 4)
// Division of a small number by a tile's extent: the product with a rounded-up
// reciprocal, exact while number x divisor < 2^20 (at most 4096 x 204 here).
struct TcDiv {
    uint32_t d, m;
};
static TcDiv tc_div(int d) { return TcDiv{(uint32_t)d, (1u << 20) / (uint32_t)d + 1u}; }
__device__ __forceinline__ int operator/(int v, TcDiv q) { return (int)(((uint32_t)v * q.m) >> 20); }
struct TcTile {
    int tx, ty, tz;      // tile extents
    int tiles;           // per batch entry
    int D;
    TcDiv qtx, qtxy;     // tile row, plane
    TcDiv qrp, qpp;      // the same with halo
    TcDiv qnx, qnxy;     // tiles per row, plane of tiles
};
// Rows are kept whole up to 32 voxels (a level's D is at most 64, and even
// above 32): 32 x 4 x 2, 16 x 4 x 4 and 8 x 8 x 4 voxels read 3.2, 2.5 and 2.3
// times their own count with the halo.
static TcTile tc_tile(int D) {
    TcTile t{};
    t.D = D;
    t.tx = D <= 32 ? D : D / 2;
    const int ty = t.tx > 8 ? 4 : 8, tz = t.tx > 16 ? 2 : 4;
    t.ty = ty < D ? ty : D;
    t.tz = tz < D ? tz : D;
    const int nx = (D + t.tx - 1) / t.tx, ny = (D + t.ty - 1) / t.ty;
    t.tiles = nx * ny * ((D + t.tz - 1) / t.tz);
    t.qtx = tc_div(t.tx);
    t.qtxy = tc_div(t.tx * t.ty);
    t.qrp = tc_div(t.tx + 2);
    t.qpp = tc_div((t.tx + 2) * (t.ty + 2));
    t.qnx = tc_div(nx);
    t.qnxy = tc_div(nx * ny);
    return t;
}

// Geometry of one tile inside a kernel.  Voxel v of the tile (x fastest) and
// halo voxel h (one more on each side) in linear indices.
struct TcGeo {
    const TcTile& t;
    int x0, y0, z0;
    int rp, pp;   // halo pitches: row, plane
    __device__ TcGeo(const TcTile& t_, int tile) : t(t_), rp(t_.qrp.d), pp(t_.qpp.d) {
        const int z = tile / t.qnxy, r = tile - z * (int)t.qnxy.d, y = r / t.qnx;
        x0 = (r - y * (int)t.qnx.d) * t.tx;
        y0 = y * t.ty;
        z0 = z * t.tz;
    }
    __device__ int nvox() const { return t.tz * (int)t.qtxy.d; }
    __device__ int nhalo() const { return pp * (t.tz + 2); }
    __device__ void split(int v, int& x, int& y, int& z) const {
        z = v / t.qtxy;
        v -= z * (int)t.qtxy.d;
        y = v / t.qtx;
        x = v - y * t.tx;
    }
    // halo index of tile voxel v's lowest neighbour (tap (0, 0, 0))
    __device__ int corner(int v) const {
        int x, y, z;
        split(v, x, y, z);
        return z * pp + y * rp + x;
    }
    // offset of tap t (z, y, x in 0..2) from that corner
    __device__ int tap(int k) const { return k / 9 * pp + k / 3 % 3 * rp + k % 3; }
    // grid offset of tile voxel v, -1 beyond the grid
    __device__ int at(int v) const {
        int x, y, z;
        split(v, x, y, z);
        x += x0;
        y += y0;
        z += z0;
        return (x < t.D && y < t.D && z < t.D && v < nvox()) ? (z * t.D + y) * t.D + x : -1;
    }
    // grid offset of halo voxel h, -1 beyond the grid; up: in a grid of half
    // the size, upsampled by nearest neighbours
    __device__ int halo_at(int h, bool up) const {
        int z = h / t.qpp;
        h -= z * pp;
        int y = h / t.qrp;
        const int x = h - y * rp + x0 - 1;
        y += y0 - 1;
        z += z0 - 1;
        const int D = t.D;
        if ((unsigned)x >= (unsigned)D || (unsigned)y >= (unsigned)D || (unsigned)z >= (unsigned)D) return -1;
        return up ? ((z >> 1) * (D >> 1) + (y >> 1)) * (D >> 1) + (x >> 1) : (z * D + y) * D + x;
    }
};

// Stages C channels of `src` (channel stride cs) with halo into
// lds[c * CS + halo voxel], zeros beyond the grid.
template <int C, int CS, int BS = TC_BS>
__device__ __forceinline__ void tc_stage(const TcGeo& G, const float* __restrict__ src, size_t cs, bool up, float* lds) {
    constexpr int NP = (TC_HALO + BS - 1) / BS;
    const int nh = G.nhalo();
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        const int h = threadIdx.x + k * BS;
        if (h >= nh) break;
        const int o = G.halo_at(h, up);
        // every load is issued (voxel 0 in place of one beyond the grid), none
        // behind a branch
        const float* p = src + (o >= 0 ? o : 0);
        float v[C];
#pragma unroll
        for (int c = 0; c < C; ++c) v[c] = p[c * cs];
#pragma unroll
        for (int c = 0; c < C; ++c) lds[c * CS + h] = o >= 0 ? v[c] : 0.0f;
    }
}

// 3x3x3 convolutions as implicit GEMMs on the FP32 matrix cores
// (v_mfma_f32_16x16x4f32: FP32 operands and accumulation, one fused
// multiply-add per k in order, twice the rate of the vector FMAs): 16 voxels
// x 16 output channels per instruction.  The input block with its halo and
// the weight block lie in LDS (channel stride 848 floats: 16 banks apart), a
// weight read serves a wavefront's two voxel blocks, and 80 KB a workgroup leaves two per
// CU, one staging while the other multiplies.  Bound by the matrix pipe.
//   Forward: K = the three taps of a row (the middle, the left, the right) and
// a zero, the row's sum added to the total afterwards; bias, channels and
// rows in order.  These are the roundings of acc += w0 v0 + w1 v1 + w2 v2
// with fused multiply-adds: an activation within rounding of zero keeps its side
// of the ReLU, which the gradient follows discontinuously.  (K = 4 channels of
// a tap, as below, would need a quarter fewer instructions.)
//   Gradient w.r.t. the input: K = four channels of one tap, a row of taps
// (48 terms) summed by itself before it joins the total.
// Measured per 16 x 16-channel block at batch 32, D = 32 (14.5 GFLOP):
// forward 258 us, gradient 148 us (98 TFLOP/s); the vector-FMA kernel, which
// read every input from the caches per tap, took 1.1 ms.
constexpr int TC_CS = 848;
constexpr int TC_W = 16 * 16 * 27;   // one 16 x 16-channel weight block, in operand order
struct ConvT {
    const float* in[2];      // 16-channel blocks of the input
    int up[2];               // the block is stored at half size and upsampled
    int nci;
    const float* wp;         // 16 x 16 layers: packed blocks [input block] (forward) or [output block]
    const float* w32;        // one-channel layers: the layer's weights, FP32
    const uint16_t* w16;     // or BF16
    const float* bias;       // nullable
    int flip;                // one-channel layers: gradient w.r.t. the input, W(o, t) = w[o][26 - t]
    float* out[2];           // 16-channel blocks of the output
    const float* mask[2];    // output block zeroed where this is not positive (nullable)
    int relu;
    TcTile t;
};

__device__ __forceinline__ float tc_weight(const float* w32, const uint16_t* w16, int i) {
    return w16 ? bf16_bits_to_f32(w16[i]) : w32[i];
}

// Packs the 16 x 16-channel weight blocks in operand order, once per forward
// or backward pass, so that every tile stages its block by contiguous loads
// (in place they were 27 strided loads a thread and tile).
//   forward:  [channel][row of taps zy][tap tc_dx(g)][o] (lane = 16 g + o)
//   backward: [tap][channel group c4][channel c % 4][o]  (lane = 16 (c % 4) + o),
//             W(o, c, t) = w[c][o][26 - t], o the layer's input channel
__device__ __forceinline__ int tc_dx(int g) { return g == 2 ? 2 : 1 - (g & 1); }   // 1, 0, 2 (g = 3 unused)
constexpr int TC_BLOCKS = 16;   // 13 layers, three of them with two input blocks
struct PackT {
    int off[TC_BLOCKS], cin[TC_BLOCKS], sub[TC_BLOCKS];
};
__global__ __launch_bounds__(256) void k_pack_weights(PackT t, const float* params, const uint16_t* params16, int back,
                                                      float* __restrict__ out) {
    const int b = blockIdx.x, cin = t.cin[b], sub = t.sub[b] * 16;
    const float* w32 = params16 ? nullptr : params + t.off[b];
    const uint16_t* w16 = params16 ? params16 + t.off[b] : nullptr;
    for (int i = threadIdx.x + blockIdx.y * 256; i < TC_W; i += 256 * gridDim.y) {
        const int o = i & 15;
        int src;
        if (back) {
            const int c = (i >> 6 & 3) * 4 + (i >> 4 & 3);
            src = (c * cin + sub + o) * 27 + 26 - (i >> 8);
        } else {
            const int q = i / 48, dx = tc_dx(i / 16 % 3);
            src = (o * cin + sub + q / 9) * 27 + q % 9 * 3 + dx;
        }
        out[(size_t)b * TC_W + i] = tc_weight(w32, w16, src);
    }
}

template <int NB, bool FWD>
__device__ __forceinline__ void tc_multiply(const TcGeo& G, const float* tile, const float* wl, const int* base,
                                            f32x4* acc) {
    const int lane = threadIdx.x & 63;
    if constexpr (FWD) {   // lane group g: tap dx = g of the row (3: zero)
        const bool tap = lane < 48;
        const float* wp = wl + (tap ? lane : 0);
#pragma unroll 1
        for (int c = 0; c < 16; ++c)
#pragma unroll 1
            for (int zz = 0; zz < 3; ++zz) {
                const float* tp = tile + c * TC_CS + zz * G.pp;
                float w[3], v[3][NB];
#pragma unroll
                for (int yy = 0; yy < 3; ++yy) {
                    w[yy] = tap ? wp[(c * 9 + zz * 3 + yy) * 48] : 0.0f;
#pragma unroll
                    for (int b = 0; b < NB; ++b) v[yy][b] = tap ? tp[yy * G.rp + base[b]] : 0.0f;
                }
#pragma unroll
                for (int yy = 0; yy < 3; ++yy) {
                    f32x4 row[NB];
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        row[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[yy][b], w[yy], f32x4{0.0f, 0.0f, 0.0f, 0.0f}, 0,
                                                                      0, 0);
#pragma unroll
                    for (int b = 0; b < NB; ++b) acc[b] += row[b];
                }
            }
    } else {               // lane group g: channel 4 c4 + g
#pragma unroll 1
        for (int zy = 0; zy < 9; ++zy) {
            const float* tp = tile + zy / 3 * G.pp + zy % 3 * G.rp;
            const float* wp = wl + zy * (3 * 256) + lane;
            f32x4 row[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) row[b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                for (int c4 = 0; c4 < 4; ++c4) {
                    const float w = wp[(dx * 4 + c4) * 64];
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        row[b] =
                            __builtin_amdgcn_mfma_f32_16x16x4f32(tp[base[b] + dx + c4 * (4 * TC_CS)], w, row[b], 0, 0, 0);
                }
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[b] += row[b];
        }
    }
}

// Writes a wave's voxel blocks b0 .. b0 + NB - 1 (blocks are dealt to the NW
// waves in turn): lane = channel lane % 16, item v = voxel
// 4 (lane / 16) + v of the block.
template <int NB, int NW>
__device__ __forceinline__ void tc_store(const TcGeo& G, const f32x4* acc, int b0, int nblk, int relu,
                                         float* __restrict__ out, const float* __restrict__ mask) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const size_t D3 = (size_t)G.t.D * G.t.D * G.t.D;
    out += (lane & 15) * D3;
    if (mask) mask += (lane & 15) * D3;
    const bool vec = (G.t.tx & 3) == 0 && (G.t.D & 3) == 0;   // four voxels of one row, 16-byte aligned
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int blk = (b0 + b) * NW + w, v0 = blk * 16 + 4 * (lane >> 4);
        if (blk >= nblk) break;
        f32x4 r = acc[b];
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (relu) r[v] = fmaxf(r[v], 0.0f);
        if (vec) {
            const int o = G.at(v0);
            if (o < 0) continue;
            if (mask) {
                const f32x4 m = *(const f32x4*)(mask + o);
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (!(m[v] > 0.0f)) r[v] = 0.0f;
            }
            *(f32x4*)(out + o) = r;
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int o = G.at(v0 + v);
                if (o >= 0) out[o] = (mask && !(mask[o] > 0.0f)) ? 0.0f : r[v];
            }
        }
    }
}

// grid (tiles, batch, output blocks); eight waves with two voxel blocks each
// (four per SIMD: the row sums and operand reads of some run under the
// products of others)
constexpr int TC_CBS = 512;
template <bool FWD>
__global__ __launch_bounds__(TC_CBS, 4) void k_conv16(ConvT a) {
    __shared__ float tile[16 * TC_CS];
    __shared__ __attribute__((aligned(16))) float wl[TC_W];
    constexpr int NW = TC_CBS / 64, NB = TC_VOX / 16 / NW;
    const TcGeo G(a.t, blockIdx.x);
    const int co = blockIdx.z, lane = threadIdx.x & 63, w = threadIdx.x >> 6, g = lane >> 4;
    const size_t D3 = (size_t)a.t.D * a.t.D * a.t.D, bo = (size_t)blockIdx.y * 16 * D3;
    const int nblk = (G.nvox() + 15) >> 4;
    int base[NB];
    f32x4 acc[NB];
    const float bias = a.bias ? a.bias[co * 16 + (lane & 15)] : 0.0f;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int v = (b * NW + w) * 16 + (lane & 15);
        base[b] = (v < G.nvox() ? G.corner(v) : 0) + (FWD ? tc_dx(g) : g * TC_CS);
        acc[b] = f32x4{bias, bias, bias, bias};
    }
    for (int ci = 0; ci < a.nci; ++ci) {
        if (ci) __syncthreads();
        const f32x4* wsrc = (const f32x4*)(a.wp + (size_t)(FWD ? ci : co) * TC_W);
        for (int i = threadIdx.x; i < TC_W / 4; i += TC_CBS) ((f32x4*)wl)[i] = wsrc[i];
        const bool up = a.up[ci];
        tc_stage<16, TC_CS, TC_CBS>(G, a.in[ci] + (up ? bo / 8 : bo), up ? D3 / 8 : D3, up, tile);
        __syncthreads();
        if (w + NW < nblk) tc_multiply<2, FWD>(G, tile, wl, base, acc);
        else if (w < nblk) tc_multiply<1, FWD>(G, tile, wl, base, acc);
    }
    tc_store<NB, NW>(G, acc, 0, nblk, a.relu, a.out[co] + bo, a.mask[co] ? a.mask[co] + bo : nullptr);
}

// One input channel to 16 outputs (the first layer; the gradient of the head
// w.r.t. its input): a product per row of taps, summed as above.  Memory
// bound (64 B written per voxel).
__global__ __launch_bounds__(TC_BS) void k_conv1(ConvT a) {
    __shared__ float tile[TC_HALO];
    const TcGeo G(a.t, blockIdx.x);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, g = lane >> 4;
    const size_t D3 = (size_t)a.t.D * a.t.D * a.t.D, bo = (size_t)blockIdx.y * 16 * D3;
    const int nblk = (G.nvox() + 15) >> 4;
    float wt[9];
#pragma unroll
    for (int zy = 0; zy < 9; ++zy) {
        const int t = zy * 3 + tc_dx(g);
        wt[zy] = g < 3 ? tc_weight(a.w32, a.w16, (lane & 15) * 27 + (a.flip ? 26 - t : t)) : 0.0f;
    }
    tc_stage<1, TC_HALO>(G, a.in[0] + blockIdx.y * D3, D3, false, tile);
    __syncthreads();
    const float bias = a.bias ? a.bias[lane & 15] : 0.0f;
#pragma unroll 1
    for (int b = 0; b * 4 < nblk; ++b) {
        const int v = (b * 4 + w) * 16 + (lane & 15);
        const int c = (v < G.nvox() ? G.corner(v) : 0) + tc_dx(g);
        f32x4 acc = f32x4{bias, bias, bias, bias};
#pragma unroll
        for (int zy = 0; zy < 9; ++zy) {
            const float in = g < 3 ? tile[c + zy / 3 * G.pp + zy % 3 * G.rp] : 0.0f;
            const f32x4 row = __builtin_amdgcn_mfma_f32_16x16x4f32(in, wt[zy], f32x4{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
            acc += row;
        }
        tc_store<1, 4>(G, &acc, b, nblk, a.relu, a.out[0] + bo, a.mask[0] ? a.mask[0] + bo : nullptr);
    }
}

// 16 channels to one (the head): a thread per voxel on the vector FMAs (a
// matrix product would fill one of 16 columns).  Bound by its 432 LDS reads
// per voxel.
__global__ __launch_bounds__(TC_BS) void k_conv_to1(ConvT a) {
    __shared__ float tile[16 * TC_CS];
    __shared__ float wl[16 * 27];
    const TcGeo G(a.t, blockIdx.x);
    const size_t D3 = (size_t)a.t.D * a.t.D * a.t.D;
    for (int i = threadIdx.x; i < 16 * 27; i += TC_BS) wl[i] = tc_weight(a.w32, a.w16, i);
    tc_stage<16, TC_CS>(G, a.in[0] + (size_t)blockIdx.y * 16 * D3, D3, false, tile);
    __syncthreads();
    const int o = G.at(threadIdx.x);
    if (o < 0) return;
    const float* tp = tile + G.corner(threadIdx.x);
    float s = a.bias ? a.bias[0] : 0.0f;
#pragma unroll 2
    for (int c = 0; c < 16; ++c)
#pragma unroll
        for (int zy = 0; zy < 9; ++zy) {
            const float* r = tp + c * TC_CS + zy / 3 * G.pp + zy % 3 * G.rp;
            const float* wr = wl + c * 27 + zy * 3;
            s += wr[0] * r[0] + wr[1] * r[1] + wr[2] * r[2];
        }
    a.out[0][blockIdx.y * D3 + o] = s;
}

// Weight and bias gradients of a 16 x 16-channel block:
// gw[o][c][t] = sum over voxels of g[o][p] in[c][p + tap t].  Per tap a
// 16 x 16 product with K = the voxels, four per instruction; the 27 taps and
// the bias (a column of ones) stay in 28 accumulators over all tiles of the
// workgroup, so a tile costs one g read per four voxels and one input read
// per instruction.  Matrix-pipe bound like k_conv16; channel strides = 2 banks
// apart (16 channels x 2 voxels of a half wave on 32 banks).  Measured at batch 32, D = 32:
// 162 us (93 TFLOP/s); the vector kernel, which read the input once per
// output channel, took 1.5 ms.
constexpr int TW_CS = 834;
constexpr int TW_GS = 258;
constexpr int TW_PART = 28 * 256;   // floats per partial record: [tap][o][c]; tap 27: the bias in every column
struct WgradT {
    const float* in[2];
    int up[2];
    const float* g;
    float* part;    // [ci][workgroup][TW_PART]
    int nb;         // batch
    TcTile t;
};
// grid (workgroups, input blocks)
__global__ __launch_bounds__(TC_BS, 2) void k_wgrad16(WgradT a) {
    __shared__ float tile[16 * TW_CS];
    __shared__ float gl[16 * TW_GS];
    __shared__ int cor[TC_VOX];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, ci = blockIdx.y;
    f32x4 acc[28];
#pragma unroll
    for (int t = 0; t < 28; ++t) acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    const bool up = a.up[ci];
    {
        const TcGeo G(a.t, 0);
        const int v = threadIdx.x;
        cor[v] = v < G.nvox() ? G.corner(v) : 0;
    }
    for (int q = blockIdx.x; q < a.t.tiles * a.nb; q += gridDim.x) {
        const int entry = q / a.t.tiles;
        const TcGeo G(a.t, q - entry * a.t.tiles);
        const size_t D3 = (size_t)a.t.D * a.t.D * a.t.D, bo = (size_t)entry * 16 * D3;
        __syncthreads();
        tc_stage<16, TW_CS>(G, a.in[ci] + (up ? bo / 8 : bo), up ? D3 / 8 : D3, up, tile);
        {
            const int o = G.at(threadIdx.x);
            const float* p = a.g + bo + (o >= 0 ? o : 0);
            float v[16];
#pragma unroll
            for (int c = 0; c < 16; ++c) v[c] = p[c * D3];
#pragma unroll
            for (int c = 0; c < 16; ++c) gl[c * TW_GS + threadIdx.x] = o >= 0 ? v[c] : 0.0f;
        }
        __syncthreads();
        const int nk = (G.nvox() + 3) >> 2;   // groups of four voxels
        for (int k = w; k < nk; k += TC_BS / 64) {
            const int v = 4 * k + (lane >> 4);
            const float gv = gl[(lane & 15) * TW_GS + v];
            const float* tp = tile + (lane & 15) * TW_CS + cor[v];
#pragma unroll
            for (int zy = 0; zy < 9; ++zy) {
                const float* r = tp + zy / 3 * G.pp + zy % 3 * G.rp;
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
                    acc[zy * 3 + dx] = __builtin_amdgcn_mfma_f32_16x16x4f32(gv, r[dx], acc[zy * 3 + dx], 0, 0, 0);
            }
            acc[27] = __builtin_amdgcn_mfma_f32_16x16x4f32(gv, 1.0f, acc[27], 0, 0, 0);
        }
    }
    // the four waves' sums, in wave order (the record fits the tile's LDS)
    static_assert(TW_PART <= 16 * TW_CS, "partial record in the tile array");
#pragma unroll 1
    for (int ww = 0; ww < TC_BS / 64; ++ww) {
        __syncthreads();
        if (w == ww) {
#pragma unroll
            for (int t = 0; t < 28; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    float* p = tile + t * 256 + (4 * (lane >> 4) + v) * 16 + (lane & 15);
                    *p = ww ? *p + acc[t][v] : acc[t][v];
                }
        }
    }
    __syncthreads();
    float* out = a.part + ((size_t)ci * gridDim.x + blockIdx.x) * TW_PART;
    for (int i = threadIdx.x; i < TW_PART; i += TC_BS) out[i] = tile[i];
}

// Gradients between 16 channels and one: R[c][t] = sum_q big[c][q]
// small[q + tap t].  The first layer: big = g, small = in (R is gw, the sum
// of big the bias).  The head: gw[c][t] = R[c][26 - t] with big = in, small
// = g, and the bias is the sum of small over the tile's own voxels.  Taps
// are the columns (two blocks of 16), K the voxels.
constexpr int TW1_PART = 3 * 256;   // [tap block][c][tap]; block 2: sums of big (columns) or small (rows)
__global__ __launch_bounds__(TC_BS) void k_wgrad1(WgradT a, const float* big, const float* small, int sum_small) {
    __shared__ float tile[TC_HALO];
    __shared__ float bl[16 * TW_GS];
    __shared__ float red[4 * TW1_PART];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    f32x4 acc[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) acc[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    for (int q = blockIdx.x; q < a.t.tiles * a.nb; q += gridDim.x) {
        const int entry = q / a.t.tiles;
        const TcGeo G(a.t, q - entry * a.t.tiles);
        const size_t D3 = (size_t)a.t.D * a.t.D * a.t.D, bo = (size_t)entry * D3;
        __syncthreads();
        tc_stage<1, TC_HALO>(G, small + bo, D3, false, tile);
        {
            const int o = G.at(threadIdx.x);
            const float* p = big + bo * 16 + (o >= 0 ? o : 0);
            float v[16];
#pragma unroll
            for (int c = 0; c < 16; ++c) v[c] = p[c * D3];
#pragma unroll
            for (int c = 0; c < 16; ++c) bl[c * TW_GS + threadIdx.x] = o >= 0 ? v[c] : 0.0f;
        }
        __syncthreads();
        const int nk = (G.nvox() + 3) >> 2;
        const int t0 = lane & 15, t1 = 16 + t0;
        const int o0 = G.tap(t0), o1 = t1 < 27 ? G.tap(t1) : 0, oc = G.tap(13);
        for (int k = w; k < nk; k += TC_BS / 64) {
            const int v = 4 * k + (lane >> 4);
            const int vc = v < G.nvox() ? v : 0;
            const float* tp = tile + G.corner(vc);
            const float bv = bl[t0 * TW_GS + v];
            acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(bv, tp[o0], acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(bv, t1 < 27 ? tp[o1] : 0.0f, acc[1], 0, 0, 0);
            const float sv = (sum_small && v < G.nvox() && G.at(v) >= 0) ? tp[oc] : 0.0f;
            acc[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(sum_small ? 1.0f : bv, sum_small ? sv : 1.0f, acc[2], 0, 0, 0);
        }
    }
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[w * TW1_PART + t * 256 + (4 * (lane >> 4) + v) * 16 + (lane & 15)] = acc[t][v];
    __syncthreads();
    float* out = a.part + (size_t)blockIdx.x * TW1_PART;
    for (int i = threadIdx.x; i < TW1_PART; i += TC_BS)
        out[i] = (red[i] + red[TW1_PART + i]) + (red[2 * TW1_PART + i] + red[3 * TW1_PART + i]);
}

// Sums a partial record over the workgroups (FP64, fixed order: four groups
// of records per entry) and scatters it to the parameter layout.
// mode 0: TW_PART records of input block blockIdx.y; 1: first layer; 2: head.
__global__ __launch_bounds__(256) void k_wgrad_sum(const float* __restrict__ part, int nwg, int rec, int mode, int cin,
                                                   float* __restrict__ gw, float* __restrict__ gb) {
    __shared__ double red[4][64];
    const int e = threadIdx.x & 63, grp = threadIdx.x >> 6, i = blockIdx.x * 64 + e, ci = blockIdx.y;
    const float* p = part + (size_t)ci * nwg * rec + i;   // rec is a multiple of 64
    double s = 0.0;
#pragma unroll 8
    for (int k = grp; k < nwg; k += 4) s += (double)p[(size_t)k * rec];
    red[grp][e] = s;
    __syncthreads();
    if (grp) return;
    const float v = (float)((red[0][e] + red[1][e]) + (red[2][e] + red[3][e]));
    const int t = i >> 8, r = i >> 4 & 15, c = i & 15;
    if (mode == 0) {
        if (t < 27) gw[((size_t)r * cin + ci * 16 + c) * 27 + t] = v;
        else if (c == 0 && ci == 0) gb[r] = v;
        return;
    }
    const int tap = t * 16 + c;   // row r: the channel of `big`
    if (t < 2) {
        if (tap < 27) gw[r * 27 + (mode == 1 ? tap : 26 - tap)] = v;
    } else if (mode == 1 ? c == 0 : (c == 0 && r == 0)) {
        gb[mode == 1 ? r : 0] = v;
    }
}

// average over 2x2x2 blocks: in [BC][D^3] -> out [BC][(D/2)^3]
__global__ void k_avgpool2(const float* __restrict__ in, float* __restrict__ out, int BC, int D) {
    const int h = D / 2;
    const long n = (long)BC * h * h * h;
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int x = i % h, y = (i / h) % h, z = (i / (h * h)) % h;
    const long bc = i / ((long)h * h * h);
    const float* s = in + bc * D * D * D;
    float acc = 0.0f;
    for (int k = 0; k < 8; ++k) acc += s[((2 * z + (k >> 2)) * D + 2 * y + ((k >> 1) & 1)) * D + 2 * x + (k & 1)];
    out[i] = 0.125f * acc;
}

// gradient through avgpool2 plus the skip connection's, masked by the ReLU
// whose output `y` both consumed: out [BC][D^3] = (g / 8 + skip) where y > 0
__global__ void k_avgpool2_bwd(const float* __restrict__ g, const float* __restrict__ skip, const float* __restrict__ y,
                               float* __restrict__ out, int BC, int D) {
    const long n = (long)BC * D * D * D;
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int h = D / 2;
    const int x = i % D, yy = (i / D) % D, z = (i / (D * D)) % D;
    const long bc = i / ((long)D * D * D);
    const float v = 0.125f * g[((bc * h + z / 2) * h + yy / 2) * h + x / 2];
    out[i] = y[i] > 0.0f ? v + skip[i] : 0.0f;
}

// gradient of the nearest x2 upsampling, masked by the ReLU output `y` it
// upsampled: out [BC][h^3] = sum of the 2x2x2 block of g [BC][(2h)^3] where y > 0
__global__ void k_up2_bwd(const float* __restrict__ g, const float* __restrict__ y, float* __restrict__ out, int BC,
                          int h) {
    const int D = 2 * h;
    const long n = (long)BC * h * h * h;
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int x = i % h, yy = (i / h) % h, z = (i / (h * h)) % h;
    const long bc = i / ((long)h * h * h);
    const float* s = g + bc * D * D * D;
    float acc = 0.0f;
    for (int k = 0; k < 8; ++k) acc += s[((2 * z + (k >> 2)) * D + 2 * yy + ((k >> 1) & 1)) * D + 2 * x + (k & 1)];
    out[i] = y[i] > 0.0f ? acc : 0.0f;
}

// MSE: g = 2 (y - t) / n; partial sums of (y - t)^2 per block
constexpr int MS_BS = 256;
__global__ __launch_bounds__(MS_BS) void k_mse(const float* __restrict__ y, const float* __restrict__ t, long n,
                                                float* __restrict__ g, double* __restrict__ part) {
    __shared__ double red[MS_BS / 64];
    const long i = (long)blockIdx.x * MS_BS + threadIdx.x;
    double s = 0.0;
    if (i < n) {
        const float d = y[i] - t[i];
        g[i] = 2.0f * d / (float)n;
        s = (double)d * d;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double tt = 0.0;
        for (int w = 0; w < MS_BS / 64; ++w) tt += red[w];
        part[blockIdx.x] = tt;
    }
}

// out = scale * sum of part (one workgroup; a fixed order)
__global__ __launch_bounds__(MS_BS) void k_sum_to(const double* __restrict__ part, int n, double scale,
                                                  double* __restrict__ out) {
    __shared__ double red[MS_BS / 64];
    double s = 0.0;
    for (int k = threadIdx.x; k < n; k += MS_BS) s += part[k];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) out[0] = ((red[0] + red[1]) + (red[2] + red[3])) * scale;
}

// Adam with bias correction; refreshes the BF16 copy of the parameters.
__global__ void k_adam(float* __restrict__ p, uint16_t* __restrict__ p16, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ g, long n, float lr, float c1, float c2) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = 0.9f * m[i] + 0.1f * gi;
    const float vi = 0.999f * v[i] + 0.001f * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float pn = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + 1e-8f);
    p[i] = pn;
    p16[i] = f32_to_bf16_bits(pn);
}

__global__ void k_to_bf16(const float* __restrict__ p, uint16_t* __restrict__ p16, long n) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p16[i] = f32_to_bf16_bits(p[i]);
}

inline unsigned nblk(long n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

// ---------------------------------------------------------------------------
// host-side network description and launch sequences

const NnLayer kNnLayers[kNnNumLayers] = {
    {"e0a", 1, 16, 1, 0},  {"e0b", 16, 16, 1, 0}, {"e1a", 16, 16, 1, 1}, {"e1b", 16, 16, 1, 1},
    {"e2a", 16, 16, 1, 2}, {"e2b", 16, 16, 1, 2}, {"e3a", 16, 16, 1, 3}, {"e3b", 16, 16, 1, 3},
    {"d2a", 32, 16, 1, 2}, {"d2b", 16, 16, 1, 2}, {"d1a", 32, 16, 1, 1}, {"d1b", 16, 16, 1, 1},
    {"d0a", 32, 16, 1, 0}, {"d0b", 16, 16, 1, 0}, {"head", 16, 1, 0, 0},
};

size_t nn_param_offset(int layer) {
    size_t off = 0;
    for (int k = 0; k < layer; ++k) off += (size_t)kNnLayers[k].co * (kNnLayers[k].ci * 27 + 1);
    return off;
}

size_t nn_param_count() { return nn_param_offset(kNnNumLayers); }

// Workgroups of a weight-gradient launch: two per CU, so that the partial
// records (28 KB each) stay few and their sum short.
static int wgrad_groups(const TcTile& t, int B) {
    const long n = (long)t.tiles * B;
    return n < 512 ? (int)n : 512;
}

// Activation buffers (floats) for batch B at input size D.
NnActLayout nn_act_layout(int B, int D) {
    NnActLayout L{};
    size_t off = 0;
    auto take = [&](size_t n) {
        size_t o = off;
        off += (n + 63) / 64 * 64;
        return o;
    };
    for (int k = 0; k < kNnNumLayers; ++k) {
        const int d = D >> kNnLayers[k].level;
        L.out[k] = take((size_t)B * kNnLayers[k].co * d * d * d);
    }
    for (int lv = 1; lv <= 3; ++lv) {
        const int d = D >> lv;
        L.pool[lv - 1] = take((size_t)B * 16 * d * d * d);
    }
    const size_t big = (size_t)B * 32 * D * D * D;
    L.g0 = take(big);
    L.g1 = take(big);
    L.g2 = take(big);
    L.gskip[0] = take((size_t)B * 16 * D * D * D);
    L.gskip[1] = take((size_t)B * 16 * (D / 2) * (D / 2) * (D / 2));
    L.gskip[2] = take((size_t)B * 16 * (D / 4) * (D / 4) * (D / 4));
    const long npos = (long)B * D * D * D;
    L.wpart = take((size_t)2 * wgrad_groups(tc_tile(D), B) * TW_PART);
    L.wpack = take((size_t)TC_BLOCKS * TC_W);
    L.grad = take(nn_param_count());
    L.mse_part = take(2 * (nblk(npos, MS_BS) + 64));  // doubles: 2 floats each
    L.total_floats = off;
    return L;
}

// The 16-channel blocks of layer k's input given the activation buffers (the
// network input, one channel, is a block of its own); up: upsampled when read.
static int layer_inputs(int k, const float* act, const NnActLayout& L, const float* x, const float* in[2], int up[2]) {
    in[1] = nullptr;
    up[0] = up[1] = 0;
    switch (k) {
        case 0: in[0] = x; return 1;                         // e0a <- input
        case 2: in[0] = act + L.pool[0]; return 1;           // e1a <- pool(s0)
        case 4: in[0] = act + L.pool[1]; return 1;           // e2a <- pool(s1)
        case 6: in[0] = act + L.pool[2]; return 1;           // e3a <- pool(s2)
        case 8:                                              // d2a <- [up(e3b), s2]
        case 10:                                             // d1a <- [up(d2b), s1]
        case 12:                                             // d0a <- [up(d1b), s0]
            in[0] = act + L.out[k - 1];
            up[0] = 1;
            in[1] = act + L.out[13 - k];
            return 2;
        default: in[0] = act + L.out[k - 1]; return 1;       // chain
    }
}

// First packed weight block of layer k (1 .. 13; layers 8, 10 and 12 have two).
static int layer_block(int k) { return k - 1 + (k > 8) + (k > 10) + (k > 12); }

static hipError_t pack_weights(const float* params, const uint16_t* params16, int back, float* out, hipStream_t s) {
    PackT t{};
    for (int k = 1; k < kNnNumLayers - 1; ++k)
        for (int sub = 0; sub < kNnLayers[k].ci / 16; ++sub) {
            const int b = layer_block(k) + sub;
            t.off[b] = (int)nn_param_offset(k);
            t.cin[b] = kNnLayers[k].ci;
            t.sub[b] = sub;
        }
    hipLaunchKernelGGL(k_pack_weights, dim3(TC_BLOCKS, 9), dim3(256), 0, s, t, params, params16, back, out);
    return hipGetLastError();
}

// Layer k's convolution arguments (weights of the layer; FP32 or BF16).
static ConvT layer_conv(int k, const float* params, const uint16_t* params16, const float* wpack, int d) {
    ConvT a{};
    const size_t off = nn_param_offset(k);
    a.w32 = params16 ? nullptr : params + off;
    a.w16 = params16 ? params16 + off : nullptr;
    a.wp = (k > 0 && k < kNnNumLayers - 1) ? wpack + (size_t)layer_block(k) * TC_W : nullptr;
    a.t = tc_tile(d);
    return a;
}

hipError_t nn_forward(const float* params, const uint16_t* params16, const float* x, float* act, const NnActLayout& L,
                      int B, int D, float* y_out, hipStream_t s) {
    NN_CHECK(pack_weights(params, params16, 0, act + L.wpack, s));
    for (int k = 0; k < kNnNumLayers; ++k) {
        const NnLayer& ly = kNnLayers[k];
        const int d = D >> ly.level;
        if (k == 2 || k == 4 || k == 6) {   // the pooled input this layer needs
            hipLaunchKernelGGL(k_avgpool2, dim3(nblk((long)B * 16 * d * d * d, 256)), dim3(256), 0, s,
                               act + L.out[k - 1], act + L.pool[k / 2 - 1], B * 16, 2 * d);
            NN_CHECK(hipGetLastError());
        }
        ConvT a = layer_conv(k, params, params16, act + L.wpack, d);
        a.nci = layer_inputs(k, act, L, x, a.in, a.up);
        a.bias = params + nn_param_offset(k) + (size_t)ly.co * ly.ci * 27;
        a.out[0] = (k == kNnNumLayers - 1 && y_out) ? y_out : act + L.out[k];
        a.relu = ly.relu;
        const dim3 grid(a.t.tiles, B);
        if (ly.ci == 1) hipLaunchKernelGGL(k_conv1, grid, dim3(TC_BS), 0, s, a);
        else if (ly.co == 1) hipLaunchKernelGGL(k_conv_to1, grid, dim3(TC_BS), 0, s, a);
        else hipLaunchKernelGGL(k_conv16<true>, grid, dim3(TC_CBS), 0, s, a);
        NN_CHECK(hipGetLastError());
    }
    return hipSuccess;
}

// Backward pass from g_out (B x D^3) into L.grad (flat, parameter layout).
// `g` is the gradient w.r.t. layer k's output before its ReLU: whoever writes
// a gradient w.r.t. a ReLU's output masks it on the way out.  g_out may be
// L.g2, which is first overwritten when the head is done.
hipError_t nn_backward(const float* params, const uint16_t* params16, const float* x, float* act, const NnActLayout& L,
                       int B, int D, const float* g_out, hipStream_t s) {
    float* grad = act + L.grad;
    const float* g = g_out;
    float* gn = act + L.g0;   // gradient w.r.t. the layer's input (next g)
    float* gf = act + L.g1;
    float* gt = act + L.g2;
    NN_CHECK(pack_weights(params, params16, 1, act + L.wpack, s));
    for (int k = kNnNumLayers - 1; k >= 0; --k) {
        const NnLayer& ly = kNnLayers[k];
        const int d = D >> ly.level;
        ConvT a = layer_conv(k, params, params16, act + L.wpack, d);
        const size_t off = nn_param_offset(k), nw = (size_t)ly.co * ly.ci * 27;
        // weight and bias gradients
        WgradT wg{};
        const int nci = layer_inputs(k, act, L, x, wg.in, wg.up);
        wg.g = g;
        wg.part = act + L.wpart;
        wg.nb = B;
        wg.t = a.t;
        const int nwg = wgrad_groups(a.t, B);
        const bool one = ly.ci == 1 || ly.co == 1;
        if (ly.ci == 1) hipLaunchKernelGGL(k_wgrad1, dim3(nwg), dim3(TC_BS), 0, s, wg, g, wg.in[0], 0);
        else if (ly.co == 1) hipLaunchKernelGGL(k_wgrad1, dim3(nwg), dim3(TC_BS), 0, s, wg, wg.in[0], g, 1);
        else hipLaunchKernelGGL(k_wgrad16, dim3(nwg, nci), dim3(TC_BS), 0, s, wg);
        NN_CHECK(hipGetLastError());
        const int rec = one ? TW1_PART : TW_PART;
        hipLaunchKernelGGL(k_wgrad_sum, dim3(rec / 64, one ? 1 : nci), dim3(256), 0, s, wg.part, nwg, rec,
                           one ? (ly.ci == 1 ? 1 : 2) : 0, ly.ci, grad + off, grad + off + nw);
        NN_CHECK(hipGetLastError());
        if (k == 0) break;  // no gradient needed for the network input
        // gradient w.r.t. the inputs: conv with flipped, transposed weights
        const float* y = act + L.out[k - 1];   // the ReLU output below
        a.flip = 1;
        a.nci = 1;
        a.in[0] = g;
        if (ly.co == 1) {
            a.out[0] = gn;
            a.mask[0] = y;
            hipLaunchKernelGGL(k_conv1, dim3(a.t.tiles, B), dim3(TC_BS), 0, s, a);
        } else if (k == 8 || k == 10 || k == 12) {
            // the upsampled half, summed to the lower level, and the skip half
            a.out[0] = gt;
            a.out[1] = act + L.gskip[(12 - k) / 2];
            hipLaunchKernelGGL(k_conv16<false>, dim3(a.t.tiles, B, 2), dim3(TC_CBS), 0, s, a);
            NN_CHECK(hipGetLastError());
            hipLaunchKernelGGL(k_up2_bwd, dim3(nblk((long)B * 16 * (d / 2) * (d / 2) * (d / 2), 256)), dim3(256), 0, s,
                               gt, y, gn, B * 16, d / 2);
        } else if (k == 2 || k == 4 || k == 6) {
            // through the average pool, plus the skip gradient of this level
            a.out[0] = gt;
            hipLaunchKernelGGL(k_conv16<false>, dim3(a.t.tiles, B), dim3(TC_CBS), 0, s, a);
            NN_CHECK(hipGetLastError());
            hipLaunchKernelGGL(k_avgpool2_bwd, dim3(nblk((long)B * 16 * 8 * d * d * d, 256)), dim3(256), 0, s, gt,
                               act + L.gskip[k / 2 - 1], y, gn, B * 16, 2 * d);
        } else {
            a.out[0] = gn;
            a.mask[0] = y;
            hipLaunchKernelGGL(k_conv16<false>, dim3(a.t.tiles, B), dim3(TC_CBS), 0, s, a);
        }
        NN_CHECK(hipGetLastError());
        g = gn;
        float* t = gn;
        gn = gf;
        gf = t;
    }
    return hipSuccess;
}

hipError_t nn_mse(const float* y, const float* t, long n, float* g, double* part, double* loss_dev, hipStream_t s) {
    const unsigned nb = nblk(n, MS_BS);
    hipLaunchKernelGGL(k_mse, dim3(nb), dim3(MS_BS), 0, s, y, t, n, g, part);
    NN_CHECK(hipGetLastError());
    hipLaunchKernelGGL(k_sum_to, dim3(1), dim3(MS_BS), 0, s, part, (int)nb, 1.0 / (double)n, loss_dev);
    return hipGetLastError();
}

hipError_t nn_adam(float* p, uint16_t* p16, float* m, float* v, const float* g, long n, float lr, int step,
                   hipStream_t s) {
    const float c1 = 1.0f - powf(0.9f, (float)step), c2 = 1.0f - powf(0.999f, (float)step);
    hipLaunchKernelGGL(k_adam, dim3(nblk(n, 256)), dim3(256), 0, s, p, p16, m, v, g, n, lr, c1, c2);
    return hipGetLastError();
}

hipError_t nn_to_bf16(const float* p, uint16_t* p16, long n, hipStream_t s) {
    hipLaunchKernelGGL(k_to_bf16, dim3(nblk(n, 256)), dim3(256), 0, s, p, p16, n);
    return hipGetLastError();
}
