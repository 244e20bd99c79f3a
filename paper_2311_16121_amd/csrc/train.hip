// Training-time decode for gfx950: forward and backward through the simulated
// BC6H decompression of Section 4.2 (eqs. 6-8), the trilinear filter (eqs. 9
// and 10) and the ReLU MLP (eq. 3).
//
//   k_train_texels    block parameters -> texel images (r, g, b, 0) per level
//   k_train_forward_mfma  queries -> G(u, v, s), one lane per query, the MLP
//                     on the matrix cores
//   k_train_bin_*     the backward's samples sorted by position (counting
//                     sort over a grid of cells on the wrapped (u, v))
//   k_train_backward  queries, dL/dG -> dL/d features per sample and dL/d MLP
//                     parameters (sums on the matrix cores, one atomic per
//                     parameter and workgroup)
//   k_train_scatter   dL/d features -> dL/d texel, one workgroup per pyramid
//                     and region of cells: fixed-point sums in LDS windows over
//                     the region's footprint, then one float atomic per touched
//                     texel channel
//   k_train_blocks    dL/d texel -> dL/d endpoints, dL/d indices (one lane
//                     per block row, sums over a block's four lanes)
//
// A texel of subset sigma blends the endpoint pair (e_{2 sigma}, e_{2 sigma+1})
// with index x. Continuous mode: y = a ((2^16 e_A + 2^15)/2^6 + x (2^16 (e_B -
// e_A))/2^6), w = eq. (8) of y. Straight-through mode: w is the format's exact
// decode of the rounded endpoints and index (i = rint(7 x)); the derivatives are
// those of the continuous chain at the rounded point (x = w_i / 64), with the
// rounding taken as the identity and eq. (8)'s slope at the decoded bits.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "bc6h_device.hpp"
#include "frame_kernels.hpp"
#include "train.hpp"
#include "unpack_device.hpp"

namespace bcf {
namespace {

constexpr float kA = 31.0f / 64.0f;      // a of eq. (6) for the unsigned format
constexpr int kTrainThreads = 256;

// What the backward accumulates into: the texel gradients (n_texels is a
// multiple of 4), the parameter gradients and the sort's cell counts.
__global__ void __launch_bounds__(256) k_train_clear(TrainDesc d)
{
    const uint32_t tid = blockIdx.x * blockDim.x + threadIdx.x, step = gridDim.x * blockDim.x;
    float4 *g = reinterpret_cast<float4 *>(d.g_texels);
    for (uint32_t i = tid; i < d.n_texels / 4u * 3u; i += step) g[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    for (uint32_t i = tid; i < d.n_params; i += step) d.g_params[i] = 0.0f;
    for (uint32_t i = tid; i < kTrainBins; i += step) d.bin_count[i] = 0u;
}

__device__ __forceinline__ void wave_sync_lds()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------------------
// one texel channel

struct TexelChan {
    float w;              // texel value
    float slope;          // dw/dy of eq. (8)
    float dy_da, dy_db;   // dy/d e_A, dy/d e_B
    float dy_dx;          // dy/d x
};

// h(y) = max(floor((y - 1) / 1024) - 1, 0) of eq. (8) for integer y >= 0
__device__ __forceinline__ int h_of_bits(uint32_t y)
{
    const int k = y ? (int)((y - 1u) >> 10) - 1 : 0;
    return k > 0 ? k : 0;
}

template <bool STE>
__device__ __forceinline__ TexelChan texel_chan(float ea, float eb, float x)
{
    TexelChan r;
    if (!STE) {
        // (2^16 e + 2^15) / 2^6 = 1024 e + 512, exact in binary32 for e in [0, 64)
        const float abar = fmaf(1024.0f, ea, 512.0f);
        const float bbar = fmaf(1024.0f, eb, 512.0f);
        const float y = kA * fmaf(x, bbar - abar, abar);
        const float h = fmaxf(floorf((y - 1.0f) * (1.0f / 1024.0f)) - 1.0f, 0.0f);
        r.w = ldexpf(y * (1.0f / 1024.0f) - h, (int)h - 14);
        r.slope = ldexpf(1.0f, (int)h - 24);
        r.dy_da = kA * 1024.0f * (1.0f - x);
        r.dy_db = kA * 1024.0f * x;
        r.dy_dx = kA * (bbar - abar);
    } else {
        // fmaxf before fminf maps NaN to 0
        const float qa = fminf(fmaxf(rintf(ea), 0.0f), 63.0f);
        const float qb = fminf(fmaxf(rintf(eb), 0.0f), 63.0f);
        const uint32_t i = (uint32_t)fminf(fmaxf(rintf(7.0f * x), 0.0f), 7.0f);
        const int32_t wt = (int32_t)((i * 585u + 32u) >> 6);       // round(64 i / 7)
        const int32_t A = unquantize<false>((int32_t)qa, 6);
        const int32_t B = unquantize<false>((int32_t)qb, 6);
        const int32_t v = ((64 - wt) * A + wt * B + 32) >> 6;
        const uint32_t y = ((uint32_t)v * 31u) >> 6;
        r.w = (float)__builtin_bit_cast(_Float16, (uint16_t)y);
        r.slope = ldexpf(1.0f, h_of_bits(y) - 24);
        const float xs = (float)wt * (1.0f / 64.0f);
        r.dy_da = kA * 1024.0f * (1.0f - xs);
        r.dy_db = kA * 1024.0f * xs;
        r.dy_dx = kA * 1024.0f * (qb - qa);
    }
    return r;
}

// Where texel t of joint block gb lives: pyramid, block within it, level and
// position; false for the texels a level below 4x4 does not have.
struct TexelSite {
    uint32_t ti, b, x, y, tex;      // tex: texel index in the images
    uint32_t wl;                    // the level's width
    bool valid;
};

__device__ __forceinline__ TexelSite texel_site(const TrainDesc &d, uint32_t gb, uint32_t t)
{
    TexelSite s;
    uint32_t ti = 0;
    while (ti + 1 < d.n_tex && gb >= d.blk_base[ti + 1]) ++ti;
    const TrainTexDesc &tx = d.tex[ti];
    const uint32_t b = gb - d.blk_base[ti];
    uint32_t l = 0;
    while (l + 1 < tx.levels && b >= tx.blk_off[l + 1]) ++l;
    const uint32_t wl = max(tx.w >> l, 1u), hl = max(tx.h >> l, 1u);
    const uint32_t bxn = (wl + 3u) >> 2;          // a power of two, as the level width is
    const uint32_t lb = b - tx.blk_off[l];
    s.ti = ti;
    s.b = b;
    s.x = (lb & (bxn - 1u)) * 4u + (t & 3u);
    s.y = (lb >> __builtin_ctz(bxn)) * 4u + (t >> 2);
    s.valid = s.x < wl && s.y < hl;
    s.tex = tx.tex_off[l] + s.y * wl + s.x;
    s.wl = wl;
    return s;
}

// One lane per block row: its four texels (a level narrower than 4 texels
// keeps the left ones), the block's endpoints and partition read once.
template <bool STE>
__global__ void __launch_bounds__(kTrainThreads) k_train_texels(TrainDesc d)
{
    const uint32_t total = d.blk_base[d.n_tex] * 4u;
    for (uint32_t g = blockIdx.x * blockDim.x + threadIdx.x; g < total; g += gridDim.x * blockDim.x) {
        const uint32_t r = g & 3u;
        const TexelSite s = texel_site(d, g >> 2, 4u * r);
        if (!s.valid) continue;
        const TrainTexDesc &tx = d.tex[s.ti];
        // partition ids are taken modulo 32
        const uint32_t pmask = kTable[kPartitionRow + (tx.partitions[s.b] & 31u)];
        float e[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) e[k] = tx.endpoints[12u * s.b + k];
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
            if (s.x + i >= s.wl) break;
            const uint32_t t = 4u * r + i, sub = (pmask >> t) & 1u;
            const float x = tx.indices[16u * s.b + t];
            float w[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) w[c] = texel_chan<STE>(sub ? e[6 + c] : e[c], sub ? e[9 + c] : e[3 + c], x).w;
            d.texels[s.tex + i] = make_float4(w[0], w[1], w[2], 0.0f);
        }
    }
}

// The straight-through texels of pyramids of one geometry, which are halves, to
// the decode's packed scratch (filter_device.hpp): lane = 4 * block position +
// pyramid, the block's palette and slots through LDS as in the unpack, so that
// whole block rows are stored and a footprint row of all pyramids is three
// 16-byte loads. Pyramids past n_tex leave zeros. ALIGNED: every pyramid's
// endpoints and indices start 16-byte aligned.
// Bound by the parameters' reads and the texels' writes (39 and 34 MB at
// 4 x 1024^2); the float images it replaces took 90 MB and a lane per block row.
template <bool ALIGNED>
__global__ void __launch_bounds__(kTrainThreads) k_train_texels_packed(TrainDesc d)
{
    __shared__ uint2 palette[16][256];
    __shared__ uint2 slots[256];
    const TrainTexDesc &t0 = d.tex[0];
    // this workgroup's level and chunk of 64 block positions
    uint32_t l = 0, chunk = blockIdx.x;
    uint32_t n_blk;
    for (;; ++l) {
        n_blk = ((max(t0.w >> l, 1u) + 3u) >> 2) * ((max(t0.h >> l, 1u) + 3u) >> 2);
        const uint32_t chunks = (n_blk + 63u) >> 6;
        if (chunk < chunks) break;
        chunk -= chunks;
    }
    const uint32_t pyr = threadIdx.x & 3u, bi = chunk * 64u + (threadIdx.x >> 2);
    uint32_t pal[16][2];
    uint32_t s0 = 0, s1 = 0;
    if (bi < n_blk && pyr < d.n_tex) {
        const float *ep = pyr == 0 ? d.tex[0].endpoints : pyr == 1 ? d.tex[1].endpoints : pyr == 2 ? d.tex[2].endpoints : d.tex[3].endpoints;
        const float *xp = pyr == 0 ? d.tex[0].indices : pyr == 1 ? d.tex[1].indices : pyr == 2 ? d.tex[2].indices : d.tex[3].indices;
        const uint8_t *pp = pyr == 0 ? d.tex[0].partitions : pyr == 1 ? d.tex[1].partitions : pyr == 2 ? d.tex[2].partitions : d.tex[3].partitions;
        const size_t b = (size_t)t0.blk_off[l] + bi;
        float e[12], x[16];
        if (ALIGNED) {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const float4 v = reinterpret_cast<const float4 *>(ep + 12u * b)[k];
                e[4 * k] = v.x, e[4 * k + 1] = v.y, e[4 * k + 2] = v.z, e[4 * k + 3] = v.w;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float4 v = reinterpret_cast<const float4 *>(xp + 16u * b)[k];
                x[4 * k] = v.x, x[4 * k + 1] = v.y, x[4 * k + 2] = v.z, x[4 * k + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int k = 0; k < 12; ++k) e[k] = ep[12u * b + k];
#pragma unroll
            for (int k = 0; k < 16; ++k) x[k] = xp[16u * b + k];
        }
        // the exported block: texel_chan's rounding of endpoints and indices
        // (fmaxf before fminf maps NaN to 0), one 8-entry palette per subset
        Bc6hHeader h;
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const float qa = fminf(fmaxf(rintf(e[6 * sub + c]), 0.0f), 63.0f);
                const float qb = fminf(fmaxf(rintf(e[6 * sub + 3 + c]), 0.0f), 63.0f);
                const int32_t A = unquantize<false>((int32_t)qa, 6), B = unquantize<false>((int32_t)qb, 6);
                h.base[sub][c] = 64 * A + 32;
                h.diff[sub][c] = B - A;
            }
        h.ib = 3;
        h.valid = 1;
        bc6h_palette<false>(h, pal);
        const uint32_t part = pp[b] & 31u;           // ids are taken modulo 32
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            s0 |= (uint32_t)fminf(fmaxf(rintf(7.0f * x[t]), 0.0f), 7.0f) << (4 * t);
            s1 |= (uint32_t)fminf(fmaxf(rintf(7.0f * x[8 + t]), 0.0f), 7.0f) << (4 * t);
        }
        s0 |= kTable[kSpreadRow + 2 * part];
        s1 |= kTable[kSpreadRow + 2 * part + 1];
    } else {
#pragma unroll
        for (int j = 0; j < 16; ++j) pal[j][0] = pal[j][1] = 0u;
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) palette[j][threadIdx.x] = make_uint2(pal[j][0], pal[j][1]);
    slots[threadIdx.x] = make_uint2(s0, s1);
    __syncthreads();
    store_positions<false>(d.packed + 6 * (size_t)d.pos_off[l], max(t0.w >> l, 1u), max(t0.h >> l, 1u),
                           chunk * 64u + ((threadIdx.x & ~63u) >> 2), n_blk, palette, slots);
}

// The continuous texels of pyramids of one geometry, in floats: positions of 48
// bytes. Lane = 4 * block row + pyramid, so that a quad fills a position and the
// four stores of a row fill its lines; pyramids past n_tex leave zeros.
__global__ void __launch_bounds__(kTrainThreads) k_train_texels_floats(TrainDesc d)
{
    const uint32_t total = (d.tex[0].n_blocks + 15u) / 16u * 256u;
    for (uint32_t g = blockIdx.x * blockDim.x + threadIdx.x; g < total; g += gridDim.x * blockDim.x) {
        // a wave's 16 positions of one block row of 16 blocks (rows outermost,
        // so that consecutive quads are consecutive blocks)
        const uint32_t pyr = g & 3u, r = (g >> 6) & 3u, b = (g >> 8) * 16u + ((g >> 2) & 15u);
        if (b >= d.tex[0].n_blocks) continue;
        const TexelSite s = texel_site(d, b, 4u * r);          // pyramid 0's site serves all
        if (!s.valid) continue;
        uint32_t l = 0;
        while (l + 1 < d.tex[0].levels && b >= d.tex[0].blk_off[l + 1]) ++l;
        float w[4][3];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int c = 0; c < 3; ++c) w[i][c] = 0.0f;
        if (pyr < d.n_tex) {
            const float *ep = pyr == 0 ? d.tex[0].endpoints : pyr == 1 ? d.tex[1].endpoints : pyr == 2 ? d.tex[2].endpoints : d.tex[3].endpoints;
            const float *xp = pyr == 0 ? d.tex[0].indices : pyr == 1 ? d.tex[1].indices : pyr == 2 ? d.tex[2].indices : d.tex[3].indices;
            const uint8_t *pp = pyr == 0 ? d.tex[0].partitions : pyr == 1 ? d.tex[1].partitions : pyr == 2 ? d.tex[2].partitions : d.tex[3].partitions;
            const uint32_t pmask = kTable[kPartitionRow + (pp[b] & 31u)] >> (4u * r);   // ids are taken modulo 32
            float e[12];
#pragma unroll
            for (int k = 0; k < 12; ++k) e[k] = ep[12u * (size_t)b + k];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool sub = (pmask >> i) & 1u;
                const float x = xp[16u * (size_t)b + 4u * r + i];
#pragma unroll
                for (int c = 0; c < 3; ++c) w[i][c] = texel_chan<false>(sub ? e[6 + c] : e[c], sub ? e[9 + c] : e[3 + c], x).w;
            }
        }
        float *row = reinterpret_cast<float *>(d.packed) +
                     12u * ((size_t)d.pos_off[l] + (size_t)s.y * row_pitch(s.wl)) + 3u * pyr;
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) {
            if (s.x + i >= s.wl) break;
#pragma unroll
            for (int c = 0; c < 3; ++c) row[12u * (s.x + i) + c] = w[i][c];
        }
        if (s.x == 0) {                          // position w repeats position 0
#pragma unroll
            for (int c = 0; c < 3; ++c) row[12u * s.wl + c] = w[0][c];
        }
    }
}

// Sum over the four lanes of a quad, in each of them. (bound_ctrl lets the move
// fold into the add; every source lane exists.)
template <int CTRL>
__device__ __forceinline__ float dpp_move(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, true));
}

__device__ __forceinline__ float quad_sum(float v)
{
    v += dpp_move<0xB1>(v);       // quad_perm [1, 0, 3, 2]
    return v + dpp_move<0x4E>(v);   // quad_perm [2, 3, 0, 1]
}

// dL/d texel -> dL/d endpoints and indices: one lane per block row, a block's
// four rows in a quad. ALIGNED: the parameters and their gradients start
// 16-byte aligned (the texel gradients' rows of four always do), so a lane's
// four indices and their gradients are one access each.
// Bound by VALU instructions (rounding, slopes and the sums) over 145 MB at
// 4 x 1024^2; one lane per texel (endpoints rounded 16 times a block, twelve
// 16-lane sums a texel) took 66 us.
template <bool STE, bool ALIGNED>
__global__ void __launch_bounds__(kTrainThreads) k_train_blocks(TrainDesc d)
{
    // total is a multiple of 4: a quad enters and leaves the loop together
    const uint32_t total = d.blk_base[d.n_tex] * 4u;
    for (uint32_t g = blockIdx.x * blockDim.x + threadIdx.x; g < total; g += gridDim.x * blockDim.x) {
        const uint32_t r = g & 3u;
        const TexelSite s = texel_site(d, g >> 2, 4u * r);
        const TrainTexDesc &tx = d.tex[s.ti];
        // partition ids are taken modulo 32
        const uint32_t pmask = kTable[kPartitionRow + (tx.partitions[s.b] & 31u)] >> (4u * r);
        const float *ep = tx.endpoints + 12u * s.b, *xp = tx.indices + 16u * s.b + 4u * r;
        float e[12], x[4], gt[12];
        if (ALIGNED) {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const float4 v = reinterpret_cast<const float4 *>(ep)[k];
                e[4 * k] = v.x, e[4 * k + 1] = v.y, e[4 * k + 2] = v.z, e[4 * k + 3] = v.w;
            }
            const float4 v = *reinterpret_cast<const float4 *>(xp);
            x[0] = v.x, x[1] = v.y, x[2] = v.z, x[3] = v.w;
        } else {
#pragma unroll
            for (int k = 0; k < 12; ++k) e[k] = ep[k];
#pragma unroll
            for (int k = 0; k < 4; ++k) x[k] = xp[k];
        }
        const float *gp = d.g_texels + 3u * s.tex;
        if (s.valid && s.wl >= 4u) {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const float4 v = reinterpret_cast<const float4 *>(gp)[k];
                gt[4 * k] = v.x, gt[4 * k + 1] = v.y, gt[4 * k + 2] = v.z, gt[4 * k + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int k = 0; k < 12; ++k) gt[k] = s.valid && (uint32_t)k < 3u * s.wl ? gp[k] : 0.0f;
        }
        float sum[4][3], gx[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int c = 0; c < 3; ++c) sum[j][c] = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool sub = (pmask >> i) & 1u;
            gx[i] = 0.0f;
            // not as a product with a zero gradient: the index of a texel that
            // the level does not have, and a subset's endpoints without a
            // texel, may hold anything
            if (!s.valid || (uint32_t)i >= s.wl) continue;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const TexelChan t = texel_chan<STE>(sub ? e[6 + c] : e[c], sub ? e[9 + c] : e[3 + c], x[i]);
                const float gy = gt[3 * i + c] * t.slope;
                gx[i] = fmaf(gy, t.dy_dx, gx[i]);
                const float ga = gy * t.dy_da, gb = gy * t.dy_db;
                sum[0][c] += sub ? 0.0f : ga;
                sum[1][c] += sub ? 0.0f : gb;
                sum[2][c] += sub ? ga : 0.0f;
                sum[3][c] += sub ? gb : 0.0f;
            }
        }
        float *xo = tx.g_indices + 16u * s.b + 4u * r;
        if (ALIGNED) {
            *reinterpret_cast<float4 *>(xo) = make_float4(gx[0], gx[1], gx[2], gx[3]);
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) xo[k] = gx[k];
        }
        // the quad's lane r writes endpoint r
        float out[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const float v = quad_sum(sum[j][c]);
                out[c] = (int)r == j ? v : out[c];
            }
#pragma unroll
        for (int c = 0; c < 3; ++c) tx.g_endpoints[12u * s.b + 3u * r + c] = out[c];
    }
}

// ---------------------------------------------------------------------------
// queries

// Per pyramid and level, for the query kernels' LDS: x = level width,
// y = level height, z = first texel of the level in the images, w = first
// position of the level in the packed scratch. A level picked
// per query indexes it; indexing the descriptor's arrays instead makes the
// compiler hold every level's values in registers across the query loop.
typedef uint4 TrainLevelLut[kMaxTextures][kMaxLevels];

// Every thread of the workgroup takes part; the caller synchronises.
__device__ __forceinline__ void load_level_lut(const TrainDesc &d, TrainLevelLut &lut)
{
    for (uint32_t e = threadIdx.x; e < (uint32_t)(kMaxTextures * kMaxLevels); e += blockDim.x) {
        const uint32_t ti = e / kMaxLevels, l = e % kMaxLevels;
        const TrainTexDesc &tx = d.tex[ti < d.n_tex ? ti : 0u];
        lut[ti][l] = l < tx.levels ? make_uint4(max(tx.w >> l, 1u), max(tx.h >> l, 1u), tx.tex_off[l], d.pos_off[l])
                                   : make_uint4(1u, 1u, 0u, 0u);
    }
}

// The four bilinear taps of wrapped (uf, vf) on one level (e = its LUT entry:
// width, height, first texel) and their weights times the level weight lw:
// columns xa, xb = xa + 1 and rows ya, yb = ya + 1 (wrapped); w[] in the order
// (ya, xa), (ya, xb), (yb, xa), (yb, xb).
struct LevelTaps {
    uint32_t xa, xb, ya, yb;
    float w[4];
};

__device__ __forceinline__ LevelTaps level_taps(uint4 e, float uf, float vf, float lw)
{
    LevelTaps r;
    const uint32_t wl = e.x, hl = e.y;
    const float x = fmaf(uf, (float)wl, -0.5f), y = fmaf(vf, (float)hl, -0.5f);
    const float x0 = floorf(x), y0 = floorf(y);
    const float fx = x - x0, fy = y - y0;
    r.xa = (uint32_t)(int)x0 & (wl - 1u);
    r.xb = (r.xa + 1u) & (wl - 1u);
    r.ya = (uint32_t)(int)y0 & (hl - 1u);
    r.yb = (r.ya + 1u) & (hl - 1u);
    r.w[0] = lw * (1.0f - fx) * (1.0f - fy);
    r.w[1] = lw * fx * (1.0f - fy);
    r.w[2] = lw * (1.0f - fx) * fy;
    r.w[3] = lw * fx * fy;
    return r;
}

// The 32 taps of a query (4 pyramids x 2 levels x 4 texels): texel index and
// weight (bilinear times trilinear); pyramids past n_tex get weight 0.
__device__ __forceinline__ void taps(const TrainDesc &d, const TrainLevelLut &lut, float u, float v, float s,
                                     uint32_t idx[32], float wt[32])
{
    const float uf = u - floorf(u), vf = v - floorf(v);          // wrap addressing
#pragma unroll
    for (int ti = 0; ti < kMaxTextures; ++ti) {
        const TrainTexDesc &tx = d.tex[ti < (int)d.n_tex ? ti : 0];
        const uint32_t slot = ti < (int)d.n_tex ? (uint32_t)ti : 0u;
        const float si = fminf(fmaxf(s + tx.bias, 0.0f), (float)(tx.levels - 1));   // NaN -> 0
        const uint32_t l0 = (uint32_t)floorf(si);
        const uint32_t l1 = min(l0 + 1u, tx.levels - 1u);
        const float lam = si - (float)l0;
        const float on = ti < (int)d.n_tex ? 1.0f : 0.0f;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const uint32_t l = k ? l1 : l0;
            const float lw = on * (k ? lam : 1.0f - lam);
            const uint4 e = lut[slot][l];
            const LevelTaps lt = level_taps(e, uf, vf, lw);
            const uint32_t wl = e.x, base = e.z;
            const int o = 8 * ti + 4 * k;
            idx[o + 0] = base + lt.ya * wl + lt.xa;
            idx[o + 1] = base + lt.ya * wl + lt.xb;
            idx[o + 2] = base + lt.yb * wl + lt.xa;
            idx[o + 3] = base + lt.yb * wl + lt.xb;
#pragma unroll
            for (int i = 0; i < 4; ++i) wt[o + i] = lt.w[i];
        }
    }
}

// z of a query: the filtered pyramids, from their images (PACK 0) or from the
// packed positions of pyramids of one geometry, halves (1) or floats (2): the
// same sums in the same order; pyramids past n_tex hold zeros.
template <int PACK>
__device__ __forceinline__ void features(const TrainDesc &d, const TrainLevelLut &lut, float u, float v, float s,
                                         float z[12])
{
    if constexpr (PACK != 0) {
        constexpr uint32_t kUnit = PACK == 1 ? 24u : 48u;            // bytes a position
        constexpr int kLoads = 2 * (int)kUnit / 16;                  // of 16 bytes, per footprint row
        const float uf = u - floorf(u), vf = v - floorf(v);          // wrap addressing
        const uint32_t levels = d.tex[0].levels;
        const float si = fminf(fmaxf(s + d.tex[0].bias, 0.0f), (float)(levels - 1));   // NaN -> 0
        const uint32_t l0 = (uint32_t)floorf(si);
        const float lam = si - (float)l0;
        const __amdgpu_buffer_rsrc_t rs = make_rsrc(d.packed, d.packed_bytes);
        texel_pair q[2][2][kLoads];
        LevelTaps lt[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const uint4 e = lut[0][k ? min(l0 + 1u, levels - 1u) : l0];
            lt[k] = level_taps(e, uf, vf, k ? lam : 1.0f - lam);
            // columns xa and xa + 1 (column w repeats column 0)
            const uint32_t pitch = row_pitch(e.x);
            const uint32_t o[2] = {kUnit * (e.w + lt[k].ya * pitch + lt[k].xa),
                                   kUnit * (e.w + lt[k].yb * pitch + lt[k].xa)};
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int j = 0; j < kLoads; ++j)
                    q[k][r][j] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(o[r] + 16u * j), 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 12; ++i) z[i] = 0.0f;
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int i = 0; i < 12; ++i) {       // i = 3 t + c: values i (xa) and 12 + i (xa + 1)
                auto value = [&](int row, int j) -> float {
                    if constexpr (PACK == 1) return packed_half(q[k][row], j);
                    const uint32_t bits = q[k][row][j >> 2][j & 3];
                    return __uint_as_float(bits);
                };
                z[i] = fmaf(lt[k].w[0], value(0, i), z[i]);
                z[i] = fmaf(lt[k].w[1], value(0, 12 + i), z[i]);
                z[i] = fmaf(lt[k].w[2], value(1, i), z[i]);
                z[i] = fmaf(lt[k].w[3], value(1, 12 + i), z[i]);
            }
    } else {
        uint32_t idx[32];
        float wt[32];
        taps(d, lut, u, v, s, idx, wt);
#pragma unroll
        for (int i = 0; i < 12; ++i) z[i] = 0.0f;
#pragma unroll
        for (int k = 0; k < 32; ++k) {
            const float4 tv = d.texels[idx[k]];
            const int t = k / 8;
            z[3 * t + 0] = fmaf(wt[k], tv.x, z[3 * t + 0]);
            z[3 * t + 1] = fmaf(wt[k], tv.y, z[3 * t + 1]);
            z[3 * t + 2] = fmaf(wt[k], tv.z, z[3 * t + 2]);
        }
    }
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// The forward with the MLP on the matrix cores (fp32 16x16x4 MFMAs, the
// decode kernels' operand layout, prepared from the parameters per call): a
// wave's 64 queries' features pass through LDS into the MFMA B layout, the
// outputs come back through LDS to each query's lane.
// Waves per SIMD the forward's registers are laid out for (the filter's loads
// in flight against the waves beside it; 0: the compiler's choice). Measured,
// 2^20 samples, the compiler's choice -> this: halves 12-32-32-10 83 -> 78 us,
// 12-16-16-10 66 -> 66, three hidden layers of 32 or 16 91 and 68 (4: 91, 67);
// floats 126 -> 106 and 109 -> 101, one layer of 16 114 -> 100, of 32 96 -> 101,
// three of 32 128 (3: 127), of 16 111 (3: 101). The images take the compiler's:
// one pyramid, three layers of 16 91 (3: 129, 4: 100), of 32 113 (3: 124, 4:
// 124); four sizes 100 (128, 114) and 120 (135, 131).
constexpr int forward_waves(int NH, int PACK)
{
    return NH == 3 || PACK == 0 ? 0 : PACK == 1 ? 4 : 3;
}

template <int H, int NH, int PACK>
__global__ void __attribute__((amdgpu_waves_per_eu(forward_waves(NH, PACK) ? forward_waves(NH, PACK) : 1,
                                                   forward_waves(NH, PACK) ? forward_waves(NH, PACK) : 8)))
__launch_bounds__(kTrainThreads) k_train_forward_mfma(TrainDesc d, const float *queries, uint32_t n,
                                                                      float *out)
{
    constexpr int kWaves = kTrainThreads / 64;
    __shared__ TrainLevelLut lut;
    __shared__ float4_t stage[kWaves][64 * kMaxOut / 4];     // features, then output rows
    load_level_lut(d, lut);
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63u, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t c = d.dims[NH + 1];
    MfmaMlp<MLP_MFMA_F32, H, NH> mlp;
    mlp.load(d.ops_ws, d.ops, lane);
    float *st = reinterpret_cast<float *>(&stage[wv][0]);
    float4_t (*feats)[4] = reinterpret_cast<float4_t (*)[4]>(&stage[wv][0]);
    const uint32_t n_chunks = (n + 63u) / 64u;
    const bool wide = ((uintptr_t)out & 15u) == 0;
    for (uint32_t ch = blockIdx.x * kWaves + wv; ch < n_chunks; ch += gridDim.x * kWaves) {
        const uint32_t q = ch * 64u + lane;
        const bool live = q < n;
        float z[12];
        features<PACK>(d, lut, live ? queries[3u * q] : 0.0f, live ? queries[3u * q + 1u] : 0.0f,
                 live ? queries[3u * q + 2u] : 0.0f, z);
        mlp_stage<false, MLP_MFMA_F32, H, NH>(z, mlp, feats, st, c, lane);
        // the chunk's rows are contiguous: 16-byte stores where they may be
        const uint32_t floats = min(64u, n - ch * 64u) * c;
        float *dst = out + (size_t)ch * 64u * c;
        if (wide && floats == 64u * c) {
            for (uint32_t k = lane; k < 16u * c; k += 64u)
                reinterpret_cast<float4_t *>(dst)[k] = reinterpret_cast<const float4_t *>(st)[k];
        } else {
            for (uint32_t k = lane; k < floats; k += 64u) dst[k] = st[k];
        }
        wave_lds_sync();                              // the stage is rewritten by the next chunk
    }
}

// ---------------------------------------------------------------------------
// the backward's sample order
//
// Texel-gradient float atomics on random lines of levels larger than the
// caches each fetch and write back a whole line. Taking the samples cell by
// cell (and each XCD a contiguous run of cells) lets the samples that share
// gradient lines update them while the lines sit in one L2.

constexpr int kBinThreads = 1024;
// Samples a thread of the count and placement kernels takes. Eight from 3 * 2^16
// samples on: a workgroup's histogram covers 8K of them, so that fewer cells of
// it reach memory (one atomic per touched cell and workgroup). Below, one: the
// workgroups would be too few. Backward of 4 x 1024^2, one and eight: 2^16 147
// and 155 us, 2^17 172 and 177, 2^18 210 and 204, 3 * 2^17 247 and 234, 2^20 388
// and 349; 4 x 256^2 and one of 1024^2 cross between 2^17 and 2^18 too. (2^20
// samples, the two kernels alone: 24 + 35 us with one, 10 + 17 with eight, 14 +
// 21 with sixteen.)
constexpr uint32_t kBinMany = 3u << 16;
constexpr uint32_t bin_per_thread(uint32_t n) { return n >= kBinMany ? 8u : 1u; }

// A query's cell: its wrapped (u, v) on the kTrainBinSide grid (NaN and
// infinities land in cell 0), numbered along a Z-order curve.
__device__ __forceinline__ uint32_t bin_of(float u, float v)
{
    const float uf = u - floorf(u), vf = v - floorf(v);
    const float side = (float)kTrainBinSide;
    const uint32_t cx = (uint32_t)fminf(fmaxf(uf * side, 0.0f), side - 1.0f);
    const uint32_t cy = (uint32_t)fminf(fmaxf(vf * side, 0.0f), side - 1.0f);
    uint32_t z = 0;
#pragma unroll
    for (uint32_t b = 0; b < 6; ++b) z |= ((cx >> b) & 1u) << (2 * b) | ((cy >> b) & 1u) << (2 * b + 1);
    return z;
}

// count[cell] += samples of the cell; PER * kBinThreads samples per workgroup
// (sample (blockIdx * PER + k) * kBinThreads + threadIdx), a histogram in LDS
template <uint32_t PER>
__global__ void __launch_bounds__(kBinThreads) k_train_bin_count(const float *queries, uint32_t n, uint32_t *count)
{
    __shared__ uint32_t hist[kTrainBins];
    for (uint32_t b = threadIdx.x; b < kTrainBins; b += kBinThreads) hist[b] = 0u;
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
        const uint32_t i = (blockIdx.x * PER + k) * kBinThreads + threadIdx.x;
        if (i < n) atomicAdd(&hist[bin_of(queries[3u * i], queries[3u * i + 1u])], 1u);
    }
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < kTrainBins; b += kBinThreads)
        if (hist[b]) atomicAdd(&count[b], hist[b]);
}

// next[cell] = samples of the cells before it (one workgroup, 4 cells a
// thread); leaves the counts clear for the next batch of samples
__global__ void __launch_bounds__(kBinThreads) k_train_bin_scan(uint32_t *count, uint32_t *next)
{
    static_assert(kTrainBins == 4 * kBinThreads, "four cells a thread");
    __shared__ uint32_t wave_sum[kBinThreads / 64];
    const uint32_t t = threadIdx.x, lane = t & 63u, wv = t >> 6;
    uint32_t c[4], own = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        c[k] = count[4 * t + k];
        count[4 * t + k] = 0u;
        own += c[k];
    }
    uint32_t incl = own;                           // inclusive scan within the wave
#pragma unroll
    for (uint32_t d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(incl, d);
        if (lane >= d) incl += o;
    }
    if (lane == 63) wave_sum[wv] = incl;
    __syncthreads();
    uint32_t base = 0;
    for (uint32_t w = 0; w < wv; ++w) base += wave_sum[w];
    uint32_t run = base + incl - own;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        next[4 * t + k] = run;
        run += c[k];
    }
}

// perm[next[cell]++] = sample: each workgroup ranks its samples (as
// k_train_bin_count takes them) per cell in LDS, then reserves one run per
// cell it holds
template <uint32_t PER>
__global__ void __launch_bounds__(kBinThreads) k_train_bin_scatter(const float *queries, uint32_t n, uint32_t *next,
                                                                   uint32_t *perm)
{
    __shared__ uint32_t hist[kTrainBins];
    for (uint32_t b = threadIdx.x; b < kTrainBins; b += kBinThreads) hist[b] = 0u;
    __syncthreads();
    uint32_t bin[PER], rank[PER];
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
        const uint32_t i = (blockIdx.x * PER + k) * kBinThreads + threadIdx.x;
        bin[k] = i < n ? bin_of(queries[3u * i], queries[3u * i + 1u]) : 0u;
        rank[k] = i < n ? atomicAdd(&hist[bin[k]], 1u) : 0u;
    }
    __syncthreads();
    for (uint32_t b = threadIdx.x; b < kTrainBins; b += kBinThreads)
        if (hist[b]) hist[b] = atomicAdd(&next[b], hist[b]);
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < PER; ++k) {
        const uint32_t i = (blockIdx.x * PER + k) * kBinThreads + threadIdx.x;
        if (i < n) perm[hist[bin[k]] + rank[k]] = i;
    }
}

// The MLP backward works on groups of 16 samples in the matrix cores' fp32
// 16x16x4 layout: lane L = (g, i), g = L / 16, holds of sample i the units
// 16 mb + 4 r + g (register r of tile mb) of every hidden activation and delta.
// A product's output rows are numbered so that this is also the operand the
// next product reads (K chunk kc: lane (g, i) supplies unit 4 kc + g = register
// kc % 4 of tile kc / 4), so the chain forward through the hidden layers and
// back through the transposes stays in registers. Row m of a tile is therefore
// unit hidden_unit(m). Only the parameter gradients, whose K runs over the
// samples, need the other operand order: 16 x 16 tiles go through the wave's
// LDS, written and read without bank conflicts.
//
// What bounds it: 5.5K multiply-adds a sample on the fp32 matrix cores (73 us
// of 2^20 samples with 12-32-32-10 at their rate) and the filter's texel
// reads, which two waves per SIMD overlap. The version before kept one row per
// sample in LDS between all products, at strides of 32 and 33 floats (up to
// 16 lanes on one bank): 390 -> 170 us for those 2^20 samples (150
// from packed texels), 173 -> 36 us for 2^18 with 12-16-16-8 (where the waves' own flushes, 3072 atomics a
// parameter, weighed more; now one per workgroup, 512).
__host__ __device__ constexpr uint32_t hidden_unit(uint32_t m) { return 4u * (m & 3u) + (m >> 2); }

constexpr int kBwdWaves = 4;
// floats per sample of the z and dL/dG rows: 16 and a pad that spreads the 64
// lanes (16 rows, 4 columns) of an operand read over all 64 banks
constexpr int kRowPad = 20;

// The weights as A operands in LDS, four K chunks of a lane per 16 bytes:
// forward rows for layer 0 (3 chunks) and the hidden layers, transposes for
// the way back, and the biases in the order of a lane's registers.
template <int H, int NH>
struct BwdOps {
    static constexpr int T = H / 16, NHID = NH > 1 ? NH - 1 : 1;
    f32x4 f0[T][64], fh[NHID][T][T][64];          // W_0, W_l rows: [tile][K chunks / 4][lane]
    f32x4 bo[T][64], bh[NHID][T][T][64], b0[T][64];   // W_out^T, W_l^T, W_0^T
    f32x4 bias[NH][T][4];                         // [layer][tile][g]
};

// A wave's share of LDS: z and dL/dG of its 64 samples, one row each, and a
// group's hidden activations and deltas, 16 x 16 tiles with one row per sample
// (column 4 g + r: register r of lane group g).
template <int H>
struct __align__(16) BwdWave {
    float z[64][kRowPad], go[64][kRowPad];
    float act[H / 16][16][16], del[H / 16][16][16];
};

template <int H, int NH>
__device__ __forceinline__ void load_ops(const TrainDesc &d, BwdOps<H, NH> &m)
{
    constexpr int T = H / 16;
    const uint32_t n0 = d.dims[0], c = d.dims[NH + 1];
    const float *P = d.params;
    for (uint32_t e = threadIdx.x; e < (uint32_t)(T * 64); e += blockDim.x) {
        const uint32_t mb = e >> 6, L = e & 63u, g = L >> 4, i = L & 15u, u = 16u * mb + hidden_unit(i);
        const uint32_t col = 3u * (i >> 2) + (i & 3u);
        f32x4 a, b, w;
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t in = 4u * k + g, hid = 16u * mb + 4u * k + g;
            a[k] = in < n0 && k < 3 ? P[d.w_off[0] + u * n0 + in] : 0.0f;
            b[k] = in < c ? P[d.w_off[NH] + in * H + u] : 0.0f;
            // row 4 t + ch: channel ch of pyramid t (ch 3: zero)
            w[k] = (i & 3u) < 3u && col < n0 ? P[d.w_off[0] + hid * n0 + col] : 0.0f;
        }
        m.f0[mb][L] = a;
        m.bo[mb][L] = b;
        m.b0[mb][L] = w;
    }
    for (uint32_t e = threadIdx.x; e < (uint32_t)((NH - 1) * T * T * 64); e += blockDim.x) {
        const uint32_t l = e / (T * T * 64), mb = e / (T * 64) % T, kq = e / 64 % T, L = e & 63u;
        const uint32_t g = L >> 4, u = 16u * mb + hidden_unit(L & 15u);
        const float *W = P + d.w_off[l + 1];
        f32x4 a, b;
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) {
            const uint32_t in = 16u * kq + 4u * k + g;
            a[k] = W[u * H + in];
            b[k] = W[in * H + u];
        }
        m.fh[l][mb][kq][L] = a;
        m.bh[l][mb][kq][L] = b;
    }
    for (uint32_t e = threadIdx.x; e < (uint32_t)(NH * T * 4); e += blockDim.x) {
        const uint32_t l = e / (T * 4), mb = e / 4 % T, g = e & 3u;
        f32x4 a;
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) a[r] = P[d.b_off[l] + 16u * mb + 4u * r + g];
        m.bias[l][mb][g] = a;
    }
}

__device__ __forceinline__ f32x4 mma4(f32x4 a, const float *b, f32x4 acc)
{
#pragma unroll
    for (int k = 0; k < 4; ++k) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[k], b[k], acc, 0, 0, 0);
    return acc;
}

// A layer's parameter gradients, dL/dW[j][i] = sum over samples of delta[j] *
// a[i], summed per wave on the matrix cores in 16 x 16 tiles, K running over
// the samples (step s of a group: lane (g, i) supplies column i of sample
// 4 s + g of both). The bias gradients are the per-lane sums of the delta
// reads, added across the four lane groups at the end.
template <int MT, int NT>
struct LayerGrad {
    f32x4 w[MT][NT];
    float b[MT];
};

template <int MT, int NT>
__device__ __forceinline__ void grad_zero(LayerGrad<MT, NT> &g)
{
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        g.b[m] = 0.0f;
#pragma unroll
        for (int n = 0; n < NT; ++n) g.w[m][n] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
    }
}

// dl, a: this lane's first element (sample g, column i) of the deltas and the
// inputs, LD floats per sample, tiles 256 floats apart
template <int MT, int NT, int LDD, int LDA>
__device__ __forceinline__ void accumulate(LayerGrad<MT, NT> &g, const float *dl, const float *a)
{
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        float av[NT], dv[MT];
#pragma unroll
        for (int n = 0; n < NT; ++n) av[n] = a[256 * n + 4 * s * LDA];
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            dv[m] = dl[256 * m + 4 * s * LDD];
            g.b[m] += dv[m];
        }
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int n = 0; n < NT; ++n) g.w[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(dv[m], av[n], g.w[m][n], 0, 0, 0);
    }
}

// Adds the workgroup's layer gradients to gw (W[n_out][n_in], row-major) and
// gb (b[n_out]): the waves' tiles are summed through LDS (red: 1024 floats), so
// that one float atomic per parameter and workgroup goes to memory. HO / HI:
// the rows / columns are hidden units (in register order), else in order.
template <bool HO, bool HI, int MT, int NT>
__device__ __forceinline__ void flush(const LayerGrad<MT, NT> &gr, float *red, float *gw, float *gb, uint32_t n_in,
                                      uint32_t n_out, uint32_t lane, uint32_t wv)
{
    static_assert(kBwdWaves == 4, "wave k sums register k of the four waves' tiles");
    const uint32_t g = lane >> 4, i = lane & 15u;
#pragma unroll
    for (int m = 0; m < MT; ++m) {
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            __syncthreads();
            *reinterpret_cast<f32x4 *>(red + 256 * wv + 4 * lane) = gr.w[m][n];
            __syncthreads();
            const float v = (red[4 * lane + wv] + red[256 + 4 * lane + wv]) +
                            (red[512 + 4 * lane + wv] + red[768 + 4 * lane + wv]);
            const uint32_t row = 4u * g + wv;
            const uint32_t j = 16u * m + (HO ? hidden_unit(row) : row), k = 16u * n + (HI ? hidden_unit(i) : i);
            if (j < n_out && k < n_in) unsafeAtomicAdd(gw + j * n_in + k, v);
        }
        float b = gr.b[m];
        b += __shfl_xor(b, 16);
        b += __shfl_xor(b, 32);
        __syncthreads();
        if (g == 0) red[16 * wv + i] = b;
        __syncthreads();
        if (threadIdx.x < 16) {
            const uint32_t j = 16u * m + (HO ? hidden_unit(i) : i);
            if (j < n_out) unsafeAtomicAdd(gb + j, (red[i] + red[16 + i]) + (red[32 + i] + red[48 + i]));
        }
    }
}

template <int H, int NH, int PACK>
__global__ void __launch_bounds__(64 * kBwdWaves, 2) k_train_backward(TrainDesc d, const float *queries, uint32_t n,
                                                                      const float *grad_out, const uint32_t *perm)
{
    constexpr int T = H / 16;                 // 16-wide tiles of a hidden layer
    __shared__ BwdWave<H> waves[kBwdWaves];
    __shared__ BwdOps<H, NH> ops;
    __shared__ TrainLevelLut lut;
    load_level_lut(d, lut);
    load_ops<H, NH>(d, ops);
    __syncthreads();

    const uint32_t lane = threadIdx.x & 63u, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t g = lane >> 4, i16 = lane & 15u;
    const uint32_t n0 = d.dims[0], c = d.dims[NH + 1];
    // layer 0 (at most 12 inputs), the hidden layers, the output layer (at most 16 rows)
    LayerGrad<T, 1> g0;
    LayerGrad<T, T> gh[NH > 1 ? NH - 1 : 1];
    LayerGrad<1, T> gl;
    grad_zero(g0);
#pragma unroll
    for (int l = 0; l < (NH > 1 ? NH - 1 : 1); ++l) grad_zero(gh[l]);
    grad_zero(gl);

    BwdWave<H> &w = waves[wv];
    // Samples in the sorted order, 64 per wave; workgroups are dealt to the
    // 8 XCDs in turn (the grid is a multiple of 8), and XCD x takes the x-th
    // eighth of the order.
    const uint32_t n_chunks = (n + 63u) / 64u, xcd = blockIdx.x & 7u, xcd_wgs = gridDim.x >> 3;
    const uint32_t c_end = (uint32_t)((uint64_t)n_chunks * (xcd + 1u) / 8u);
    for (uint32_t ch = (uint32_t)((uint64_t)n_chunks * xcd / 8u) + (blockIdx.x >> 3) * kBwdWaves + wv; ch < c_end;
         ch += xcd_wgs * kBwdWaves) {
        const uint32_t slot = ch * 64u + lane;
        const bool live = slot < n;
        const uint32_t q = live ? perm[slot] : 0u;
        const float u = live ? queries[3u * q] : 0.0f;
        const float v = live ? queries[3u * q + 1u] : 0.0f;
        const float s = live ? queries[3u * q + 2u] : 0.0f;
        if (live) d.bin_q[slot] = make_float4(u, v, s, 0.0f);      // in the sorted order, for the scatter
        float go[kMaxOut];
#pragma unroll
        for (int j = 0; j < kMaxOut; ++j) go[j] = live && (uint32_t)j < c ? grad_out[(size_t)q * c + j] : 0.0f;
        float z[12];
        features<PACK>(d, lut, u, v, s, z);
#pragma unroll
        for (int k = 0; k < 3; ++k)
            *reinterpret_cast<f32x4 *>(&w.z[lane][4 * k]) = (f32x4){z[4 * k], z[4 * k + 1], z[4 * k + 2], z[4 * k + 3]};
#pragma unroll
        for (int k = 0; k < 4; ++k)
            *reinterpret_cast<f32x4 *>(&w.go[lane][4 * k]) =
                (f32x4){go[4 * k], go[4 * k + 1], go[4 * k + 2], go[4 * k + 3]};
        wave_sync_lds();
#pragma unroll 1
        for (uint32_t grp = 0; grp < 4; ++grp) {
            const uint32_t row = 16u * grp + i16;
            // the hidden layers
            f32x4 act[NH][T];
            {
                float zb[4];
#pragma unroll
                for (int k = 0; k < 3; ++k) zb[k] = w.z[row][4 * k + g];
#pragma unroll
                for (int mb = 0; mb < T; ++mb) {
                    const f32x4 a = ops.f0[mb][lane];
                    f32x4 acc = ops.bias[0][mb][g];
#pragma unroll
                    for (int k = 0; k < 3; ++k) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[k], zb[k], acc, 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < 4; ++r) act[0][mb][r] = fmaxf(acc[r], 0.0f);
                }
            }
#pragma unroll
            for (int l = 1; l < NH; ++l) {
                f32x4 acc[T];
#pragma unroll
                for (int mb = 0; mb < T; ++mb) acc[mb] = ops.bias[l][mb][g];
#pragma unroll
                for (int kq = 0; kq < T; ++kq) {
                    const float x[4] = {act[l - 1][kq][0], act[l - 1][kq][1], act[l - 1][kq][2], act[l - 1][kq][3]};
#pragma unroll
                    for (int mb = 0; mb < T; ++mb) acc[mb] = mma4(ops.fh[l - 1][mb][kq][lane], x, acc[mb]);
                }
#pragma unroll
                for (int mb = 0; mb < T; ++mb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) act[l][mb][r] = fmaxf(acc[mb][r], 0.0f);
            }
            // back through them: del = delta of hidden layer l's pre-activation
            f32x4 del[T];
            {
                float x[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) x[k] = w.go[row][4 * k + g];
#pragma unroll
                for (int mb = 0; mb < T; ++mb) {
                    const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
                    const f32x4 p = mma4(ops.bo[mb][lane], x, zero);
#pragma unroll
                    for (int r = 0; r < 4; ++r) del[mb][r] = act[NH - 1][mb][r] > 0.0f ? p[r] : 0.0f;
                }
            }
#pragma unroll
            for (int mb = 0; mb < T; ++mb) {
                *reinterpret_cast<f32x4 *>(&w.act[mb][i16][4 * g]) = act[NH - 1][mb];
                *reinterpret_cast<f32x4 *>(&w.del[mb][i16][4 * g]) = del[mb];
            }
            wave_sync_lds();
            accumulate<1, T, kRowPad, 16>(gl, &w.go[16 * grp + g][i16], &w.act[0][g][i16]);
#pragma unroll
            for (int l = NH - 1; l >= 1; --l) {
                // the inputs of layer l, then its delta goes one layer down
                wave_sync_lds();
#pragma unroll
                for (int mb = 0; mb < T; ++mb) *reinterpret_cast<f32x4 *>(&w.act[mb][i16][4 * g]) = act[l - 1][mb];
                wave_sync_lds();
                accumulate<T, T, 16, 16>(gh[l - 1], &w.del[0][g][i16], &w.act[0][g][i16]);
                f32x4 p[T];
#pragma unroll
                for (int mb = 0; mb < T; ++mb) p[mb] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int kq = 0; kq < T; ++kq) {
                    const float x[4] = {del[kq][0], del[kq][1], del[kq][2], del[kq][3]};
#pragma unroll
                    for (int mb = 0; mb < T; ++mb) p[mb] = mma4(ops.bh[l - 1][mb][kq][lane], x, p[mb]);
                }
#pragma unroll
                for (int mb = 0; mb < T; ++mb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) del[mb][r] = act[l - 1][mb][r] > 0.0f ? p[mb][r] : 0.0f;
                wave_sync_lds();
#pragma unroll
                for (int mb = 0; mb < T; ++mb) *reinterpret_cast<f32x4 *>(&w.del[mb][i16][4 * g]) = del[mb];
                wave_sync_lds();
            }
            accumulate<T, 1, 16, kRowPad>(g0, &w.del[0][g][i16], &w.z[16 * grp + g][i16]);
            // dL/dz = W_0^T delta: lane (g, i) receives the three channels of
            // pyramid g of sample i; stored per pyramid in the sorted order
            f32x4 dz = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int kq = 0; kq < T; ++kq) {
                const float x[4] = {del[kq][0], del[kq][1], del[kq][2], del[kq][3]};
                dz = mma4(ops.b0[kq][lane], x, dz);
            }
            const uint32_t to = ch * 64u + row;
            if (g < d.n_tex && to < n) *reinterpret_cast<f32x4 *>(d.bin_dz + (size_t)g * d.bin_batch + to) = dz;
            wave_sync_lds();
        }
    }
    float *red = &waves[0].z[0][0];
    static_assert(sizeof(waves[0].z) >= 1024 * sizeof(float), "the flush's sums fit a wave's rows");
    flush<true, false>(g0, red, d.g_params + d.w_off[0], d.g_params + d.b_off[0], n0, H, lane, wv);
#pragma unroll
    for (int l = 1; l < NH; ++l)
        flush<true, true>(gh[l - 1], red, d.g_params + d.w_off[l], d.g_params + d.b_off[l], H, H, lane, wv);
    flush<false, true>(gl, red, d.g_params + d.w_off[NH], d.g_params + d.b_off[NH], H, c, lane, wv);
}

// ---------------------------------------------------------------------------
// dL/dz -> dL/d texel

// Threads of a region's workgroup: 512 where its windows take more than 8 KB of
// LDS (fewer workgroups are then resident) and there are 2^18 samples, else 256.
// Backward with 256 and 512: 4 x 1024^2 (40 KB) 2^16 samples 147 and 145 us, 2^18
// 209 and 206, 2^20 367 and 347; 4 x 512^2 (12 KB) 2^12 87 and 94, 2^18 177 and
// 175, 2^20 389 and 381; 4 x 256^2 (5 KB) 2^18 146 and 148, 2^20 343 and 362.
constexpr unsigned kScatterThreads = 512;
constexpr uint32_t kScatterWide = 1u << 18, kScatterWidePool = 8 * 1024;
// LDS for a workgroup's windows at most: two workgroups a CU
constexpr uint32_t kScatterPoolMax = 72 * 1024;
// A window of one level: the texels x0 .. x0 + w - 1 (wrapped) of rows y0 ..
// y0 + h - 1, three sums each from `off` in the pool; off = ~0u: the level's
// gradients go straight to memory. div_w = ceil(2^32 / w) (w > 1), so that
// p / w = umulhi(p, div_w) for the window's texels p (p < 2^13).
struct TexWindow {
    uint32_t x0, y0, w, h, off, div_w;
};

// Texels of a window's side on a level of `wl` texels: a region of `cells`
// cells spans cells * wl / side texels; its samples' taps span at most ceil of
// that + 2 from floor(first cell * wl / side - 0.5).
__host__ __device__ inline uint32_t window_side(uint32_t wl, uint32_t cells)
{
    const uint32_t span = (cells * wl + kTrainBinSide - 1) / kTrainBinSide + 2u;
    return wl < span ? wl : span;
}

// The least e with |x| < 2^e, of a finite |x| as bits (-125 for those below
// 2^-125).
__device__ __forceinline__ int exponent_above(uint32_t bits) { return max((int)(bits >> 23), 1) - 126; }

// The wave's largest value, in its last lane.
__device__ __forceinline__ uint32_t wave_max_63(uint32_t v)
{
    auto up = [&](auto ctrl) {                      // lanes without a source read 0
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, 0xF, 0xF, true);
    };
    v = max(v, up(std::integral_constant<int, 0x111>()));       // row_shr 1, 2, 4, 8
    v = max(v, up(std::integral_constant<int, 0x112>()));
    v = max(v, up(std::integral_constant<int, 0x114>()));
    v = max(v, up(std::integral_constant<int, 0x118>()));
    v = max(v, up(std::integral_constant<int, 0x142>()));       // row_bcast 15, 31
    return max(v, up(std::integral_constant<int, 0x143>()));
}

__device__ __forceinline__ int bit_width(uint32_t n) { return 32 - __clz((int)n); }

// Bits of a fixed-point contribution so that n of them sum up in 63.
__device__ __forceinline__ int fixed_bits(uint32_t n) { return min(51, 62 - bit_width(n)); }

// One workgroup per region (1 << region_log2 cells of the sample sort a side,
// consecutive in the sort) and pyramid: the region's samples (sorted positions
// begin .. end) add wt * dL/dz to the texels of their taps. Every tap of a
// region's samples at one level lies in a small box around the region's
// footprint, so the sums go to LDS windows over those boxes (the coarsest
// levels first, while the pool lasts; a level without a window goes straight to
// memory) and then to memory, one float atomic per touched channel.
//
// What bounds it (2^20 samples, 4 x 1024^2, 12-32-32-10): set-up, clearing and
// flush of the windows 46 us, the samples' taps 55 us (half of it the LDS
// sums), the flush's atomics 20 us. The version before took single cells, all
// pyramids in one workgroup, and one thread a sample with two dependent
// gathers (sorted index, query): 250 us, 100 of them 18M atomics of 4-texel
// windows; 2 x 2 cells a region and one pyramid a workgroup need 10M, and the
// backward leaves queries and dL/dz in the sorted order. Plain stores inside
// the windows, where no other region's samples reach, were much slower than
// atomics everywhere (225 against 155 us): lines that both touch. So were the
// coarse levels in workgroups of their own (155 against 122 us: their samples'
// sums meet on few LDS addresses). LDS float atomics cost about 40 times
// integer ones on this GPU, so the windows sum in fixed point: contribution v
// adds rint(v 2^k), with 2^k chosen from the largest |dL/dz| so that a
// contribution (whose weight is at most 1) stays below 2^51, in which it is
// exact or within 2^-51 of that largest one, and the 64-bit sums cannot
// overflow (a float times 2^k plus 1.5 2^52 as doubles has the integer in its
// low bits: as many instructions as a 32-bit integer takes, which kept 30
// bits). A region whose cells differ by more than that leaves room for is
// taken cell by cell, each at its own scale. Non-finite gradients take float
// atomics.
__global__ void __launch_bounds__(kScatterThreads) k_train_scatter(TrainDesc d, uint32_t region_log2,
                                                                   uint32_t pool_sums)
{
    extern __shared__ unsigned long long pool[];
    __shared__ TexWindow win[kMaxLevels];
    __shared__ uint32_t pool_used, cell_at[5], cell_max[4];     // of the region's cells (at most four)
    // the pyramids of one region on one XCD (workgroups are dealt to the 8 in turn)
    const uint32_t k8 = blockIdx.x >> 3, t = k8 % d.n_tex, region = (k8 / d.n_tex) * 8u + (blockIdx.x & 7u);
    const uint32_t cell0 = region << (2u * region_log2), cells = 1u << region_log2, n_cells = cells * cells;
    const uint32_t begin = cell0 ? d.bin_next[cell0 - 1u] : 0u, end = d.bin_next[cell0 + n_cells - 1u];
    if (begin == end) return;                          // uniform over the workgroup
    // where the second, third and fourth cell's samples start
    uint32_t from[3];
#pragma unroll
    for (uint32_t c = 0; c < 3; ++c) from[c] = c + 1u < n_cells ? d.bin_next[cell0 + c] : end;
    const TrainTexDesc &tx = d.tex[t];
    const uint32_t levels = tx.levels;
    const float bias = tx.bias;
    const float4 *dzs = d.bin_dz + (size_t)t * d.bin_batch;
    if (threadIdx.x < 64u) {
        // lane i: level 15 - i, the coarsest first; the pool goes to a prefix
        const uint32_t i = threadIdx.x, l = (kMaxLevels - 1u - i) & (kMaxLevels - 1u);
        // the region's corner from its Z-order number
        uint32_t cx = 0, cy = 0;
#pragma unroll
        for (uint32_t b = 0; b < 6; ++b) {
            cx |= ((cell0 >> (2 * b)) & 1u) << b;
            cy |= ((cell0 >> (2 * b + 1)) & 1u) << b;
        }
        const bool have = i < kMaxLevels && l < levels;
        const uint32_t wl = max(tx.w >> l, 1u), hl = max(tx.h >> l, 1u);
        const uint32_t ww = window_side(wl, cells), wh = window_side(hl, cells);
        const uint32_t size = have ? 3u * ww * wh : 0u;
        uint32_t upto = size;                      // inclusive prefix over the order
#pragma unroll
        for (uint32_t k = 1; k < kMaxLevels; k <<= 1) {
            const uint32_t o = __shfl_up(upto, k);
            if (i >= k) upto += o;
        }
        const float fx = floorf((float)cx * ((float)wl / (float)kTrainBinSide) - 0.5f);
        const float fy = floorf((float)cy * ((float)hl / (float)kTrainBinSide) - 0.5f);
        TexWindow W;
        W.x0 = ww == wl ? 0u : (uint32_t)(int)fx & (wl - 1u);
        W.y0 = wh == hl ? 0u : (uint32_t)(int)fy & (hl - 1u);
        W.w = ww;
        W.h = wh;
        W.off = have && upto <= pool_sums ? upto - size : ~0u;
        W.div_w = ww > 1u ? 0xFFFFFFFFu / ww + 1u : 0u;
        if (i < kMaxLevels) win[l] = W;
        // the pool in use: the end of the last window that fits
        uint32_t in_use = have && upto <= pool_sums ? upto : 0u;
#pragma unroll
        for (uint32_t k = 1; k < kMaxLevels; k <<= 1) in_use = max(in_use, __shfl_xor(in_use, k));
        if (i == 0u) pool_used = in_use;
        if (i < 4u) cell_max[i] = 0u;
        if (i < 5u) cell_at[i] = i == 0u ? begin : i == 1u ? from[0] : i == 2u ? from[1] : i == 3u ? from[2] : end;
    }
    // the largest |dL/dz| of each cell's samples (as bits: NaN and infinity
    // above every finite value)
    uint32_t mb[4] = {0u, 0u, 0u, 0u};
    for (uint32_t j = begin + threadIdx.x; j < end; j += blockDim.x) {
        const uint4 z = *reinterpret_cast<const uint4 *>(dzs + j);
        const uint32_t m = max(max(z.x & 0x7FFFFFFFu, z.y & 0x7FFFFFFFu), z.z & 0x7FFFFFFFu);
        const uint32_t c = (j >= from[0] ? 1u : 0u) + (j >= from[1] ? 1u : 0u) + (j >= from[2] ? 1u : 0u);
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) mb[i] = max(mb[i], c == i ? m : 0u);
    }
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) mb[i] = wave_max_63(mb[i]);
    __syncthreads();
    if ((threadIdx.x & 63u) == 63u) {
#pragma unroll
        for (uint32_t i = 0; i < 4; ++i) atomicMax(&cell_max[i], mb[i]);
    }
    const uint32_t used = pool_used;
    for (uint32_t e = threadIdx.x; e < used; e += blockDim.x) pool[e] = 0ull;
    __syncthreads();
    uint32_t region_max = 0;
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) region_max = max(region_max, uniform(cell_max[i]));
    // One scale for the region, unless it is coarser for some cell than 2^-29
    // of the cell's largest gradient times its samples (rounded up to powers of
    // two), or a cell's gradients are not finite: then cell by cell.
    bool apart = region_max >= 0x7F800000u;
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) {
        const uint32_t m = uniform(cell_max[i]);
        apart = apart || (m != 0u && exponent_above(region_max) - fixed_bits(end - begin) >
                                         exponent_above(m) + bit_width(uniform(cell_at[i + 1] - cell_at[i])) - 29);
    }
    const uint32_t passes = apart ? n_cells : 1u;
    for (uint32_t pass = 0;;) {
        const uint32_t first = apart ? uniform(cell_at[pass]) : begin, last = apart ? uniform(cell_at[pass + 1]) : end;
        const uint32_t mbits = apart ? uniform(cell_max[pass]) : region_max;
        const bool fixed = mbits < 0x7F800000u;
        const int kexp = fixed ? fixed_bits(last - first) - exponent_above(mbits) : 0;
        const double scale = ldexp(1.0, kexp), unscale = ldexp(1.0, -kexp);
        for (uint32_t j = first + threadIdx.x; j < last; j += blockDim.x) {
            const float4 q = d.bin_q[j], z4 = dzs[j];
            const float dz[3] = {z4.x, z4.y, z4.z};
            const float uf = q.x - floorf(q.x), vf = q.y - floorf(q.y);       // wrap addressing
            // the two levels of eq. (10) as the forward takes them
            const float si = fminf(fmaxf(q.z + bias, 0.0f), (float)(levels - 1u));   // NaN -> 0
            const uint32_t l0 = (uint32_t)floorf(si);
            const uint32_t l1 = min(l0 + 1u, levels - 1u);
            const float lam = si - (float)l0;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const uint32_t l = k ? l1 : l0;
                const float lw = k ? lam : 1.0f - lam;
                // a zero weight (an unused second level) adds nothing
                if (lw == 0.0f) continue;
                const uint32_t wl = max(tx.w >> l, 1u), hl = max(tx.h >> l, 1u);
                const LevelTaps lt = level_taps(make_uint4(wl, hl, 0u, 0u), uf, vf, lw);
                const TexWindow W = win[l];
                const uint32_t dxa = (lt.xa - W.x0) & (wl - 1u), dxb = (lt.xb - W.x0) & (wl - 1u);
                const uint32_t dya = (lt.ya - W.y0) & (hl - 1u), dyb = (lt.yb - W.y0) & (hl - 1u);
                const bool inside = W.off != ~0u && max(dxa, dxb) < W.w && max(dya, dyb) < W.h;
                const uint32_t ra = W.off + 3u * __umul24(dya, W.w), rb = W.off + 3u * __umul24(dyb, W.w);
                const uint32_t at[4] = {ra + 3u * dxa, ra + 3u * dxb, rb + 3u * dxa, rb + 3u * dxb};
                if (inside && fixed) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int c = 0; c < 3; ++c) {
                            const double sum = fma((double)(lt.w[i] * dz[c]), scale, 6755399441055744.0);
                            atomicAdd(pool + at[i] + c,
                                      (unsigned long long)__double_as_longlong(sum) - 0x4338000000000000ull);
                        }
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float wt = lt.w[i];
                        if (wt == 0.0f) continue;
                        const uint32_t x = i & 1 ? lt.xb : lt.xa, y = i & 2 ? lt.yb : lt.ya;
                        float *gp = d.g_texels + 3u * (tx.tex_off[l] + y * wl + x);
#pragma unroll
                        for (int c = 0; c < 3; ++c) {
                            if (inside) atomicAdd(reinterpret_cast<float *>(pool + at[i] + c), wt * dz[c]);
                            else unsafeAtomicAdd(gp + c, wt * dz[c]);
                        }
                    }
                }
            }
        }
        __syncthreads();
        // Sums e = first, first + step, ... of level l's window to memory, the
        // lanes along the channels of a row's texels.
        auto flush = [&](uint32_t l, uint32_t first, uint32_t step) {
            const TexWindow W = win[l];
            const uint32_t wl = max(tx.w >> l, 1u), hl = max(tx.h >> l, 1u), base = tx.tex_off[l];
            for (uint32_t e = first; e < 3u * W.w * W.h; e += step) {
                const unsigned long long raw = pool[W.off + e];
                const uint32_t lo = (uint32_t)raw;
                const float v = fixed ? (float)(fma((double)(int32_t)(raw >> 32), 4294967296.0, (double)lo) * unscale)
                                      : __uint_as_float(lo);
                const uint32_t p = e / 3u, c = e - 3u * p;
                const uint32_t dy = W.w > 1u ? __umulhi(p, W.div_w) : p, dx = p - dy * W.w;
                if (v != 0.0f)
                    unsafeAtomicAdd(
                        d.g_texels + 3u * (base + ((W.y0 + dy) & (hl - 1u)) * wl + ((W.x0 + dx) & (wl - 1u))) + c, v);
            }
        };
        // the large windows by every wave, the small ones by one wave each
        constexpr uint32_t kWaveSums = 256;
        const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        for (uint32_t l = 0; l < levels; ++l) {
            if (win[l].off == ~0u) continue;
            if (3u * win[l].w * win[l].h > kWaveSums) flush(l, threadIdx.x, blockDim.x);
            else if (l % (blockDim.x / 64) == wv) flush(l, threadIdx.x & 63u, 64u);
        }
        if (++pass == passes) return;
        __syncthreads();
        for (uint32_t e = threadIdx.x; e < used; e += blockDim.x) pool[e] = 0ull;
        __syncthreads();
    }
}

unsigned grid_for(size_t work, unsigned per_block, unsigned cap)
{
    const size_t g = (work + per_block - 1) / per_block;
    return (unsigned)(g < 1 ? 1 : (g > cap ? cap : g));
}

// The scatter's regions: 2 x 2 cells, where a window then still spans at most
// 34 texels (level 0 of 1024) or samples are few, else single cells. Backward
// with single cells and 2 x 2: 4 x 512^2 2^18 samples 284 and 177 us, 2^20 631
// and 381; 4 x 1024^2 303 and 211, 436 and 348; 4 x 2048^2 (whose level 0 goes
// straight to memory from 2 x 2) 2^14 421 and 317, 2^18 505 and 449, 2^19 548 and
// 551, 2^20 654 and 734; one of 4096^2 2^14 450 and 421, 2^18 610 and 543, 2^20
// 753 and 757.
uint32_t scatter_region_log2(const TrainDesc &d, uint32_t samples)
{
    uint32_t side = 0;
    for (uint32_t t = 0; t < d.n_tex; ++t) side = std::max(side, std::max(d.tex[t].w, d.tex[t].h));
    return side <= 1024 || samples < (1u << 19) ? 1u : 0u;
}

// LDS sums for the windows of the largest pyramid, the coarsest levels first,
// as far as two workgroups share a CU.
uint32_t scatter_pool_sums(const TrainDesc &d, uint32_t region_log2)
{
    uint32_t pool_sums = 0;
    for (uint32_t t = 0; t < d.n_tex; ++t) {
        uint32_t sums = 0;
        for (uint32_t l = d.tex[t].levels; l-- > 0;) {
            const uint32_t more = 3u * window_side(std::max(d.tex[t].w >> l, 1u), 1u << region_log2) *
                                  window_side(std::max(d.tex[t].h >> l, 1u), 1u << region_log2);
            if ((sums + more) * 8u > kScatterPoolMax) break;
            sums += more;
        }
        pool_sums = std::max(pool_sums, sums);
    }
    return pool_sums;
}

hipError_t launch_texels(const TrainDesc &d, hipStream_t s)
{
    if (d.packed && !d.ste) {
        const unsigned grid = grid_for(((size_t)d.tex[0].n_blocks + 15u) / 16u * 256u, kTrainThreads, 16384);
        k_train_texels_floats<<<grid, kTrainThreads, 0, s>>>(d);
        return hipGetLastError();
    }
    if (d.packed) {
        unsigned chunks = 0;
        bool al = true;
        for (uint32_t l = 0; l < d.tex[0].levels; ++l)
            chunks += (((std::max(d.tex[0].w >> l, 1u) + 3u) / 4u) * ((std::max(d.tex[0].h >> l, 1u) + 3u) / 4u) + 63u) / 64u;
        for (uint32_t t = 0; t < d.n_tex; ++t)
            al = al && ((uintptr_t)d.tex[t].endpoints & 15u) == 0 && ((uintptr_t)d.tex[t].indices & 15u) == 0;
        if (al) k_train_texels_packed<true><<<chunks, kTrainThreads, 0, s>>>(d);
        else k_train_texels_packed<false><<<chunks, kTrainThreads, 0, s>>>(d);
        return hipGetLastError();
    }
    const unsigned grid = grid_for((size_t)d.blk_base[d.n_tex] * 4u, kTrainThreads, 16384);
    if (d.ste) k_train_texels<true><<<grid, kTrainThreads, 0, s>>>(d);
    else k_train_texels<false><<<grid, kTrainThreads, 0, s>>>(d);
    return hipGetLastError();
}

template <int H, int NH>
hipError_t forward_hn(const TrainDesc &d, const float *queries, uint32_t n, float *out, hipStream_t s)
{
    hipError_t e = launch_prepare_weights(d.params, nullptr, d.ops_shape, MLP_MFMA_F32, d.ops, d.ops_ws, nullptr, s);
    if (e != hipSuccess) return e;
    const unsigned grid = grid_for(n, kTrainThreads, 8192);
    auto *forward = !d.packed ? k_train_forward_mfma<H, NH, 0>
                  : d.ste ? k_train_forward_mfma<H, NH, 1> : k_train_forward_mfma<H, NH, 2>;
    forward<<<grid, kTrainThreads, 0, s>>>(d, queries, n, out);
    return hipGetLastError();
}

template <int H, int NH>
hipError_t backward_hn(const TrainDesc &d, const float *queries, uint32_t n, const float *grad_out, hipStream_t s)
{
    // the workgroups resident at once (two per CU), a multiple of the 8 XCDs
    const unsigned grid = (grid_for((n + 63u) / 64u, kBwdWaves, 512) + 7u) & ~7u;
    auto *backward = !d.packed ? k_train_backward<H, NH, 0>
                   : d.ste ? k_train_backward<H, NH, 1> : k_train_backward<H, NH, 2>;
    backward<<<grid, 64 * kBwdWaves, 0, s>>>(d, queries, n, grad_out, d.bin_perm);
    return hipGetLastError();
}

#define BCF_TRAIN_DISPATCH(fn, ...)                                                           \
    do {                                                                                      \
        const uint32_t H = d.dims[1], NH = d.n_layers - 1;                                    \
        if (H == 16 && NH == 1) return fn<16, 1>(d, __VA_ARGS__);                             \
        if (H == 16 && NH == 2) return fn<16, 2>(d, __VA_ARGS__);                             \
        if (H == 16 && NH == 3) return fn<16, 3>(d, __VA_ARGS__);                             \
        if (H == 32 && NH == 1) return fn<32, 1>(d, __VA_ARGS__);                             \
        if (H == 32 && NH == 2) return fn<32, 2>(d, __VA_ARGS__);                             \
        if (H == 32 && NH == 3) return fn<32, 3>(d, __VA_ARGS__);                             \
        return hipErrorInvalidValue;                                                          \
    } while (0)

hipError_t dispatch_forward(const TrainDesc &d, const float *queries, uint32_t n, float *out, hipStream_t s)
{
    BCF_TRAIN_DISPATCH(forward_hn, queries, n, out, s);
}

hipError_t dispatch_backward(const TrainDesc &d, const float *queries, uint32_t n, const float *grad_out,
                             hipStream_t s)
{
    BCF_TRAIN_DISPATCH(backward_hn, queries, n, grad_out, s);
}

#undef BCF_TRAIN_DISPATCH

}  // namespace

hipError_t launch_train_forward(const TrainDesc &d, const float *queries, size_t n, float *out, hipStream_t s)
{
    hipError_t e = launch_texels(d, s);
    if (e != hipSuccess || n == 0) return e;
    return dispatch_forward(d, queries, (uint32_t)n, out, s);
}

hipError_t launch_train_backward(const TrainDesc &d, const float *queries, size_t n, const float *grad_out,
                                 hipStream_t s)
{
    hipError_t e = launch_texels(d, s);
    if (e != hipSuccess) return e;
    k_train_clear<<<grid_for(std::max<size_t>((size_t)d.n_texels / 4u * 3u, kTrainBins), 256, 8192), 256, 0, s>>>(d);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const uint32_t c = d.dims[d.n_layers];
    // batches of one size
    const size_t batches = (n + d.bin_batch - 1) / d.bin_batch;
    const size_t batch = batches ? ((n + batches - 1) / batches + 63u) & ~(size_t)63u : 1;
    for (size_t off = 0; off < n; off += batch) {
        const uint32_t m = (uint32_t)std::min(n - off, batch);
        const float *q = queries + 3 * off;
        const uint32_t per = bin_per_thread(m);
        const unsigned bins = (m + per * kBinThreads - 1) / (per * kBinThreads);
        if (per == 1) k_train_bin_count<1><<<bins, kBinThreads, 0, s>>>(q, m, d.bin_count);
        else k_train_bin_count<8><<<bins, kBinThreads, 0, s>>>(q, m, d.bin_count);
        k_train_bin_scan<<<1, kBinThreads, 0, s>>>(d.bin_count, d.bin_next);
        if (per == 1) k_train_bin_scatter<1><<<bins, kBinThreads, 0, s>>>(q, m, d.bin_next, d.bin_perm);
        else k_train_bin_scatter<8><<<bins, kBinThreads, 0, s>>>(q, m, d.bin_next, d.bin_perm);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if ((e = dispatch_backward(d, q, m, grad_out + (size_t)c * off, s)) != hipSuccess) return e;
        const uint32_t region_log2 = scatter_region_log2(d, m), pool_sums = scatter_pool_sums(d, region_log2);
        const unsigned threads = m >= kScatterWide && pool_sums * 8u > kScatterWidePool ? kScatterThreads
                                                                                       : kScatterThreads / 2;
        k_train_scatter<<<(kTrainBins >> (2 * region_log2)) * d.n_tex, threads, pool_sums * 8u, s>>>(
            d, region_log2, pool_sums);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    const unsigned grid = grid_for((size_t)d.blk_base[d.n_tex] * 4u, kTrainThreads, 16384);
    uintptr_t bits = 0;
    for (uint32_t t = 0; t < d.n_tex; ++t)
        bits |= (uintptr_t)d.tex[t].endpoints | (uintptr_t)d.tex[t].indices | (uintptr_t)d.tex[t].g_indices;
    auto *blocks = (bits & 15u) == 0 ? (d.ste ? k_train_blocks<true, true> : k_train_blocks<false, true>)
                                     : (d.ste ? k_train_blocks<true, false> : k_train_blocks<false, false>);
    blocks<<<grid, kTrainThreads, 0, s>>>(d);
    return hipGetLastError();
}

}  // namespace bcf
