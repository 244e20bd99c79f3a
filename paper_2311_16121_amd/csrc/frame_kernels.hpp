// The decode and calibration kernels, instantiated per MLP precision in
// frame_<precision>.hip (separate translation units compile in parallel).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "filter_device.hpp"
#include "internal.hpp"
#include "mlp_device.hpp"

namespace bcf {

typedef uint32_t uint4_t __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// BCF_FP32 takes the fp32 MFMAs too (the binary32 operands and accumulation of
// fp32 FMAs in the lanes, the sums in another order; the error against binary64
// is as large, about 1e-7 relative): at 64 FMA lanes a CU clock the vector ALU
// was its bound.
// A 1920 x 1080 frame with 12-32-32-10: 154 -> 86 us (74 with what else this
// file does); 501 queries of 12-16-16-9: 17 -> 13 us with the unpack.
//
// The decode kernel: one query per lane filters the four pyramid slots, then
// the MLP on the matrix cores: the wave's 64 feature vectors go through LDS
// into the operand layout of mlp_device.hpp, four groups of 16 queries per
// wave. Outputs are staged in LDS so each wave writes its 64 rows with
// coalesced buffer stores.

constexpr int kFrameThreads = 256;
constexpr int kFrameWaves = kFrameThreads / 64;
// a wave's 64 feature vectors (4 x float4 each) fit its output stage
static_assert(64 * 4 <= 64 * kMaxOut / 4, "feature vectors must fit the output stage");

// Cache policy of the output stores: non-temporal (streamed). The kernels
// never read their outputs back; on the frame benchmark the decode runs about
// a quarter faster with its output stream marked so.
constexpr int kStoreNT = 2;   // the buffer intrinsics' cache-policy bit for "nt"

struct FrameArgs {
    LevelLut lut;
    float levels_bias[2 * kMaxTextures];   // per slot: level count (bits), b_i
    uint32_t stride;                       // shared geometry: bytes between slots' scratch
    const uint8_t *ws;
    WsLayout lay;
    const float *queries;
    float *out;
    uint32_t n;                            // queries of this launch
    uint32_t out_dim;
    float *absmax;                         // k_calibrate: per-layer largest |input|
    // 2D work items: with grid_w > 0 the queries are image rows of grid_w and
    // a wave takes a tile of kTileW columns by kTileH rows (lane = row *
    // kTileW + column) of the image's `rows`; with 0, 64 consecutive queries.
    // row_rest: tile rows of this image can end in 1..3 floats that no 16-byte
    // chunk takes (its rows or its n * out_dim are no multiple of 4 floats)
    uint32_t grid_w, rows, tiles_x, n_items, row_rest;
    uint32_t tiles_x_inv, per_inv;    // divide_by's for tiles_x and strip_rows * tiles_x
    // tiled work: tiles_y rows of tiles; strip_rows > 0: the tile rows form
    // strips of that many, dealt to the XCDs in turn (0: items round-robin).
    // Linear work is laid out the same way, as rows of tiles_x items.
    uint32_t tiles_y, strip_rows;
};

// Work-item tiles for queries declared as an image: 16 x 4.
constexpr uint32_t kTileLog2 = 4, kTileW = 1u << kTileLog2, kTileH = 64u >> kTileLog2;

// The grid is a multiple of the 8 XCDs, to which workgroups are dispatched
// round-robin (workgroup b runs on XCD b % 8), and at most what is resident
// at once, so the waves sweep the image nearly together. Tiled
// work deals strips of whole tile rows to the XCDs in turn (strip j to XCD
// j % 8); an XCD's waves walk its strips tile by tile. Texels are shared
// along a strip -- a textured plane that wraps repeats the same texels
// across the image's width -- so whole-width strips keep that sharing inside
// one XCD's L2, while the strips of different XCDs share only their edge
// rows. Linear work is dealt the same way in runs of kLinearRun items
// (consecutive queries share texels along a scanline); images or runs too
// few to give every XCD one go round-robin over all waves.
constexpr uint32_t kXcds = 8;
constexpr uint32_t kLinearRun = 64;     // 64-query items per run of linear work dealt to one XCD

// A wave's share of the work: items first, first + step, ... below end. In
// strip mode item k is tile k % per of strip (k / per) * kXcds + xcd, per =
// strip_rows * tiles_x tiles; otherwise item k is tile k (row-major).
struct WaveWork {
    uint32_t first, end, step, xcd, per;
};

__device__ __forceinline__ WaveWork wave_work(const FrameArgs &a, uint32_t wv)
{
    if (a.strip_rows) {
        const uint32_t x = blockIdx.x % kXcds;
        const uint32_t n_strips = (a.tiles_y + a.strip_rows - 1) / a.strip_rows;
        const uint32_t mine = n_strips > x ? (n_strips - x + kXcds - 1) / kXcds : 0;   // strips x, x + 8, ...
        const uint32_t per = a.strip_rows * a.tiles_x;
        // the last strip ends with the last item
        const uint32_t past = (n_strips - 1) % kXcds == x ? n_strips * per - a.n_items : 0;
        return WaveWork{(blockIdx.x / kXcds) * kFrameWaves + wv, mine * per - past, (gridDim.x / kXcds) * kFrameWaves,
                        x, per};
    }
    return WaveWork{blockIdx.x * kFrameWaves + wv, a.n_items, gridDim.x * kFrameWaves, 0, 0};
}

struct ItemRange {
    uint32_t first, end, step;
};

// k / d and k % d from inv = (2^32 - 1) / d: the high product is the quotient
// or one less. For scalars that is six scalar instructions, and a division's
// float reciprocal is some fifteen vector ones and three moves between the files.
__device__ __forceinline__ uint32_t divide_by(uint32_t k, uint32_t d, uint32_t inv, uint32_t &rem)
{
    uint32_t q = __umulhi(k, inv);
    rem = k - q * d;
    if (rem >= d) {
        ++q;
        rem -= d;
    }
    return q;
}

struct Query {
    float u, v, s;
};

// One 12-byte query through the buffer descriptor (reads past the end give 0).
// The vector's elements go through plain integers before the bit casts.
__device__ __forceinline__ Query load_query(__amdgpu_buffer_rsrc_t rq, uint32_t q)
{
    const auto qv = __builtin_amdgcn_raw_buffer_load_b96(rq, (int)(q * 12u), 0, 0);
    const uint32_t u = qv[0], v = qv[1], s = qv[2];
    return Query{__builtin_bit_cast(float, u), __builtin_bit_cast(float, v), __builtin_bit_cast(float, s)};
}

// The MLP parameters do not change during a launch: reading them through the
// constant address space lets the compiler use scalar loads and SGPR operands.
typedef const __attribute__((address_space(4))) float const_float;

__device__ __forceinline__ const_float *constant_floats(const uint8_t *p)
{
    return (const_float *)p;
}

// Row j of a layer's weights and its bias, through the constant address
// space (scalar loads, SGPR operands). The pointer goes through an empty asm
// per row, so the optimiser can neither hoist the loads out of the caller's
// query loop nor keep more than about a row's weights live: 1-2k weights do
// not fit in SGPRs and would be spilled.
__device__ __forceinline__ const_float *weight_row(const uint8_t *ws, size_t off, uint32_t row, uint32_t n_in)
{
    asm volatile("" : "+s"(ws));
    return constant_floats(ws + off) + row * n_in;
}

template <int N_IN>
__device__ __forceinline__ float neuron(const uint8_t *ws, const WsLayout &lay, int l, uint32_t j, const float *x)
{
    const_float *w = weight_row(ws, lay.layer_w_off[l], j, N_IN);
    float acc = constant_floats(ws + lay.layer_b_off[l])[j];
#pragma unroll
    for (int i = 0; i < N_IN; ++i) acc = fmaf(w[i], x[i], acc);
    return acc;
}

// amax[l] = max(amax[l], the largest |input| of layer l) for the feature vector z.
template <int H, int NH>
__device__ __forceinline__ void mlp_maxima(const uint8_t *ws, const WsLayout &lay, const float z[12], float *amax)
{
#pragma unroll
    for (int i = 0; i < 12; ++i) amax[0] = fmaxf(amax[0], fabsf(z[i]));
    float hcur[H];
#pragma unroll
    for (int j = 0; j < H; ++j) hcur[j] = relu(neuron<12>(ws, lay, 0, j, z));
#pragma unroll
    for (int l = 1; l <= NH; ++l) {
#pragma unroll
        for (int i = 0; i < H; ++i) amax[l] = fmaxf(amax[l], hcur[i]);
        if (l == NH) break;                       // the outputs are no layer's input
        float hn[H];
#pragma unroll
        for (int j = 0; j < H; ++j) hn[j] = relu(neuron<H>(ws, lay, l, j, hcur));
#pragma unroll
        for (int j = 0; j < H; ++j) hcur[j] = hn[j];
    }
}

__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ void copy_lut(const LevelLut &src, LevelLut &dst)
{
    const uint4 *s = &src.e[0][0];
    uint4 *d = &dst.e[0][0];
    for (int i = threadIdx.x; i < kMaxTextures * kMaxLevels; i += blockDim.x) d[i] = s[i];
    __syncthreads();
}

// MLP (eq. 3) of a wave's 64 feature vectors z (one per lane); the outputs
// land in the wave's LDS stage, lane L's at st[L * out_dim ...]. The feature
// vectors pass through `feats`, which may be the same LDS as st (both 4 KB).
// YIELD: the other waves of the SIMD go first while this one feeds the matrix
// cores, so that their loads and filters run beside its products (k_frame's
// waves otherwise meet in the MLP one after the other: 1920 x 1080 fp32 91 ->
// 88 us, 2^22 points fp32 178 -> 173, 2720 x 1530 fp16 76.5 -> 74.9; k_batch and
// the training forward, which do not load ahead, lost 1 to 4%).
template <bool YIELD, MlpKind K, int H, int NH>
__device__ __forceinline__ void mlp_stage(const float z[12], const MfmaMlp<K, H, NH> &mlp, float4_t (*feats)[4],
                                          float *st, uint32_t out_dim, uint32_t lane)
{
    const uint32_t g = lane >> 4, qi = lane & 15;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const float4_t v4 = {z[3 * t], z[3 * t + 1], z[3 * t + 2], 0.0f};
        feats[lane][t] = v4;
    }
    wave_lds_sync();
    float4_t fin[4];
#pragma unroll
    for (int grp = 0; grp < 4; ++grp) fin[grp] = feats[16 * grp + qi][g];
    wave_lds_sync();                      // feats and st share the wave's LDS
    float f[4][4];
#pragma unroll
    for (int grp = 0; grp < 4; ++grp)
#pragma unroll
        for (int i = 0; i < 4; ++i) f[grp][i] = fin[grp][i];
    float4_t o[4];
    if (YIELD) __builtin_amdgcn_s_setprio(0);
    mlp.template run_groups<4>(f, o);
    if (YIELD) __builtin_amdgcn_s_setprio(3);
    // lane (g, qi) holds outputs 4g .. 4g + 3 of its query in each group: the
    // lanes that have output 4g + j write the four groups' under one mask (an
    // address select per output and group was forty instructions per item)
    float *row = st + qi * out_dim + 4 * g;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (4 * g + j < out_dim) {
#pragma unroll
            for (int grp = 0; grp < 4; ++grp) row[16 * grp * out_dim + j] = o[grp][j];
        }
    wave_lds_sync();
}

// One wave's 64 queries: filter (eqs. 9, 10), concatenate, MLP.
template <bool YIELD, MlpKind K, int H, int NH, int LAYOUT, bool IN_TURN = false>
__device__ __forceinline__ void decode_wave(const Query &qq, __amdgpu_buffer_rsrc_t rs, const LevelLut &lut,
                                            const float *levels_bias, uint32_t stride,
                                            const MfmaMlp<K, H, NH> &mlp, float4_t (*feats)[4], float *st, uint32_t out_dim, uint32_t lane)
{
    float z[12];
    filter4<LAYOUT, IN_TURN>(rs, lut, levels_bias, stride, qq.u, qq.v, qq.s, z);
    mlp_stage<YIELD, K, H, NH>(z, mlp, feats, st, out_dim, lane);
}

// decode_wave for a material with a position-interleaved scratch
template <bool YIELD, MlpKind K, int H, int NH>
__device__ __forceinline__ void decode_wave_interleaved(const Query &qq, __amdgpu_buffer_rsrc_t rs,
                                                        const LevelLut &lut, const float *levels_bias,
                                                        const MfmaMlp<K, H, NH> &mlp, float4_t (*feats)[4],
                                                        float *st, uint32_t out_dim, uint32_t lane)
{
    PendingPacked taps;
    fetch4_packed(rs, lut, levels_bias, qq.u, qq.v, qq.s, taps);
    float z[12];
    filter_pending_packed(taps, z);
    mlp_stage<YIELD, K, H, NH>(z, mlp, feats, st, out_dim, lane);
}

// Item `it` of a run of n consecutive queries: its (up to) 64 staged rows go
// to out as 16-byte stores, the last partial item as 4-byte stores.
__device__ __forceinline__ void store_run(const float4_t *stage, __amdgpu_buffer_rsrc_t ro, uint32_t it, uint32_t n,
                                          uint32_t out_dim, uint32_t lane)
{
    const uint32_t base = it * 64u * out_dim * 4u;
    if (it * 64 + 64 <= n) {
        for (uint32_t k = lane; k < 16 * out_dim; k += 64)
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uint4_t, stage[k]), ro, (int)(base + 16u * k),
                                                   0, kStoreNT);
    } else {
        const float *st = reinterpret_cast<const float *>(stage);
        const uint32_t floats = (n - it * 64) * out_dim;
        for (uint32_t k = lane; k < floats; k += 64)
            __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, st[k]), ro, (int)(base + 4u * k), 0,
                                                  kStoreNT);
    }
}

// How the items of a launch map to queries and outputs, known to the loop
// when it is compiled: 64 consecutive queries, a tile of an image, or a tile
// of an image with FrameArgs::row_rest.
enum ItemKind { kItemLinear, kItemTile, kItemTileRest };

// A wave's current item: its first query; tiles: the columns and rows that
// the image has from there.
struct Item {
    uint32_t q0, cols, rows;
};

// What a lane adds to every item, so that an item costs its lanes a few
// instructions and the rest scalar ones: its query's byte offset from the
// item's first, and of the item's output its first float in the stage, the
// same float's index in its run (below) and its byte offset from the first.
struct LaneItem {
    uint32_t query, stage, run, out;
};

template <ItemKind KIND>
__device__ __forceinline__ LaneItem lane_item(const FrameArgs &a, uint32_t lane)
{
    if (KIND == kItemLinear) return LaneItem{12u * lane, 4u * lane, 4u * lane, 16u * lane};
    const uint32_t r = lane >> kTileLog2, c = lane & (kTileW - 1u);
    return LaneItem{12u * (r * a.grid_w + c), r * kTileW * a.out_dim + 4u * c, 4u * c,
                    4u * (r * a.grid_w * a.out_dim + 4u * c)};
}

// The query of this lane in an item; past the image's right edge and past n
// (below it) zeros, by the buffer range check.
template <ItemKind KIND>
__device__ __forceinline__ Query item_query(const FrameArgs &a, __amdgpu_buffer_rsrc_t rq, const Item &item,
                                            const LaneItem &li, uint32_t lane)
{
    uint32_t at = 12u * item.q0 + li.query;
    if (KIND != kItemLinear) at = (lane & (kTileW - 1u)) < item.cols ? at : 12u * a.n;
    const auto qv = __builtin_amdgcn_raw_buffer_load_b96(rq, (int)at, 0, 0);
    const uint32_t u = qv[0], v = qv[1], s = qv[2];
    return Query{__builtin_bit_cast(float, u), __builtin_bit_cast(float, v), __builtin_bit_cast(float, s)};
}

// Stores of one work item: always 4 buffer stores of 4 floats per lane (tiles
// with row_rest one more of 1), and no branches around them. Buffer stores
// ask for dword alignment only, so neither the output nor its rows need a
// 16-byte boundary: 1366 x 768 of 9 channels (fp16) 25.5 us with the 16
// four-byte stores per lane that such rows once took, 22.0 with these. An
// item's output is a set of runs of contiguous floats: one run of 64 *
// out_dim for linear items, one of kTileW * out_dim per tile row for tiles.
// The lanes of a run take its 4-float chunks in turn, and with row_rest its
// last lim % 4 floats; a chunk with nowhere to go (past the run, the image's
// right edge or the output's end) is sent to `oob`, the first byte past the
// output buffer, which the buffer range check drops. Stores count in the same
// in-order counter as loads; a fixed count lets the compiler wait for a load
// issued before these stores without waiting for the stores themselves.
template <ItemKind KIND>
__device__ __forceinline__ void store_item(const FrameArgs &a, uint32_t oob, const float *st,
                                           __amdgpu_buffer_rsrc_t ro, const Item &item, const LaneItem &li,
                                           uint32_t lane)
{
    const uint32_t n_out = a.n * a.out_dim, base = item.q0 * a.out_dim, r = lane >> kTileLog2;
    constexpr uint32_t step = KIND == kItemLinear ? 64u * 4u : kTileW * 4u;
    uint32_t lim;                         // floats of the lane's run
    if (KIND == kItemLinear) {
        lim = min(64u * a.out_dim, n_out - base);
    } else {
        lim = r < item.rows ? min(kTileW, item.cols) * a.out_dim : 0u;
        // the last row may end early: its chunks past the output's end are
        // dropped whole, and only with row_rest can one straddle it
        if (KIND == kItemTileRest) {
            const uint32_t first = base + r * a.grid_w * a.out_dim;
            lim = min(lim, n_out - min(first, n_out));
        }
    }
    const uint32_t out = 4u * base + li.out;
#pragma unroll
    for (uint32_t m = 0; m < 4; ++m) {
        const float4_t v = *reinterpret_cast<const float4_t *>(st + li.stage + step * m);
        const uint32_t off = (li.run + step * m + 3u < lim ? out : oob) + 4u * step * m;
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uint4_t, v), ro, (int)off, 0, kStoreNT);
    }
    if (KIND == kItemTileRest) {
        const uint32_t e = (lim & ~3u) + (lane & (kTileW - 1u)), k = li.stage - li.run + e;
        const uint32_t off = e < lim ? out - 4u * li.run + 4u * e : oob;
        const float v = st[min(k, 64u * kMaxOut - 1u)];
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), ro, (int)off, 0, kStoreNT);
    }
}

// The last n * out_dim % 4 floats of a linear launch, which its 16-byte chunks
// leave out, from the stage of the wave that took the last item (an item that
// no other follows in its wave).
__device__ __forceinline__ void store_rest(const FrameArgs &a, const float *st, __amdgpu_buffer_rsrc_t ro,
                                           const Item &last, uint32_t lane)
{
    const uint32_t n_out = a.n * a.out_dim, rest = n_out & 3u, at = n_out - rest;
    if (last.q0 + 64u < a.n || lane >= rest) return;
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, st[at + lane - last.q0 * a.out_dim]), ro,
                                          (int)((at + lane) * 4u), 0, 0);
}

// As many stores past the output's end: the loop's entry then has the same
// stores outstanding as its back edge.
template <ItemKind KIND>
__device__ __forceinline__ void store_dummies(__amdgpu_buffer_rsrc_t ro, uint32_t oob)
{
#pragma unroll
    for (int m = 0; m < (KIND == kItemTileRest ? 5 : 4); ++m) {
        uint32_t o = oob;
        asm volatile("" : "+v"(o));           // separate stores, not merged into wider ones
        if (m < 4)
            __builtin_amdgcn_raw_buffer_store_b128(uint4_t{0, 0, 0, 0}, ro, (int)o, 0, kStoreNT);
        else
            __builtin_amdgcn_raw_buffer_store_b32(0u, ro, (int)o, 0, kStoreNT);
    }
}

template <MlpKind K, int H, int NH, int LAYOUT>
__global__ void __launch_bounds__(kFrameThreads) k_frame(FrameArgs a)
{
    __shared__ LevelLut lut;
    // per wave 4 KB: the feature vectors, then the staged output rows
    __shared__ float4_t stage[kFrameWaves][64 * kMaxOut / 4];
    // A small launch is a chain of memory latencies: the table's entries, the
    // weights and the first queries are all on their way before the first wait.
    static_assert(kMaxTextures * kMaxLevels <= kFrameThreads, "one table entry per thread");
    uint4 entry;
    if (threadIdx.x < kMaxTextures * kMaxLevels) entry = (&a.lut.e[0][0])[threadIdx.x];

    // the wave index is uniform across the wave: say so, so that everything
    // derived from it (work items, materials, offsets) lives in SGPRs
    const uint32_t lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(a.ws + a.lay.scratch_off, (uint32_t)a.lay.scratch_bytes);
    const __amdgpu_buffer_rsrc_t rq = make_rsrc(a.queries, a.n * 12u);
    const __amdgpu_buffer_rsrc_t ro = make_rsrc(a.out, a.n * a.out_dim * 4u);
    MfmaMlp<K, H, NH> mlp;
    mlp.load(a.ws, a.lay, lane);
    float *st = reinterpret_cast<float *>(&stage[wv][0]);
    float4_t (*feats)[4] = reinterpret_cast<float4_t (*)[4]>(&stage[wv][0]);

    const uint32_t oob = a.n * a.out_dim * 4u;
    const WaveWork w = wave_work(a, wv);
    // the table to LDS; a wave without items only helps with that
    auto have_items = [&]() {
        if (threadIdx.x < kMaxTextures * kMaxLevels) (&lut.e[0][0])[threadIdx.x] = entry;
        __syncthreads();
        return w.first < w.end;
    };
    const ItemRange items{w.first, w.end, w.step};
    auto run = [&](auto kind) {
        constexpr ItemKind KIND = decltype(kind)::value;
        const LaneItem li = lane_item<KIND>(a, lane);
        // item k of this wave's share, all scalar
        auto locate = [&](uint32_t k) -> Item {
            uint32_t tr, tc;
            if (w.per) {
                uint32_t rem;
                const uint32_t j = divide_by(k, w.per, a.per_inv, rem);
                tr = (j * kXcds + w.xcd) * a.strip_rows + divide_by(rem, a.tiles_x, a.tiles_x_inv, tc);
            } else {
                tr = divide_by(k, a.tiles_x, a.tiles_x_inv, tc);
            }
            if (KIND == kItemLinear) return Item{64u * (tr * a.tiles_x + tc), 0, 0};   // rows of tiles_x items
            return Item{tr * kTileH * a.grid_w + tc * kTileW, a.grid_w - tc * kTileW, a.rows - tr * kTileH};
        };
        auto query = [&](uint32_t k) { return item_query<KIND>(a, rq, locate(k), li, lane); };
        Item item{0, 0, 0};
        const Query q0 = query(w.first < w.end ? w.first : 0);
        if (!have_items()) return;
        if (LAYOUT != kLayoutSplit) {
            // Per item: blend its texels, run the MLP, issue the next item's
            // texel loads and the query after that, then store -- so the
            // wait for the next texels never includes these stores. The loop
            // is entered the way it repeats (texel loads, a query load, the
            // stores), and the last item fetches its first item again, so
            // every path into the loop's top has the same loads and stores
            // outstanding.
            using Taps = std::conditional_t<LAYOUT == kLayoutPacked, PendingPacked, PendingTaps>;
            auto fetch = [&](const Query &q, Taps &t) {
                if constexpr (LAYOUT == kLayoutPacked) fetch4_packed(rs, lut, a.levels_bias, q.u, q.v, q.s, t);
                else fetch4_shared(rs, lut, a.levels_bias, a.stride, q.u, q.v, q.s, t);
            };
            auto clamp_item = [&](uint32_t k) { return k < items.end ? k : items.first; };
            Taps taps;
            fetch(q0, taps);
            Query qnext = query(clamp_item(items.first + items.step));
            store_dummies<KIND>(ro, oob);
            for (uint32_t k = items.first; k < items.end; k += items.step) {
                item = locate(k);
                float z[12];
                if constexpr (LAYOUT == kLayoutPacked) filter_pending_packed(taps, z);
                else filter_pending(taps, z);
                mlp_stage<true, K, H, NH>(z, mlp, feats, st, a.out_dim, lane);
                fetch(qnext, taps);
                qnext = query(clamp_item(k + 2 * items.step));
                store_item<KIND>(a, oob, st, ro, item, li, lane);
                wave_lds_sync();
            }
        } else {
            // the next item's query is loaded while this item's texels are
            // fetched; fetching texels ahead too costs registers and so waves:
            // 1366 x 768 bf16 27.9 -> 28.0 us, 300,000 points 29.6 -> 42.5
            Query next = q0;
            for (uint32_t k = items.first; k < items.end; k += items.step) {
                item = locate(k);
                const Query qq = next;
                if (k + items.step < items.end) next = query(k + items.step);
                decode_wave<true, K, H, NH, kLayoutSplit>(qq, rs, lut, a.levels_bias, a.stride, mlp, feats, st,
                                                          a.out_dim, lane);
                store_item<KIND>(a, oob, st, ro, item, li, lane);
                wave_lds_sync();
            }
        }
        if constexpr (KIND == kItemLinear) store_rest(a, st, ro, item, lane);
    };
    if (!a.grid_w)
        run(std::integral_constant<ItemKind, kItemLinear>());
    else if (a.row_rest)
        run(std::integral_constant<ItemKind, kItemTileRest>());
    else
        run(std::integral_constant<ItemKind, kItemTile>());
}

// The fp32 features and hidden layers on the vector ALU, recording each layer's
// largest input magnitude (the static fp8 activation scales come from a
// calibration batch).
template <int H, int NH, int LAYOUT>
__global__ void __launch_bounds__(kFrameThreads) k_calibrate(FrameArgs a)
{
    __shared__ LevelLut lut;
    copy_lut(a.lut, lut);
    const __amdgpu_buffer_rsrc_t rs = make_rsrc(a.ws + a.lay.scratch_off, (uint32_t)a.lay.scratch_bytes);
    const __amdgpu_buffer_rsrc_t rq = make_rsrc(a.queries, a.n * 12u);
    float amax[NH + 1];
#pragma unroll
    for (int l = 0; l <= NH; ++l) amax[l] = 0.0f;
    for (uint32_t q = blockIdx.x * blockDim.x + threadIdx.x; q < a.n; q += gridDim.x * blockDim.x) {
        const Query qq = load_query(rq, q);
        float z[12];
        filter4<LAYOUT>(rs, lut, a.levels_bias, a.stride, qq.u, qq.v, qq.s, z);
        mlp_maxima<H, NH>(a.ws, a.lay, z, amax);
    }
#pragma unroll
    for (int l = 0; l <= NH; ++l) {
        // non-negative floats order like their bit patterns
        atomicMax(reinterpret_cast<unsigned int *>(a.absmax) + l, __builtin_bit_cast(unsigned int, amax[l]));
    }
}

// ---------------------------------------------------------------------------
// Many materials in one launch. Every material has its own pyramids, texel
// scratch and MLP weights (one MLP shape for all); its queries are a
// contiguous range of the concatenated query array. Work items are runs of 64
// queries of one material, numbered material after material.

// A wave-uniform value loaded from memory, moved to SGPRs.
__device__ __forceinline__ uint32_t uniform(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ uint64_t uniform64(uint64_t v)
{
    return ((uint64_t)uniform((uint32_t)(v >> 32)) << 32) | uniform((uint32_t)v);
}

struct BatchMat {
    LevelLut lut;                          // as FrameArgs, offsets within the material's scratch
    float levels_bias[2 * kMaxTextures];
    uint64_t scratch_off, weights_off;     // bytes from the workspace start
    uint32_t scratch_bytes, stride, shared, interleaved;   // interleaved: as MaterialDesc
    uint32_t seg_chunk[kMaxLevels];        // interleaved: first unpack chunk of each level's segment
};

struct BatchArgs {
    const uint8_t *ws;
    const BatchMat *mats;                  // [n_mats], in the workspace
    const uint32_t *offsets;               // caller's [n_mats + 1] first query of each material
    uint32_t *items;                       // [n_mats + 1] first item of each material (BatchItems: past 64)
    WsLayout lay;                          // weight layout relative to a material's weights_off
    const float *queries;
    float *out;
    uint32_t n_mats, n_total, out_dim;
    uint32_t interleave;                   // 1: waves interleave runs of items; 0: contiguous ranges
    uint32_t run;                          // interleaved: consecutive items (of 64 queries) a wave takes
};

// Query range of material k: the caller's offsets clamped to [0, n_total],
// made non-decreasing, at most kMaxQueriesPerLaunch queries.
__device__ __forceinline__ void batch_range(const BatchArgs &a, uint32_t k, uint32_t &q0, uint32_t &cnt)
{
    q0 = min(a.offsets[k], a.n_total);
    const uint32_t q1 = max(min(a.offsets[k + 1], a.n_total), q0);
    cnt = min(q1 - q0, (uint32_t)kMaxQueriesPerLaunch);
}

// The work items of a batch as a wave sees them: which material an item
// belongs to, and a material's queries and first items. Up to 64 materials,
// lane k holds material k and every wave adds the prefix up by itself, so
// there is no launch for it and finding an item's material is a ballot; more
// are read from BatchArgs::items (k_batch_items), by binary search. Two
// materials of some thousand queries, with their unpack: 25.2 -> 21.0 us; eight
// with the touched blocks' 88.7 -> 84.1; 24 of 5.5 million 455.5 -> 454.9.
constexpr uint32_t kWaveItems = 64;

struct BatchItems {
    const BatchArgs &a;
    bool held;                             // in lanes
    uint32_t start, q0, cnt, total;        // held: of this lane's material; start = total past n_mats

    __device__ __forceinline__ BatchItems(const BatchArgs &args, uint32_t lane)
        : a(args), held(args.n_mats <= kWaveItems), start(0), q0(0), cnt(0), total(0)
    {
        if (!held) {
            total = uniform(a.items[a.n_mats]);
            return;
        }
        if (lane < a.n_mats) batch_range(a, lane, q0, cnt);
        const uint32_t n = (cnt + 63u) / 64u;
        uint32_t v = n;                    // inclusive scan across the wave
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t t = __shfl_up(v, d);
            if (lane >= (uint32_t)d) v += t;
        }
        start = v - n;
        total = __builtin_amdgcn_readlane(v, 63);
    }

    static __device__ __forceinline__ uint32_t lane_of(uint32_t v, uint32_t k)
    {
        return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)k);
    }

    // the material of item `it` < total: the last one that starts at or before
    // it (empty materials share their first item with the next one)
    __device__ __forceinline__ uint32_t find(uint32_t it) const
    {
        if (held) return (uint32_t)__popcll(__ballot(start <= it)) - 1u;
        uint32_t lo = 0, hi = a.n_mats;
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (a.items[mid] <= it) lo = mid;
            else hi = mid;
        }
        return uniform(lo);
    }

    // material k: its first query and query count, its first item and the next material's
    __device__ __forceinline__ void range(uint32_t k, uint32_t &first_q, uint32_t &n, uint32_t &first,
                                          uint32_t &next) const
    {
        if (held) {
            first_q = lane_of(q0, k);
            n = lane_of(cnt, k);
            first = lane_of(start, k);
            next = first + (n + 63u) / 64u;
            return;
        }
        batch_range(a, k, first_q, n);
        first_q = uniform(first_q);
        n = uniform(n);
        first = uniform(a.items[k]);
        next = uniform(a.items[k + 1]);
    }
};

// W waves per workgroup (the autotuner picks 2 or 4).
template <MlpKind K, int H, int NH, int W>
__global__ void __launch_bounds__(64 * W) k_batch(BatchArgs a)
{
    __shared__ LevelLut lut[W];                           // each wave's current material
    __shared__ float4_t stage[W][64 * kMaxOut / 4];       // features, then output rows
    // the wave index is uniform across the wave: say so, so that everything
    // derived from it (work items, materials, offsets) lives in SGPRs
    const uint32_t lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float *st = reinterpret_cast<float *>(&stage[wv][0]);
    float4_t (*feats)[4] = reinterpret_cast<float4_t (*)[4]>(&stage[wv][0]);
    const BatchItems all(a, lane);
    const uint32_t total = all.total;

    // interleaved: wave g takes runs of `run` consecutive items, g-th run of
    // every gridDim.x * W; contiguous: the XCD's band split into one range per wave
    ItemRange items;
    uint32_t run = 1;
    if (a.interleave) {
        run = max(a.run, 1u);
        items = ItemRange{(blockIdx.x * W + wv) * run, total, gridDim.x * W * run};
    } else {
        const uint32_t xcd = blockIdx.x % kXcds, local = blockIdx.x / kXcds;
        const uint32_t waves = (gridDim.x / kXcds) * W, w = local * W + wv;
        const uint64_t lo = (uint64_t)total * xcd / kXcds, hi = (uint64_t)total * (xcd + 1) / kXcds;
        items.first = (uint32_t)(lo + (hi - lo) * w / waves);
        items.end = (uint32_t)(lo + (hi - lo) * (w + 1) / waves);
        items.step = 1;
    }

    MfmaMlp<K, H, NH> mlp;
    uint32_t cur = 0xFFFFFFFFu, first_item = 0, n_k = 0, shared = 0, interleaved = 0, stride = 0;
    float lb[2 * kMaxTextures];
    __amdgpu_buffer_rsrc_t rs = make_rsrc(a.ws, 0), rq = rs, ro = rs;
    for (uint32_t it0 = items.first; it0 < items.end; it0 += items.step)
    for (uint32_t it = it0; it < min(it0 + run, items.end); ++it) {
        const uint32_t k = all.find(it);
        if (k != cur) {
            cur = k;
            const BatchMat &M = a.mats[cur];
            lut[wv].e[lane >> 4][lane & 15] = M.lut.e[lane >> 4][lane & 15];
#pragma unroll
            for (int j = 0; j < 2 * kMaxTextures; ++j)
                lb[j] = __builtin_bit_cast(float, uniform(__builtin_bit_cast(uint32_t, M.levels_bias[j])));
            shared = uniform(M.shared);
            interleaved = uniform(M.interleaved);
            stride = uniform(M.stride);
            rs = make_rsrc(a.ws + uniform64(M.scratch_off), uniform(M.scratch_bytes));
            uint32_t q0, next_item;
            all.range(cur, q0, n_k, first_item, next_item);
            rq = make_rsrc(a.queries + 3ull * q0, n_k * 12u);
            ro = make_rsrc(a.out + (uint64_t)a.out_dim * q0, n_k * a.out_dim * 4u);
            mlp.load(a.ws + uniform64(M.weights_off), a.lay, lane);
            wave_lds_sync();
        }
        const uint32_t j = it - first_item;
        const Query qq = load_query(rq, j * 64 + lane);   // past n_k: zeros, not stored
        if (interleaved)
            decode_wave_interleaved<false, K, H, NH>(qq, rs, lut[wv], lb, mlp, feats, st, a.out_dim, lane);
        else if (shared)
            decode_wave<false, K, H, NH, kLayoutShared>(qq, rs, lut[wv], lb, stride, mlp, feats, st, a.out_dim, lane);
        else
            decode_wave<false, K, H, NH, kLayoutSplit, true>(qq, rs, lut[wv], lb, stride, mlp, feats, st, a.out_dim, lane);
        store_run(stage[wv], ro, j, n_k, a.out_dim, lane);
        wave_lds_sync();
    }
}

template <MlpKind K>
hipError_t launch_batch_kind(const BatchArgs &a, const MlpShape &sh, unsigned grid, uint32_t waves, hipStream_t s)
{
#define BCF_CASE(H, NH)                                                                       \
    if (sh.hidden == H && sh.n_hidden == NH) {                                               \
        if (waves == 2) k_batch<K, H, NH, 2><<<grid, 128, 0, s>>>(a);                      \
        else k_batch<K, H, NH, 4><<<grid, 256, 0, s>>>(a);                                 \
        return hipGetLastError();                                                             \
    }
    BCF_CASE(16, 1) BCF_CASE(16, 2) BCF_CASE(16, 3)
    BCF_CASE(32, 1) BCF_CASE(32, 2) BCF_CASE(32, 3)
    BCF_CASE(64, 1) BCF_CASE(64, 2) BCF_CASE(64, 3)
#undef BCF_CASE
    return hipErrorInvalidValue;
}

// Workgroups of KERNEL resident at once on the current device, 0 if the
// runtime cannot say (cached per kernel and device; concurrent first calls
// compute the same value).
template <auto KERNEL>
unsigned resident_workgroups()
{
    static std::atomic<int> cache[16];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) return 0;
    if (dev < 16) {
        const int c = cache[dev].load(std::memory_order_relaxed);
        if (c > 0) return (unsigned)c;
    }
    int per_cu = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, KERNEL, kFrameThreads, 0) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    const int r = std::max(per_cu, 1) * std::max(cus, 1);
    if (dev < 16) cache[dev].store(r, std::memory_order_relaxed);
    return (unsigned)r;
}

// One workgroup per kFrameWaves items, at most `cap`, a multiple of the XCDs.
// The cap is the workgroups resident at once: every wave then loads its weights
// and fills its pipeline once and takes the same share of the items. With twice
// as many, the later half of the workgroups paid both again, which a 4K frame
// does not show (158 against 161 us with fp16) and smaller work does: 1920 x
// 1080 fp16 37 against 47 us, 960 x 540 15 / 18, 2^20 points 33 / 36, the same
// points with fp32 55 / 60.
inline unsigned frame_launch_grid(uint32_t n_items, unsigned cap)
{
    const unsigned want = (n_items + kFrameWaves - 1) / kFrameWaves;
    cap = std::max(kXcds, cap / kXcds * kXcds);
    return std::min(std::max(kXcds, (want + kXcds - 1) / kXcds * kXcds), cap);
}

template <MlpKind K, int SH>
hipError_t launch_frame_kind(const FrameArgs &a, const MlpShape &sh, hipStream_t s)
{
#define BCF_CASE(H, NH)                                                                       \
    if (sh.hidden == H && sh.n_hidden == NH) {                                               \
        const unsigned res = resident_workgroups<k_frame<K, H, NH, SH>>();                \
        k_frame<K, H, NH, SH>                                                                 \
            <<<frame_launch_grid(a.n_items, res ? res : 1024u), kFrameThreads, 0, s>>>(a); \
        return hipGetLastError();                                                             \
    }
    BCF_CASE(16, 1) BCF_CASE(16, 2) BCF_CASE(16, 3)
    BCF_CASE(32, 1) BCF_CASE(32, 2) BCF_CASE(32, 3)
    BCF_CASE(64, 1) BCF_CASE(64, 2) BCF_CASE(64, 3)
#undef BCF_CASE
    return hipErrorInvalidValue;
}

// per-precision entry points (frame_<precision>.hip)
// layout: kLayoutSplit, kLayoutShared or kLayoutPacked (filter_device.hpp)
hipError_t launch_frame_f32(const FrameArgs &a, const MlpShape &sh, int layout, hipStream_t s);
hipError_t launch_frame_f16(const FrameArgs &a, const MlpShape &sh, int layout, hipStream_t s);
hipError_t launch_frame_bf16(const FrameArgs &a, const MlpShape &sh, int layout, hipStream_t s);
hipError_t launch_frame_fp8(const FrameArgs &a, const MlpShape &sh, int layout, hipStream_t s);
hipError_t launch_calibrate_kernel(const FrameArgs &a, const MlpShape &sh, int layout, unsigned grid,
                                   hipStream_t s);
hipError_t launch_batch_f16(const BatchArgs &a, const MlpShape &sh, unsigned grid, uint32_t waves, hipStream_t s);
hipError_t launch_batch_f32(const BatchArgs &a, const MlpShape &sh, unsigned grid, uint32_t waves, hipStream_t s);

}  // namespace bcf
