// Stores of the unpacked texels, shared by the unpack kernels and the training
// texels: a workgroup's block palettes and slots in LDS to the texel scratch.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "bc6h_device.hpp"
#include "filter_device.hpp"

namespace bcf {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
// Global-memory views of the scratch and of the blocks. Pointers that the
// batch kernel reads from its segment table are generic to the compiler,
// which would access them with flat instructions (a flat store also counts
// against the LDS wait counter, so every LDS read after one waits for the
// store); these casts keep every access a global one.
typedef __attribute__((address_space(1))) u32x4_t global_u32x4;
typedef __attribute__((address_space(1))) const u32x4_t global_block;
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(1))) u32x2_t global_texel;

// Two texels to the scratch as one 16-byte store. NT: non-temporal, past the
// caches (unpack_past_caches in api.cpp says when).
template <bool NT>
__device__ __forceinline__ void store_pair(uint2 *dst, uint2 t0, uint2 t1)
{
    const u32x4_t v = {t0.x, t0.y, t1.x, t1.y};
    if (NT) __builtin_nontemporal_store(v, (global_u32x4 *)dst);
    else *(global_u32x4 *)dst = v;
}

typedef uint32_t u32x3_t __attribute__((ext_vector_type(3)));
typedef __attribute__((address_space(1))) u32x3_t global_u32x3;

// Two pyramids' texels of one position of a packed scratch, (r, g, b) halves
// each, as one 12-byte store (dst 4-byte aligned). NT: as store_pair.
template <bool NT>
__device__ __forceinline__ void store_packed_pair(uint32_t *dst, uint2 t0, uint2 t1)
{
    const u32x3_t v = {t0.x, pack_lo_hi(t0.y, t1.x), pack_lo_hi(t1.x >> 16, t1.y)};
    if (NT) __builtin_nontemporal_store(v, (global_u32x3 *)dst);
    else *(global_u32x3 *)dst = v;
}

// Texel t (row-major) of the block in lane lb of the workgroup: its palette
// entry, (r | g << 16, b).
__device__ __forceinline__ uint2 palette_texel(const uint2 (*palette)[256], const uint2 *slots, uint32_t lb, uint32_t t)
{
    const uint2 sl = slots[lb];
    return palette[((t < 8 ? sl.x : sl.y) >> (4 * (t & 7))) & 15u][lb];
}

// The texels of a wave's 16 block positions (four lanes each, one per pyramid)
// to the packed scratch of a level of lw x lh texels: first, the wave's first
// position in the level (of n_blk); with `list` (LDS), the workgroup's positions
// are list[0 .. n_list) instead.
// Each block row is four 24-byte positions, 96 contiguous bytes; a store
// instruction writes eight block rows: lane L takes the 12 bytes of pyramids
// 2(L%2) and 2(L%2)+1 at position L % 8 / 2 of the row of block 8h + L / 8, read
// through LDS from that block's lanes. The store policy: store_packed_pair.
template <bool NT>
__device__ __forceinline__ void store_positions(uint32_t *pdst, uint32_t lw, uint32_t lh, uint32_t first,
                                                uint32_t n_blk, const uint2 (*palette)[256], const uint2 *slots,
                                                const uint32_t *list = nullptr, uint32_t n_list = 0)
{
    const uint32_t bx = (lw + 3) / 4, bxm = bx - 1u, bxs = (uint32_t)__builtin_ctz(bx), pitch = row_pitch(lw);
    const uint32_t lane = threadIdx.x & 63u, wave0 = threadIdx.x & ~63u;
    const uint32_t chunk8 = lane & 7u, pp = 2 * (lane & 1u), cpos = chunk8 >> 1;
    // a level's scratch is below 2 GB: byte offsets in 32 bits
    auto store = [&](uint32_t off, uint2 t0, uint2 t1) {
        store_packed_pair<NT>(reinterpret_cast<uint32_t *>(reinterpret_cast<uint8_t *>(pdst) + off), t0, t1);
    };
#pragma unroll
    for (uint32_t h = 0; h < 2; ++h) {
        const uint32_t blw = 8 * h + (lane >> 3);                     // block within the wave
        const uint32_t p = (wave0 >> 2) + blw;                        // within the chunk
        if (list ? p >= n_list : first + blw >= n_blk) continue;
        const uint32_t bj = list ? list[p] : first + blw;             // its index in the level
        const uint32_t lb = wave0 + 4 * blw + pp;                     // LDS lane of pyramid pp
        const uint32_t x0 = 4 * (bj & bxm), y0 = 4 * (bj >> bxs);
        if (lw >= 4 && lh >= 4) {
            // four whole rows: this lane's column of both blocks' slots, then
            // a nibble and a palette read per row and pyramid
            const uint2 sa = slots[lb], sb = slots[lb + 1];
            const uint32_t sh = 4 * cpos;
            const uint32_t wa[2] = {sa.x >> sh, sa.y >> sh}, wb[2] = {sb.x >> sh, sb.y >> sh};
            uint32_t off = 24u * (__umul24(y0, pitch) + x0 + cpos) + 12u * (pp >> 1);
#pragma unroll
            for (int r = 0; r < 4; ++r, off += 24u * pitch) {
                const uint2 p0 = palette[(wa[r >> 1] >> (16 * (r & 1))) & 15u][lb];
                const uint2 p1 = palette[(wb[r >> 1] >> (16 * (r & 1))) & 15u][lb + 1];
                store(off, p0, p1);
                if (x0 == 0 && cpos < 2) store(off + 24u * lw, p0, p1);   // wrap positions w, w + 1
            }
            continue;
        }
        for (uint32_t r = 0; r < 4; ++r) {
            if (y0 + r >= lh) break;
            // position index within the level (below 2^31: levels are at most 32768^2)
            const uint32_t prow = __umul24(y0 + r, pitch);
            // lw >= 4: texel column cpos; lw = 2: columns 0 1 0 1 (pitch 4);
            // lw = 1: texel 0 at positions 0 1 2 (pitch 3)
            if (lw == 1 && cpos >= 3) continue;
            const uint32_t col = lw >= 4 ? cpos : lw == 2 ? (cpos & 1u) : 0u;
            const uint2 p0 = palette_texel(palette, slots, lb, 4 * r + col);
            const uint2 p1 = palette_texel(palette, slots, lb + 1, 4 * r + col);
            store(24u * (prow + x0 + cpos) + 12u * (pp >> 1), p0, p1);
            if (lw >= 4 && x0 == 0 && cpos < 2)                        // wrap positions w, w + 1
                store(24u * (prow + lw + cpos) + 12u * (pp >> 1), p0, p1);
        }
    }
}

}  // namespace bcf
