// BC6H block unpacking for the decode kernels (gfx950).
//
// Implements the BC6H format definition that Section 4.2 of the paper
// ("Trainable BC6 decompression") defers to, in its exact integer form:
// endpoint unquantisation (the integer form of eq. 6), weighted blending of
// the two endpoints of the texel's subset (eq. 7), and the scale by 31/64
// (unsigned) or 31/32 (signed) whose result is reinterpreted as a half
// (eq. 8).
//
// Layout strategy (branch-free across lanes holding different modes):
//  * In every two-subset mode the main runs of the header fields sit at the
//    same block positions: w at 5/15/25, x at 35/45/55, gy[3:0] at 41,
//    gz[3:0] at 51, by[3:0] at 61, ry at 65, rz at 71, partition at 77.
//    Only their lengths change with the mode.
//  * The remaining header bits are single "extra" bits (gy4, gy5, by4, by5,
//    gz4, gz5, bz0..bz5 and bit 10 of w) whose positions a small per-mode
//    table lists.
//  * One-subset modes store x in the 10-bit chunks at 35/45/55 and the
//    endpoint bits above 10 of w reversed at the top of those chunks.
// So one instruction stream decodes all 14 modes.
//
// Everything here is __host__ __device__ so the same code can be exercised
// on the CPU.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace bcf {

// ---------------------------------------------------------------------------
// bit helpers (the device compiler maps them to v_bfe / v_alignbit / v_bfrev)

// x's bits off .. off + len - 1, zero- or sign-extended; len 0 gives 0. Both
// use the low five bits of off and len (as v_bfe does).
__host__ __device__ __forceinline__ uint32_t ubits(uint32_t x, uint32_t off, uint32_t len)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_ubfe(x, off, len);
#else
    len &= 31u;
    return len ? (x >> (off & 31u)) & (0xFFFFFFFFu >> (32u - len)) : 0u;
#endif
}

__host__ __device__ __forceinline__ int32_t sbits(uint32_t x, uint32_t off, uint32_t len)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_sbfe((int32_t)x, off, len);
#else
    const uint32_t v = ubits(x, off, len), s = 32u - (len & 31u);
    return (len & 31u) ? (int32_t)(v << s) >> s : 0;
#endif
}

__host__ __device__ __forceinline__ int32_t sext(uint32_t x, uint32_t len)
{
    // sign-extend the low `len` (1..32) bits
    const uint32_t s = 32u - len;
    return (int32_t)(x << s) >> s;
}

__host__ __device__ __forceinline__ uint32_t funnel(uint32_t hi, uint32_t lo, uint32_t s)
{
    return (uint32_t)((((uint64_t)hi << 32) | lo) >> s);
}

// the high halves of lo and hi, packed
__host__ __device__ __forceinline__ uint32_t pack_high(uint32_t lo, uint32_t hi)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_perm(hi, lo, 0x07060302u);
#else
    return (lo >> 16) | (hi & 0xFFFF0000u);
#endif
}

// lo | hi << 16 for 16-bit lo and hi. On the GPU one byte permute: written as
// a shift, the compiler folds the shift into the multiply that produced hi,
// turning a full-rate 24-bit multiply into a quarter-rate 32-bit one.
__host__ __device__ __forceinline__ uint32_t pack_lo_hi(uint32_t lo, uint32_t hi)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
#else
    return (lo & 0xFFFFu) | (hi << 16);
#endif
}

// ---------------------------------------------------------------------------
// per-mode descriptors

// word 0: [0] valid [1] two subsets [2] transformed [3..7] endpoint bits
//         [8..11] delta bits r [12..15] g [16..19] b
//         [20..23] one-subset modes: w bits above 10 stored reversed in x's chunk
//         [24..31] where extra bits sit when not in their usual word (kIn...),
//         and whether w has an 11th bit of its own (two-subset modes)
// words 1..4: extra bits, one byte each, 0x80 | block position, 0 = absent:
//         gy4 gy5 by4 by5 | gz4 gz5 bz0 bz1 | bz2 bz3 bz4 bz5 | rw10 gw10 bw10 -
// (an absent bit lies above its field's width and is dropped with the rest)
constexpr int kModeWords = 5;
constexpr int kModes = 15;                 // row 0: reserved codes
constexpr int kPartitions = 32;
// mode rows, a word per partition (kPartitionRow on), then per partition two words: bit t of
// its mask at bit 4 t + 3 (texels 0..7, 8..15), as the palette slots take it
constexpr int kPartitionRow = kModes * kModeWords;
constexpr int kSpreadRow = kPartitionRow + kPartitions;
constexpr int kTableWords = kSpreadRow + 2 * kPartitions;

// Words of the extra bits by mode: most sit in one of the block's words except
// in the few modes that these flags mark.
constexpr uint32_t kIn2710 = 1u << 24, kIn4 = 1u << 25, kIn5 = 1u << 26, kIn2810 = 1u << 27, kIn2910 = 1u << 28,
                   kIn1 = 1u << 29, kIn8 = 1u << 30, kW10 = 1u << 31;

#define BCF_INFO(two, tr, eb, dr, dg, db, kh)                                                 \
    (1u | ((uint32_t)(two) << 1) | ((uint32_t)(tr) << 2) | ((uint32_t)(eb) << 3) |          \
     ((uint32_t)(dr) << 8) | ((uint32_t)(dg) << 12) | ((uint32_t)(db) << 16) |               \
     ((uint32_t)(kh) << 20))
// bit t of m at bit 4 t + 3, texels 0..7 and 8..15
#define BCF_SPREAD4(m)                                                                        \
    (((m) & 1u) << 3 | ((m) & 2u) << 6 | ((m) & 4u) << 9 | ((m) & 8u) << 12 | ((m) & 16u) << 15 |   \
     ((m) & 32u) << 18 | ((m) & 64u) << 21 | ((m) & 128u) << 24)
#define BCF_SPREAD(m) BCF_SPREAD4((m) & 0xFFu), BCF_SPREAD4((m) >> 8)
#define BCF_AT(p) (0x80u | (uint32_t)(p))
#define BCF_BYTES(a, b, c, d)                                                                 \
    ((uint32_t)(a) | ((uint32_t)(b) << 8) | ((uint32_t)(c) << 16) | ((uint32_t)(d) << 24))

// mode rows, then per partition: subset-1 mask (bit t: texel t) | anchor << 16
static constexpr uint32_t kTable[kTableWords] = {
    // reserved
    0, 0, 0, 0, 0,
    // 1: 10-bit w, deltas 5/5/5
    BCF_INFO(1, 1, 10, 5, 5, 5, 0) | kIn1,
    BCF_BYTES(BCF_AT(2), 0, BCF_AT(3), 0), BCF_BYTES(BCF_AT(40), 0, BCF_AT(50), BCF_AT(60)),
    BCF_BYTES(BCF_AT(70), BCF_AT(76), BCF_AT(4), 0), 0,
    // 2: 7-bit w, deltas 6/6/6
    BCF_INFO(1, 1, 7, 6, 6, 6, 0) | kIn2710 | kIn2810 | kIn2910,
    BCF_BYTES(BCF_AT(24), BCF_AT(2), BCF_AT(14), BCF_AT(22)),
    BCF_BYTES(BCF_AT(3), BCF_AT(4), BCF_AT(12), BCF_AT(13)),
    BCF_BYTES(BCF_AT(23), BCF_AT(32), BCF_AT(34), BCF_AT(33)), 0,
    // 3: 11-bit w, deltas 5/4/4
    BCF_INFO(1, 1, 11, 5, 4, 4, 0) | kW10,
    0, BCF_BYTES(0, 0, BCF_AT(50), BCF_AT(60)), BCF_BYTES(BCF_AT(70), BCF_AT(76), 0, 0),
    BCF_BYTES(BCF_AT(40), BCF_AT(49), BCF_AT(59), 0),
    // 4: 11-bit w, deltas 4/5/4
    BCF_INFO(1, 1, 11, 4, 5, 4, 0) | kIn4 | kW10,
    BCF_BYTES(BCF_AT(75), 0, 0, 0), BCF_BYTES(BCF_AT(40), 0, BCF_AT(69), BCF_AT(60)),
    BCF_BYTES(BCF_AT(70), BCF_AT(76), 0, 0), BCF_BYTES(BCF_AT(39), BCF_AT(50), BCF_AT(59), 0),
    // 5: 11-bit w, deltas 4/4/5
    BCF_INFO(1, 1, 11, 4, 4, 5, 0) | kIn5 | kW10,
    BCF_BYTES(0, 0, BCF_AT(40), 0), BCF_BYTES(0, 0, BCF_AT(50), BCF_AT(69)),
    BCF_BYTES(BCF_AT(70), BCF_AT(76), BCF_AT(75), 0), BCF_BYTES(BCF_AT(39), BCF_AT(49), BCF_AT(60), 0),
    // 6: 9-bit w, deltas 5/5/5
    BCF_INFO(1, 1, 9, 5, 5, 5, 0),
    BCF_BYTES(BCF_AT(24), 0, BCF_AT(14), 0), BCF_BYTES(BCF_AT(40), 0, BCF_AT(50), BCF_AT(60)),
    BCF_BYTES(BCF_AT(70), BCF_AT(76), BCF_AT(34), 0), 0,
    // 7: 8-bit w, deltas 6/5/5
    BCF_INFO(1, 1, 8, 6, 5, 5, 0) | kIn2710,
    BCF_BYTES(BCF_AT(24), 0, BCF_AT(14), 0), BCF_BYTES(BCF_AT(13), 0, BCF_AT(50), BCF_AT(60)),
    BCF_BYTES(BCF_AT(23), BCF_AT(33), BCF_AT(34), 0), 0,
    // 8: 8-bit w, deltas 5/6/5
    BCF_INFO(1, 1, 8, 5, 6, 5, 0) | kIn2810 | kIn8,
    BCF_BYTES(BCF_AT(24), BCF_AT(23), BCF_AT(14), 0),
    BCF_BYTES(BCF_AT(40), BCF_AT(33), BCF_AT(13), BCF_AT(60)),
    BCF_BYTES(BCF_AT(70), BCF_AT(76), BCF_AT(34), 0), 0,
    // 9: 8-bit w, deltas 5/5/6
    BCF_INFO(1, 1, 8, 5, 5, 6, 0) | kIn2910,
    BCF_BYTES(BCF_AT(24), 0, BCF_AT(14), BCF_AT(23)),
    BCF_BYTES(BCF_AT(40), 0, BCF_AT(50), BCF_AT(13)),
    BCF_BYTES(BCF_AT(70), BCF_AT(76), BCF_AT(34), BCF_AT(33)), 0,
    // 10: four untransformed 6-bit endpoints
    BCF_INFO(1, 0, 6, 6, 6, 6, 0) | kIn2710 | kIn2810 | kIn2910,
    BCF_BYTES(BCF_AT(24), BCF_AT(21), BCF_AT(14), BCF_AT(22)),
    BCF_BYTES(BCF_AT(11), BCF_AT(31), BCF_AT(12), BCF_AT(13)),
    BCF_BYTES(BCF_AT(23), BCF_AT(32), BCF_AT(34), BCF_AT(33)), 0,
    // 11..14: one subset; x in the 10-bit chunks, top kh bits of a chunk = w[10..] reversed
    BCF_INFO(0, 0, 10, 10, 10, 10, 0), 0, 0, 0, 0,
    BCF_INFO(0, 1, 11, 9, 9, 9, 1), 0, 0, 0, 0,
    BCF_INFO(0, 1, 12, 8, 8, 8, 2), 0, 0, 0, 0,
    BCF_INFO(0, 1, 16, 4, 4, 4, 6), 0, 0, 0, 0,
    // partitions
    0xCCCCu | 15u << 16, 0x8888u | 15u << 16, 0xEEEEu | 15u << 16, 0xECC8u | 15u << 16,
    0xC880u | 15u << 16, 0xFEECu | 15u << 16, 0xFEC8u | 15u << 16, 0xEC80u | 15u << 16,
    0xC800u | 15u << 16, 0xFFECu | 15u << 16, 0xFE80u | 15u << 16, 0xE800u | 15u << 16,
    0xFFE8u | 15u << 16, 0xFF00u | 15u << 16, 0xFFF0u | 15u << 16, 0xF000u | 15u << 16,
    0xF710u | 15u << 16, 0x008Eu | 2u << 16,  0x7100u | 8u << 16,  0x08CEu | 2u << 16,
    0x008Cu | 2u << 16,  0x7310u | 8u << 16,  0x3100u | 8u << 16,  0x8CCEu | 15u << 16,
    0x088Cu | 2u << 16,  0x3110u | 8u << 16,  0x6666u | 2u << 16,  0x366Cu | 2u << 16,
    0x17E8u | 8u << 16,  0x0FF0u | 8u << 16,  0x718Eu | 2u << 16,  0x399Cu | 2u << 16,
    // spread masks
    BCF_SPREAD(0xCCCCu), BCF_SPREAD(0x8888u), BCF_SPREAD(0xEEEEu), BCF_SPREAD(0xECC8u),
    BCF_SPREAD(0xC880u), BCF_SPREAD(0xFEECu), BCF_SPREAD(0xFEC8u), BCF_SPREAD(0xEC80u),
    BCF_SPREAD(0xC800u), BCF_SPREAD(0xFFECu), BCF_SPREAD(0xFE80u), BCF_SPREAD(0xE800u),
    BCF_SPREAD(0xFFE8u), BCF_SPREAD(0xFF00u), BCF_SPREAD(0xFFF0u), BCF_SPREAD(0xF000u),
    BCF_SPREAD(0xF710u), BCF_SPREAD(0x008Eu), BCF_SPREAD(0x7100u), BCF_SPREAD(0x08CEu),
    BCF_SPREAD(0x008Cu), BCF_SPREAD(0x7310u), BCF_SPREAD(0x3100u), BCF_SPREAD(0x8CCEu),
    BCF_SPREAD(0x088Cu), BCF_SPREAD(0x3110u), BCF_SPREAD(0x6666u), BCF_SPREAD(0x366Cu),
    BCF_SPREAD(0x17E8u), BCF_SPREAD(0x0FF0u), BCF_SPREAD(0x718Eu), BCF_SPREAD(0x399Cu),
};

#undef BCF_INFO
#undef BCF_SPREAD
#undef BCF_SPREAD4
#undef BCF_AT
#undef BCF_BYTES

// Mode number (1..14, 0 = reserved) for each value of the low five bits: two
// bits 00/01 select modes 1/2 whatever follows; otherwise all five bits count.
__host__ __device__ __forceinline__ uint32_t mode_of(uint32_t d0)
{
    const uint32_t code = d0 & 31u;
    const uint64_t lut = code < 16 ? 0xE621D521C421B321ull : 0x0A21092108210721ull;
    return (uint32_t)(lut >> ((code & 15u) * 4u)) & 15u;
}

// ---------------------------------------------------------------------------
// unpacked header: for subset s and channel c the texel value before the final
// scale is (base[s][c] + w * diff[s][c]) >> 6, w = weight of the texel's index

struct Bc6hHeader {
    int32_t base[2][3];      // 64 * first endpoint + 32
    int32_t diff[2][3];      // second endpoint - first endpoint
    uint32_t mask;           // texels in subset 1 (0 for one-subset modes)
    uint64_t idx;            // texel t's index at bits [ib*t, ib*t+ib)
    uint32_t s0, s1;         // texel t's palette slot at bits 4t..4t+3 of s0 (t < 8) or s1
    uint32_t ib;             // index bits per texel: 3 or 4
    uint32_t valid;
};

// Eight 3-bit fields (bits 3k..3k+2 of x) moved to 4-bit nibbles (bits 4k..4k+2).
__host__ __device__ __forceinline__ uint32_t spread3to4(uint32_t x)
{
    x = (x & 0x00000FFFu) | ((x & 0x00FFF000u) << 4);      // fields 4..7 up by 4
    x = (x & 0x003F003Fu) | ((x & 0x0FC00FC0u) << 2);      // fields 2, 3, 6, 7 up by 2
    return (x & 0x07070707u) | ((x & 0x38383838u) << 1);   // fields 1, 3, 5, 7 up by 1
}

template <bool SIGNED>
__host__ __device__ __forceinline__ int32_t unquantize(int32_t e, uint32_t eb)
{
    if (!SIGNED) {
        // ((e << 16) + 2^15) >> eb; 0 and the top code map to 0 and 0xFFFF.
        // For eb = 16 the general expression already returns e.
        uint32_t u = (((uint32_t)e << 16) | 0x8000u) >> eb;
        u = e == 0 ? 0u : u;
        u = (uint32_t)e == (0xFFFFFFFFu >> (32u - eb)) ? 0xFFFFu : u;
        return (int32_t)u;
    } else {
        const uint32_t m = (uint32_t)(e < 0 ? -e : e);
        uint32_t u = ((m << 15) | 0x4000u) >> (eb - 1u);
        u = m == 0 ? 0u : u;
        u = m >= ((1u << (eb - 1u)) - 1u) ? 0x7FFFu : u;
        int32_t r = e < 0 ? -(int32_t)u : (int32_t)u;
        return eb >= 16u ? e : r;
    }
}

template <bool SIGNED>
__host__ __device__ __forceinline__ void bc6h_header(uint32_t d0, uint32_t d1, uint32_t d2,
                                                     uint32_t d3, const uint32_t *table,
                                                     Bc6hHeader &h)
{
    const uint32_t mode = mode_of(d0);
    const uint32_t *md = table + kModeWords * mode;
    const uint32_t info = md[0];
    const uint32_t o0 = md[1], o1 = md[2], o2 = md[3], o3 = md[4];   // extra bits: offsets in their low five bits
    const uint32_t two = (info >> 1) & 1u;
    const uint32_t eb = (info >> 3) & 31u;
    const uint32_t dw[3] = {(info >> 8) & 15u, (info >> 12) & 15u, (info >> 16) & 15u};
    const uint32_t kh = (info >> 20) & 15u, kw = info >> 31;
    h.valid = info & 1u;

    // w: low min(eb,10) bits at 5/15/25, then (bit 10 on) one extra bit in
    // two-subset modes, or the top kh bits of x's 10-bit chunk (35/45/55),
    // reversed, in one-subset modes; kw or kh is the count, the other 0
    const uint32_t wlen = eb < 10u ? eb : 10u;
    const uint32_t c2 = funnel(d2, d1, 23);                  // chunk 2 from bit 0
    const uint32_t r1 = __builtin_bitreverse32(d1), r2 = __builtin_bitreverse32(c2);
    const uint32_t w[3] = {
        ubits(d0, 5, wlen) | (ubits(d1, o3, kw) | ubits(r1, 19, kh)) << 10,
        ubits(d0, 15, wlen) | (ubits(d1, o3 >> 8, kw) | ubits(r1, 9, kh)) << 10,
        ubits(funnel(d1, d0, 25), 0, wlen) | (ubits(d1, o3 >> 16, kw) | ubits(r2, 22, kh)) << 10};
    // x, y, z: sign-extended (which the endpoint mask below undoes where they
    // are not deltas: there they have eb bits). The widths drop absent extras.
    const uint32_t g4 = ubits(info & kIn4 ? d2 : d0, o0, 1), g5 = ubits(d0, o0 >> 8, 1);
    const uint32_t b4 = ubits(info & kIn5 ? d1 : d0, o0 >> 16, 1), b5 = ubits(d0, o0 >> 24, 1);
    const uint32_t h4 = ubits(info & kIn2710 ? d0 : d1, o1, 1), h5 = ubits(info & kIn8 ? d1 : d0, o1 >> 8, 1);
    const uint32_t z0 = ubits(info & kIn2810 ? d0 : info & kIn4 ? d2 : d1, o1 >> 16, 1);
    const uint32_t z1 = ubits(info & kIn2910 ? d0 : info & kIn5 ? d2 : d1, o1 >> 24, 1);
    const uint32_t z2 = ubits(info & kIn2710 ? d0 : d2, o2, 1), z3 = ubits(info & kIn2710 ? d1 : d2, o2 >> 8, 1);
    const uint32_t z4 = ubits(info & kIn1 ? d0 : info & kIn5 ? d2 : d1, o2 >> 16, 1), z5 = ubits(d1, o2 >> 24, 1);
    const uint32_t gy = ubits(d1, 9, 4) | g4 << 4 | g5 << 5;                       // gy[3:0] at 41
    const uint32_t by = ubits(funnel(d2, d1, 29), 0, 4) | b4 << 4 | b5 << 5;       // by[3:0] at 61
    const uint32_t gz = ubits(d1, 19, 4) | h4 << 4 | h5 << 5;                      // gz[3:0] at 51
    const uint32_t bz = z0 | z1 << 1 | z2 << 2 | z3 << 3 | z4 << 4 | z5 << 5;
    const int32_t f[3][3] = {{sbits(d1, 3, dw[0]), sbits(d1, 13, dw[1]), sbits(c2, 0, dw[2])},
                             {sbits(d2, 1, dw[0]), sbits(gy, 0, dw[1]), sbits(by, 0, dw[2])},    // ry at 65
                             {sbits(d2, 7, dw[0]), sbits(gz, 0, dw[1]), sbits(bz, 0, dw[2])}};   // rz at 71

    // endpoints: x, y, z are deltas from w in transformed modes
    const uint32_t emask = 0xFFFFFFFFu >> ((32u - eb) & 31u);    // eb = 0 (reserved): every field is 0
    int32_t e[4][3];
    for (int c = 0; c < 3; ++c) {
        e[0][c] = SIGNED ? sext(w[c], eb ? eb : 1u) : (int32_t)w[c];
        const uint32_t from = info & 4u ? w[c] : 0u;
        for (int j = 0; j < 3; ++j) {
            const uint32_t v = (from + (uint32_t)f[j][c]) & emask;
            e[j + 1][c] = SIGNED ? sext(v, eb ? eb : 1u) : (int32_t)v;
        }
    }
    const uint32_t ebq = eb ? eb : 16u;      // reserved rows: any valid shift
    for (int s = 0; s < 2; ++s)
        for (int c = 0; c < 3; ++c) {
            const int32_t a = unquantize<SIGNED>(e[2 * s][c], ebq);
            const int32_t b = unquantize<SIGNED>(e[2 * s + 1][c], ebq);
            h.base[s][c] = 64 * a + 32;
            h.diff[s][c] = b - a;
        }

    // indices, every texel at its full width: the implicit zero top bit of
    // texel 0 and of the subset-1 anchor (texel 2, 8 or 15) re-inserted
    const uint32_t part = ubits(d2, 13, 5);
    if (two) {
        const uint32_t pinfo = table[kPartitionRow + part], anchor = pinfo >> 16;
        h.mask = pinfo & 0xFFFFu;
        h.ib = 3;
        // the stream starts at bit 82; lo: its bits 0..31 with texel 0's top
        // bit inserted, hi: bits 23..46 of that
        const uint32_t lo = (funnel(d3, d2, 17) & ~7u) | ubits(d2, 18, 2), hi = d3 >> 8;
        const uint32_t i0 = anchor == 2u ? (lo & 0xFFu) | (lo & 0x7FFF00u) << 1 : lo & 0xFFFFFFu;
        const uint32_t i1 = anchor == 2u ? hi : anchor == 8u ? (ubits(hi, 1, 2) | (hi & ~7u)) : hi >> 1;
        h.idx = (uint64_t)i1 << 24 | i0;
        const uint32_t *sp = table + kSpreadRow + 2 * part;
        h.s0 = spread3to4(i0) | sp[0];
        h.s1 = spread3to4(i1) | sp[1];
    } else {
        // bits 65..127, with texel 0's top bit inserted
        h.mask = 0;
        h.ib = 4;
        h.s0 = (d2 & ~15u) | ubits(d2, 1, 3);
        h.s1 = d3;
        h.idx = (uint64_t)d3 << 32 | h.s0;
    }
}

// Half bit pattern of texel t (0..15), channel c. Weights are the format's
// round(64 i / 7) and round(64 i / 15), computed as (i * 585 + 32) >> 6 and
// (i * 273 + 32) >> 6.
template <bool SIGNED>
__host__ __device__ __forceinline__ uint32_t bc6h_texel(const Bc6hHeader &h, uint32_t t, int c)
{
    // operands masked to their known widths (no-ops here) so the compiler can
    // use the full-rate 24-bit multiplies
    const uint32_t i = (uint32_t)(h.idx >> (h.ib * t)) & ((1u << h.ib) - 1u) & 15u;
    const uint32_t wt = (i * (h.ib == 3 ? 585u : 273u) + 32u) >> 6;
    const uint32_t s = (h.mask >> t) & 1u;
    const int32_t base = s ? h.base[1][c] : h.base[0][c];
    // |diff| < 2^17 and wt <= 64
    const int32_t diff = (int32_t)((uint32_t)(s ? h.diff[1][c] : h.diff[0][c]) << 8) >> 8;
    const int32_t v = (base + (int32_t)(wt & 127u) * diff) >> 6;   // arithmetic: floor
    uint32_t out;
    if (!SIGNED) {
        out = (((uint32_t)v & 0xFFFFFFu) * 31u) >> 6;                 // v <= 0xFFFF
    } else {
        const uint32_t m = (uint32_t)(v < 0 ? -v : v);
        out = (((m & 0xFFFFFFu) * 31u) >> 5) | (v < 0 ? 0x8000u : 0u); // |v| <= 0x7FFF
    }
    return h.valid ? out : 0u;
}

// The at most 16 distinct values a block's texels take, channels packed as
// (r | g << 16, b): entry j = 8 s + i for two-subset modes (3-bit index i of
// subset s), j = i for one-subset modes (4-bit index i). Each entry is the
// blend and finish of bc6h_texel for that subset and index (a reserved mode's
// endpoints are all 0: base 32, zeros). The finish (v 31) >> 6 (signed: >> 5) is
// taken as the high half of v (31 << 10) (31 << 11), which one byte permute
// packs for two channels.
template <bool SIGNED>
__host__ __device__ __forceinline__ void bc6h_palette(const Bc6hHeader &h, uint32_t pal[16][2])
{
    const bool two = h.ib == 3;
    // entries 0..7 blend subset 0; entries 8..15 subset 1 (two subsets) or
    // subset 0 again (one subset). |diff| < 2^17 and wt <= 64, so the products
    // fit the 24-bit multiply once diff is restated as a 24-bit value.
    int32_t base[2][3], diff[2][3];
    for (int c = 0; c < 3; ++c) {
        base[0][c] = h.base[0][c];
        diff[0][c] = (int32_t)((uint32_t)h.diff[0][c] << 8) >> 8;
        base[1][c] = two ? h.base[1][c] : h.base[0][c];
        diff[1][c] = (int32_t)((uint32_t)(two ? h.diff[1][c] : h.diff[0][c]) << 8) >> 8;
    }
#pragma unroll
    for (uint32_t j = 0; j < 16; ++j) {
        const int32_t wt = (int32_t)(two ? (((j & 7u) * 585u + 32u) >> 6) : ((j * 273u + 32u) >> 6));
        uint32_t ch[3];                              // in the high half
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const int32_t v = (base[j >> 3][c] + wt * diff[j >> 3][c]) >> 6;
            if (!SIGNED) {
                ch[c] = ((uint32_t)v & 0xFFFFFFu) * 31744u;                                      // v <= 0xFFFF
            } else {
                const uint32_t m = (uint32_t)(v < 0 ? -v : v);
                ch[c] = ((m & 0xFFFFFFu) * 63488u) | ((uint32_t)v & 0x80000000u);                // |v| <= 0x7FFF
            }
        }
        pal[j][0] = pack_high(ch[0], ch[1]);
        pal[j][1] = ch[2] >> 16;
    }
}

// Palette entry of texel t (0..15).
__host__ __device__ __forceinline__ uint32_t bc6h_slot(const Bc6hHeader &h, uint32_t t)
{
    const uint32_t i = (uint32_t)(h.idx >> (h.ib * t)) & ((1u << h.ib) - 1u);
    return h.ib == 3 ? ((((h.mask >> t) & 1u) << 3) | i) : i;
}

// Palette entries of all 16 texels, four bits each: texel t's bc6h_slot at
// bits 4t..4t+3 of s0 (t < 8) or s1 (t >= 8).
__host__ __device__ __forceinline__ void bc6h_slots(const Bc6hHeader &h, uint32_t &s0, uint32_t &s1)
{
    s0 = h.s0;
    s1 = h.s1;
}

}  // namespace bcf
