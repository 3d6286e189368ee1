// Codes as matrix-core operands, shared by the kernels that run the up projection of several tokens on the matrix cores
// (up_gemv_mfma.hip, up_wide.hip, up_split.hip): how the codes of a unit are dealt to the lanes of an instruction, and how they become
// fp16 numbers without a conversion.
#pragma once

#include "floe_dev.h"

namespace floe {

typedef _Float16 h16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// How the 64 codes of a unit are dealt to the four lane quarters g and the two MFMAs j.
//  kLaneWords           code words a lane loads per unit
//  word(k, g)           index (inside the unit) of the lane's k-th word
//  code(j, g, s)        code index (0..63 inside the unit) that slot s of MFMA j holds in quarter g
//  pos(j, s)            bit position of that code's field inside its 16-bit half
//  kPmax                every product carries 2^(kPmax - 24)
// With one quantization group per unit (G32 = false) any dealing works because both MFMAs are summed
// before scaling; with groups of 32 MFMA j must cover exactly the codes 32j .. 32j+31.
template <int BITS, bool G32> struct MfmaTraits;
template <> struct MfmaTraits<2, false> {  // quarter g owns word g (codes 16g .. 16g+15)
    static constexpr int kLaneWords = 1;
    static constexpr int kPmax = 8;
    __device__ static constexpr int word(int k, int g) { (void)k; return g; }
    __device__ static constexpr int code(int j, int g, int s) {
        constexpr int t[2][8] = {{0, 8, 1, 9, 2, 10, 3, 11}, {4, 12, 5, 13, 6, 14, 7, 15}};
        return 16 * g + t[j][s];
    }
    __device__ static constexpr int pos(int j, int s) {
        constexpr int t[2][8] = {{4, 4, 6, 6, 4, 4, 6, 6}, {8, 8, 4, 4, 6, 6, 8, 8}};
        return t[j][s];
    }
};
template <bool G32> struct MfmaTraits<4, G32> {  // MFMA j reads word 4j + g: it covers codes 32j .. 32j+31
    static constexpr int kLaneWords = 2;
    static constexpr int kPmax = 6;
    __device__ static constexpr int word(int k, int g) { return 4 * k + g; }
    __device__ static constexpr int code(int j, int g, int s) {
        constexpr int t[8] = {0, 4, 1, 5, 2, 6, 3, 7};
        return 32 * j + 8 * g + t[s];
    }
    __device__ static constexpr int pos(int j, int s) {
        constexpr int t[8] = {4, 4, 4, 4, 2, 2, 6, 6};
        (void)j;
        return t[s];
    }
};

// INT3: the 32 codes of a half unit are 96 contiguous bits; quarter g owns the 24 bits [24g, 24g + 24) of them, which
// lie in words a, a + 1 of the half unit with a = g / 2.  A lane loads those two words itself (kOwnWords) and shifts
// its field down; codes 0..3 of the field stay in the low 16-bit half, codes 4..7 move to the high half.
template <bool G32> struct MfmaTraits<3, G32> {
    static constexpr int kLaneWords = 4;  // two words for each of the two MFMAs
    static constexpr int kPmax = 6;
    __device__ static constexpr int word(int k, int g) { return 3 * (k >> 1) + (g >> 1) + (k & 1); }
    __device__ static constexpr int code(int j, int g, int s) {
        constexpr int t[8] = {0, 4, 1, 5, 2, 6, 3, 7};
        return 32 * j + 8 * g + t[s];
    }
    __device__ static constexpr int pos(int j, int s) {
        constexpr int t[8] = {0, 0, 3, 3, 6, 6, 6, 6};
        (void)j;
        return t[s];
    }
};

// the 4 registers (8 fp16 subnormals) of MFMA j from the lane's code words
template <int BITS, bool G32>
__device__ __forceinline__ void weight_frag(const uint32_t* w, int j, int g, uint32_t (&r)[4]) {
    if (BITS == 3) {
        // w[2j], w[2j+1]: the two words that hold the quarter's 24 bits, at bit 24g - 32(g/2) of the pair
        const uint64_t pair = ((uint64_t)w[2 * j + 1] << 32) | w[2 * j];
        const uint32_t c24 = (uint32_t)(pair >> (24 * g - 32 * (g >> 1)));
        const uint32_t t = (c24 & 0x00000FFFu) | ((c24 << 4) & 0x0FFF0000u);
        r[0] = t & 0x00070007u;         // codes (0, 4) at bits [0,3)
        r[1] = t & 0x00380038u;         // codes (1, 5) at bits [3,6)
        r[2] = t & 0x01C001C0u;         // codes (2, 6) at bits [6,9)
        r[3] = (t >> 3) & 0x01C001C0u;  // codes (3, 7) from bits [9,12) to [6,9)
    } else if (BITS == 2 && !G32) {
        const uint32_t W = w[0], a = W << 4, b = W >> 6;
        if (j == 0) {
            r[0] = a & 0x00300030u;  // codes (0, 8)  at bits [4,6)
            r[1] = a & 0x00C000C0u;  // codes (1, 9)  at bits [6,8)
            r[2] = W & 0x00300030u;  // codes (2, 10) at bits [4,6)
            r[3] = W & 0x00C000C0u;  // codes (3, 11) at bits [6,8)
        } else {
            r[0] = W & 0x03000300u;  // codes (4, 12) at bits [8,10)
            r[1] = b & 0x00300030u;  // codes (5, 13) at bits [4,6)
            r[2] = b & 0x00C000C0u;  // codes (6, 14) at bits [6,8)
            r[3] = b & 0x03000300u;  // codes (7, 15) at bits [8,10)
        }
    } else {
        const uint32_t W = w[j], a = W << 4, b = W >> 6;
        r[0] = a & 0x00F000F0u;      // codes (0, 4) at bits [4,8)
        r[1] = W & 0x00F000F0u;      // codes (1, 5) at bits [4,8)
        r[2] = b & 0x003C003Cu;      // codes (2, 6) at bits [2,6)
        r[3] = b & 0x03C003C0u;      // codes (3, 7) at bits [6,10)
    }
}

// the same from operand words that are already the lane's own: INT2 w[0], INT4 w[j], INT3 the quarter's 24-bit field of half
// j in the low bits of w[j] (anything above)
template <int BITS, bool G32>
__device__ __forceinline__ void weight_frag24(const uint32_t* w, int j, uint32_t (&r)[4]) {
    if constexpr (BITS == 3) {
        const uint32_t t = (w[j] & 0x00000FFFu) | ((w[j] << 4) & 0x0FFF0000u);
        r[0] = t & 0x00070007u;
        r[1] = t & 0x00380038u;
        r[2] = t & 0x01C001C0u;
        r[3] = (t >> 3) & 0x01C001C0u;
    } else {
        weight_frag<BITS, G32>(w, j, 0, r);
    }
}

__device__ __forceinline__ h16x8 as_h8(const uint32_t (&r)[4]) {
    uint4 q = make_uint4(r[0], r[1], r[2], r[3]);
    return __builtin_bit_cast(h16x8, q);
}

__device__ __forceinline__ void transpose4(uint4& q) {  // across the four lane quarters: register k <- word g of quarter k's vector
    u32x2 t;
    t = __builtin_amdgcn_permlane32_swap(q.x, q.z, false, false); q.x = t.x; q.z = t.y;
    t = __builtin_amdgcn_permlane32_swap(q.y, q.w, false, false); q.y = t.x; q.w = t.y;
    t = __builtin_amdgcn_permlane16_swap(q.x, q.y, false, false); q.x = t.x; q.y = t.y;
    t = __builtin_amdgcn_permlane16_swap(q.z, q.w, false, false); q.z = t.x; q.w = t.y;
}

// word of quarter k -> rk in every lane
__device__ __forceinline__ void quarters_to_all(uint32_t w, uint32_t& r0, uint32_t& r1, uint32_t& r2, uint32_t& r3) {
    const u32x2 h = __builtin_amdgcn_permlane32_swap(w, w, false, false);  // lower and upper half, twice each
    const u32x2 a = __builtin_amdgcn_permlane16_swap(h.x, h.x, false, false), b = __builtin_amdgcn_permlane16_swap(h.y, h.y, false, false);
    r0 = a.x; r1 = a.y; r2 = b.x; r3 = b.y;
}

// A lane's codes (units 2 g and 2 g + 1 of quarter g) -> the operand words of units p, p + 2, p + 4, p + 6
template <int BITS, int VECS, int WORDS>
__device__ __forceinline__ void deal_units(const uint4 (&q)[VECS], int p, uint32_t (&wd)[4][WORDS]) {
    if constexpr (BITS == 3) {
        // a unit is two halves of 96 bits, four 24-bit fields each; field k goes to quarter k
        const uint32_t w[12] = {q[0].x, q[0].y, q[0].z, q[0].w, q[1].x, q[1].y, q[1].z, q[1].w, q[2].x, q[2].y, q[2].z, q[2].w};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t w0 = w[6 * p + 3 * h], w1 = w[6 * p + 3 * h + 1], w2 = w[6 * p + 3 * h + 2];
            uint4 fld = make_uint4(w0, __builtin_amdgcn_alignbit(w1, w0, 24), __builtin_amdgcn_alignbit(w2, w1, 16), w2 >> 8);
            transpose4(fld);
            wd[0][h] = fld.x; wd[1][h] = fld.y; wd[2][h] = fld.z; wd[3][h] = fld.w;
        }
    } else {
#pragma unroll
        for (int r = 0; r < WORDS; ++r) {
            uint4 w = q[p * WORDS + r];
            transpose4(w);
            wd[0][r] = w.x; wd[1][r] = w.y; wd[2][r] = w.z; wd[3][r] = w.w;
        }
    }
}

}  // namespace floe
