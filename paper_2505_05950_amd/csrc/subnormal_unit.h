// A unit of 64 codes against 64 activations in full fp32 precision, for every code width: a code field that is masked out of
// a 16-bit half and left where it is, at bits [p, p + b) with p + b <= 10, IS the fp16 subnormal q * 2^(p - 24), which a
// mixed-precision FMA widens exactly; two codes cost one AND, there is no conversion and no offset to take off again.  The
// activation that meets the field is pre-multiplied by 2^(kPmax - p), so that every product carries the same 2^(kPmax - 24).
// (v_dot2_f32_f16 would do both products at once, but drops low bits of products with subnormals: 1.5e-5 of v at INT2
// against 8e-8 here.)
#pragma once

#include "floe_dev.h"

namespace floe {

// Register reg (0..31) of a unit holds the activations of codes (lo, hi); their fields sit at bit pos of the two halves.
// Registers 0..15 belong to the first half unit (codes 0..31), 16..31 to the second.
//  INT1: word w gives registers 16 w + m, m < 16: codes (32 w + m, + 16); bits 10..15 after a shift by 6
//  INT2: word w gives registers 8 w + m,  m < 8:  codes (16 w + m, + 8);  fields at 10, 12, 14 after a shift by 6
//  INT3: half h (96 bits) gives registers 16 h + 5 k + i for three 30-bit chunks k, i < 5: codes (32 h + 10 k + i, + 5);
//        fields at 9 and 12 after a shift by 6; register 16 h + 15: codes (32 h + 30, 32 h + 31)
//  INT4: word w gives registers 4 w + m,  m < 4:  codes (8 w + m, + 4);   fields at 8 and 12 after a shift by 8
//  INT8: word w gives registers 2 w + m,  m < 2:  codes (4 w + m, + 2);   m = 1 after a shift by 8
template <int BITS> struct SubTraits;
template <> struct SubTraits<1> { static constexpr int kPmax = 9; };
template <> struct SubTraits<2> { static constexpr int kPmax = 8; };
template <> struct SubTraits<3> { static constexpr int kPmax = 6; };
template <> struct SubTraits<4> { static constexpr int kPmax = 4; };
template <> struct SubTraits<8> { static constexpr int kPmax = 0; };

template <int BITS>
__device__ constexpr void sub_layout(int reg, int& lo, int& hi, int& pos) {
    if (BITS == 1) {
        const int w = reg >> 4, m = reg & 15;
        lo = 32 * w + m; hi = lo + 16; pos = m < 10 ? m : m - 6;
    } else if (BITS == 2) {
        const int w = reg >> 3, m = reg & 7;
        lo = 16 * w + m; hi = lo + 8; pos = m < 5 ? 2 * m : 2 * m - 6;
    } else if (BITS == 4) {
        const int w = reg >> 2, m = reg & 3;
        lo = 8 * w + m; hi = lo + 4; pos = 4 * (m & 1);
    } else if (BITS == 8) {
        const int w = reg >> 1, m = reg & 1;
        lo = 4 * w + m; hi = lo + 2; pos = 0;
    } else {
        const int h = reg >> 4, r = reg & 15;
        if (r == 15) { lo = 32 * h + 30; hi = lo + 1; pos = 0; }
        else {
            const int k = r / 5, i = r % 5;
            lo = 32 * h + 10 * k + i; hi = lo + 5; pos = i < 3 ? 3 * i : 3 * i - 6;
        }
    }
}

// power-of-two down-scaling exponent: x' = x * 2^-down keeps 2^kPmax * |x'| below 2^15 in fp16
template <int BITS>
__device__ __forceinline__ int sub_down(float token_amax) {
    constexpr int kKeepBelow = 15 - SubTraits<BITS>::kPmax;
    const float lim = (float)(1 << (kKeepBelow - 1));
    return (token_amax >= lim && token_amax < 3.0e38f) ? ilogbf(token_amax) - (kKeepBelow - 1) : 0;
}

// raw[r] = (x[2r], x[2r+1]) of the unit -> xs[32], and Xg[h] = 2^(kPmax - 24) * sum of x' over half unit h
template <int BITS>
__device__ __forceinline__ void sub_prepare(const uint32_t (&raw)[32], int down, uint32_t (&xs)[32], float (&Xg)[2]) {
    constexpr int kPmax = SubTraits<BITS>::kPmax;
    const h16 ps = (h16)ldexpf(1.0f, -down);
    const h16x2 ps2 = {ps, ps};
    Xg[0] = Xg[1] = 0.0f;
#pragma unroll
    for (int reg = 0; reg < 32; ++reg) {
        int lo = 0, hi = 0, pos = 0;
        sub_layout<BITS>(reg, lo, hi, pos);
        const uint32_t A = raw[lo >> 1], B = raw[hi >> 1];
        const uint32_t a16 = (lo & 1) ? (A >> 16) : (A & 0xFFFFu), b16 = (hi & 1) ? (B & 0xFFFF0000u) : (B << 16);
        h16x2 p = as_h2(a16 | b16) * ps2;
        Xg[reg >> 4] += (float)p.x + (float)p.y;
        const h16 c = (h16)(float)(1 << (kPmax - pos));
        xs[reg] = as_u32(p * (h16x2){c, c});
    }
    Xg[0] *= 1.0f / (float)(1 << (24 - kPmax));
    Xg[1] *= 1.0f / (float)(1 << (24 - kPmax));
}

// four chains (two picked by `odd`): shorter chains of roundings
__device__ __forceinline__ void sub_fma2(uint32_t x2, uint32_t q2, float (&a)[4], int odd) {
    const h16x2 xp = as_h2(x2), qp = as_h2(q2);
    a[2 * odd] = fmaf((float)xp.x, (float)qp.x, a[2 * odd]);
    a[2 * odd + 1] = fmaf((float)xp.y, (float)qp.y, a[2 * odd + 1]);
}

// 2^(kPmax - 24) * sum over half unit h of x' q; cw: the unit's 2 * BITS code words
template <int BITS>
__device__ __forceinline__ float sub_half_dot(const uint32_t* cw, const uint32_t* xs, int h) {
    float a[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (BITS == 3) {
        const uint32_t w0 = cw[3 * h], w1 = cw[3 * h + 1], w2 = cw[3 * h + 2];
        const uint32_t chunk[3] = {w0, __builtin_amdgcn_alignbit(w1, w0, 30), __builtin_amdgcn_alignbit(w2, w1, 28)};
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const uint32_t t = (chunk[k] & 0x7FFFu) | ((chunk[k] << 1) & 0x7FFF0000u), b = t >> 6;
            const uint32_t* xr = xs + 16 * h + 5 * k;
            sub_fma2(xr[0], t & 0x00070007u, a, 0);
            sub_fma2(xr[1], t & 0x00380038u, a, 1);
            sub_fma2(xr[2], t & 0x01C001C0u, a, 0);
            sub_fma2(xr[3], b & 0x00380038u, a, 1);
            sub_fma2(xr[4], b & 0x01C001C0u, a, 0);
        }
        sub_fma2(xs[16 * h + 15], ((w2 >> 26) & 7u) | ((w2 >> 13) & 0x00070000u), a, 1);
        return (a[0] + a[1]) + (a[2] + a[3]);
    }
    constexpr int kShift = BITS <= 2 ? 6 : 8;
    constexpr int kRegs = 16 / BITS;                 // registers per word
    constexpr int kDirect = BITS == 1 ? 10 : (BITS == 2 ? 5 : (BITS == 4 ? 2 : 1));
#pragma unroll
    for (int w = BITS * h; w < BITS * h + BITS; ++w) {
        const uint32_t W = cw[w], b = W >> kShift;
#pragma unroll
        for (int m = 0; m < kRegs; ++m) {
            const int pos = m < kDirect ? BITS * m : BITS * m - kShift;
            const uint32_t mask = ((1u << BITS) - 1u) * 0x00010001u << pos;
            sub_fma2(xs[kRegs * w + m], (m < kDirect ? W : b) & mask, a, BITS == 1 ? m & 1 : w & 1);
        }
    }
    return (a[0] + a[1]) + (a[2] + a[3]);
}

}  // namespace floe
