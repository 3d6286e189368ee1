// S0: asymmetric uniform group quantizer for the up projection (paper Sec. 3.2.2).
// Bit-exact contract (stated in include/floe.h): strict IEEE binary32, one rounding per operation,
// no fused multiply-add, correctly rounded division, round-half-even to integer and to fp16.
#include "floe_dev.h"
#include "launch.h"

namespace floe {

#pragma clang fp contract(off)

// A thread owns a half unit of 32 consecutive weights (four 16-byte loads); 1, 2, 4 or 8 neighbouring lanes make up a
// group, whose minimum and maximum meet by lane exchange.  Every thread derives its group's scale and zero, and its 32
// codes are exactly BITS words of the stream, so nothing is exchanged for the packing.  Channels follow one another in
// memory and a row is a whole number of half units, so the kernel walks the matrix as one sequence of them.
// What bounds it: the division per weight.  a / S is formed as a product with the reciprocal of S and two fused
// corrections (the remainder a - q S is exact in one FMA), which gives the correctly rounded quotient for the operands that
// occur here: S is an fp16 number of at least 2^-14 and a an fp16 number, so neither the quotient nor the remainder leaves
// the normal range unless a is zero (Markstein's correction; every pair of fp16 significands is checked in the tests).
// d 4096 f 14336 INT2: 50.6 us with a workgroup per channel, byte-wise packing through LDS and the compiler's division,
// 28.9 us (4.7 TB/s, the rate of a large copy) so.
__device__ __forceinline__ float div_by(float a, float s, float rcp) {
    float q = a * rcp;
    q = __builtin_fmaf(__builtin_fmaf(-q, s, a), rcp, q);
    return __builtin_fmaf(__builtin_fmaf(-q, s, a), rcp, q);
}

template <int BITS>
__global__ __launch_bounds__(256) void quantize_kernel(const h16* __restrict__ w, uint32_t* __restrict__ codes,
                                                       h16* __restrict__ scale, h16* __restrict__ zero, long long halves,
                                                       int lanes_per_group) {
    const float qmax = (float)((1 << BITS) - 1);
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    const bool live = i < halves;  // groups never straddle the end: halves is a multiple of lanes_per_group
    const uint4* src = reinterpret_cast<const uint4*>(w) + (live ? i : halves - 1) * 4;
    uint4 raw[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) raw[r] = src[r];
    float a[32];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint32_t wds[4] = {raw[r].x, raw[r].y, raw[r].z, raw[r].w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const h16x2 p = as_h2(wds[k]);
            a[8 * r + 2 * k] = (float)p.x;
            a[8 * r + 2 * k + 1] = (float)p.y;
        }
    }
    float mn = a[0], mx = a[0];
#pragma unroll
    for (int k = 1; k < 32; ++k) {
        mn = fminf(mn, a[k]);
        mx = fmaxf(mx, a[k]);
    }
    for (int o = 1; o < lanes_per_group; o <<= 1) {
        mn = fminf(mn, __shfl_xor(mn, o, kWave));
        mx = fmaxf(mx, __shfl_xor(mx, o, kWave));
    }
    h16 sh = (h16)((mx - mn) / qmax);  // v_cvt_f16_f32, round to nearest even
    const float S = (float)sh;
    const bool degenerate = !(mx > mn) || !(S >= 6.103515625e-05f) || __builtin_isinf(S);
    h16 zh;
    uint32_t q[32];
    if (degenerate) {
        sh = (h16)1.0f;
        zh = (h16)(-mn);
#pragma unroll
        for (int k = 0; k < 32; ++k) q[k] = 0;
    } else {
        float z32 = (-mn) / S;
        z32 = fminf(fmaxf(z32, -65504.0f), 65504.0f);
        zh = (h16)z32;
        const float Z = (float)zh;
        const float rcp = 1.0f / S;
#pragma unroll
        for (int k = 0; k < 32; ++k) {
            const float u = div_by(a[k], S, rcp) + Z;
            const float r = fminf(fmaxf(__builtin_rintf(u), 0.0f), qmax);
            q[k] = (uint32_t)r;
        }
    }
    if (!live) return;
    // word b of the half unit holds bits [32 b, 32 b + 32) of its stream
    uint32_t out[BITS];
#pragma unroll
    for (int b = 0; b < BITS; ++b) out[b] = 0u;
#pragma unroll
    for (int k = 0; k < 32; ++k) {
        const int bit = k * BITS, b = bit >> 5, s = bit & 31;
        out[b] |= q[k] << s;
        if (s + BITS > 32) out[b + 1 < BITS ? b + 1 : b] |= q[k] >> (32 - s);
    }
    uint32_t* dst = codes + i * BITS;
#pragma unroll
    for (int b = 0; b < BITS; ++b) dst[b] = out[b];
    if ((i & (lanes_per_group - 1)) == 0) {
        const long long g = i / lanes_per_group;
        scale[g] = sh;
        zero[g] = zh;
    }
}

hipError_t launch_quantize(const h16* w, uint32_t* codes, h16* scale, h16* zero, int d, int f, int bits, int group,
                           hipStream_t stream) {
    if (f == 0) return hipSuccess;
    const long long halves = (long long)f * (d / 32);
    dim3 grid((unsigned)((halves + 255) / 256)), block(256);
    const int lpg = group / 32;
    switch (bits) {
        case 1: quantize_kernel<1><<<grid, block, 0, stream>>>(w, codes, scale, zero, halves, lpg); break;
        case 8: quantize_kernel<8><<<grid, block, 0, stream>>>(w, codes, scale, zero, halves, lpg); break;
        case 2: quantize_kernel<2><<<grid, block, 0, stream>>>(w, codes, scale, zero, halves, lpg); break;
        case 3: quantize_kernel<3><<<grid, block, 0, stream>>>(w, codes, scale, zero, halves, lpg); break;
        default: quantize_kernel<4><<<grid, block, 0, stream>>>(w, codes, scale, zero, halves, lpg); break;
    }
    return hipGetLastError();
}

}  // namespace floe
