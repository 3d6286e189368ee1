// S3 of one task by a workgroup of 16 waves (the stand-alone select kernel and the combine kernel that carries it along).
#pragma once

#include "floe_dev.h"

namespace floe {

// idx[0 .. count) = ascending { j : |v_j| > th }.  Each wave owns a contiguous slice of the channels and requests all its
// values (or kHold chunks of it at a time) before it looks at the first one: taken chunk by chunk, the slice cost one round
// trip to memory per chunk and pass (two tasks, f 14336: 10.4 -> 5.4 us).  pad: entries past count become -1, otherwise they
// stay as they are.
__device__ __forceinline__ void select_task(const float* __restrict__ vt, int f, float th, int32_t* __restrict__ it,
                                            int32_t* __restrict__ count, bool pad) {
    constexpr int kWaves = 16;
    constexpr int kHold = 16;  // chunks whose values a wave holds: one request round up to f = 16384
    __shared__ int wave_total[kWaves];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    // slice of this wave: a multiple of 64 channels
    const int chunks = (f + kWave - 1) / kWave;
    const int chunks_per_wave = (chunks + kWaves - 1) / kWaves;
    const int c0 = wave * chunks_per_wave;
    const int c1 = min(chunks, c0 + chunks_per_wave);
    // the selected channels of chunk c + k as a wave mask
    uint64_t m[kHold];
    auto look = [&](int c) {
        float a[kHold];
#pragma unroll
        for (int k = 0; k < kHold; ++k) a[k] = vt[min((c + k) * kWave + lane, f - 1)];
#pragma unroll
        for (int k = 0; k < kHold; ++k) m[k] = __ballot(c + k < c1 && (c + k) * kWave + lane < f && fabsf(a[k]) > th);
    };

    int total = 0;
    for (int c = c0; c < c1; c += kHold) {
        look(c);
#pragma unroll
        for (int k = 0; k < kHold; ++k) total += __popcll(m[k]);
    }
    if (lane == 0) wave_total[wave] = total;
    __syncthreads();
    int base = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const int n = wave_total[w];
        base += w < wave ? n : 0;
        all += n;
    }
    if (tid == 0) *count = all;
    if (pad)
        for (int i = all + tid; i < f; i += kWaves * kWave) it[i] = -1;
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    for (int c = c0; c < c1; c += kHold) {
        if (c1 - c0 > kHold) look(c);  // (a slice of one round is still in its masks)
#pragma unroll
        for (int k = 0; k < kHold; ++k) {
            if ((m[k] >> lane) & 1ull) it[base + __popcll(m[k] & below)] = (c + k) * kWave + lane;
            base += __popcll(m[k]);
        }
    }
}

}  // namespace floe
