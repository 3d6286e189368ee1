// S2 for batches in which an expert sees many tokens: V = X . W_up^Q on the matrix cores (Alg. 1 line 2; the paper itself is
// batch-1, each token keeps its own threshold, mask and result).  The arithmetic is that of up_gemv_mfma.hip: codes masked
// in place as fp16 subnormals, activations scaled by powers of two, scale and zero applied per quantization group in fp32.
//
//   x_frag_kernel   per token, once: the activations in the order and scaling of the matrix instruction's operand, their
//                   sums per quantization group, the factor that undoes the scaling.  (Every workgroup of the grouped
//                   kernel prepares them for itself; with many tokens per expert that would be most of its work.)
//   up_wide_kernel  a wave takes 32 channels (two tiles of 16) for all tokens of a group (up to 64: four token tiles); one
//                   slice of activations brought into LDS serves the 512 channels of sixteen waves.  Codes stream from
//                   memory into registers, a slice of four units (256 columns) ahead; activations pass through LDS in the
//                   same slices.
//
// What bounds it: vector instructions beside the matrix ones (54 % and 24 % of the cycles at 512 tokens): 18 per tile and
// unit to mask the codes, 8 per tile, unit and token tile for scale and zero.  Tiles without tokens are skipped for that
// reason.  8 experts d 4096 f 14336 INT2, 512 tokens: 386 us with the grouped kernel -> 296 us (both kernels; 280 on another
// card); tried: four channel tiles per wave with eight waves 395 us, two workgroups of eight waves per compute unit 344 us.
//
// Division of work: the blocks of 32 channels of all groups form one sequence that is cut into equal pieces, one workgroup
// each (see wide_batch.hip).
#include "floe_dev.h"
#include "launch.h"
#include "mfma_codes.h"

namespace floe {

constexpr int kUpWaves = 16;
constexpr int kUpThreads = kUpWaves * 64;
constexpr int kUpTiles = 2;                  // channel tiles per wave
constexpr int kUpChan = 16 * kUpTiles;       // channels per wave: one mask word
constexpr int kUpWgChan = kUpWaves * kUpChan;
constexpr int kSliceUnits = 4;               // units of 64 codes per slice

// fragment order and scaling of up_gemv_mfma.hip, one token per workgroup, one unit per thread (d <= 8192)
template <int BITS, bool G32>
__global__ __launch_bounds__(128) void x_frag_kernel(const h16* __restrict__ x, int d, uint4* __restrict__ frag,
                                                     float* __restrict__ gsum, float* __restrict__ back) {
    using Tr = MfmaTraits<BITS, G32>;
    constexpr int kGroups = G32 ? 2 : 1;
    constexpr float kScaleBack = (float)(1 << (24 - Tr::kPmax));
    __shared__ float wmax[2];
    const int t = blockIdx.x, U = threadIdx.x, units = d >> 6;
    const bool live = U < units;
    uint4 q[8];
    float amax = 0.0f;
    const uint4* xr = reinterpret_cast<const uint4*>(x + (size_t)t * d) + (live ? U : 0) * 8;
#pragma unroll
    for (int r = 0; r < 8; ++r) q[r] = xr[r];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const uint32_t wds[4] = {q[r].x, q[r].y, q[r].z, q[r].w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const h16x2 p = as_h2(wds[k]);
            amax = fmaxf(amax, fmaxf(fabsf((float)p.x), fabsf((float)p.y)));
        }
    }
    amax = wave_allreduce_max_nonneg(amax);
    if ((U & 63) == 0) wmax[U >> 6] = amax;
    __syncthreads();
    amax = fmaxf(wmax[0], wmax[1]);
    const int down = (amax >= 512.0f && amax < 3.0e38f) ? ilogbf(amax) - 8 : 0;  // |x'| < 512: 2^(pmax - p) x' stays finite
    if (U == 0) back[t] = ldexpf(1.0f, down) * kScaleBack;
    if (!live) return;
    const h16 ps = (h16)ldexpf(1.0f, -down);
    const h16x2 ps2 = {ps, ps}, ones = {(h16)1.0f, (h16)1.0f};
    uint32_t xv[32];
    float sum[2] = {0.0f, 0.0f};
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const uint32_t wds[4] = {q[r].x, q[r].y, q[r].z, q[r].w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const h16x2 p = as_h2(wds[k]) * ps2;
            xv[4 * r + k] = as_u32(p);
            sum[G32 ? (r >> 2) : 0] = __builtin_amdgcn_fdot2(p, ones, sum[G32 ? (r >> 2) : 0], false);
        }
    }
    uint4* out = frag + ((size_t)t * units + U) * 8;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            uint32_t w[4];
#pragma unroll
            for (int pr = 0; pr < 4; ++pr) {
                const int lo = Tr::code(j, g, 2 * pr), hi = Tr::code(j, g, 2 * pr + 1);
                const uint32_t wl = xv[lo >> 1], wh = xv[hi >> 1];
                const uint32_t l16 = (lo & 1) ? (wl >> 16) : (wl & 0xFFFFu);
                const uint32_t h16b = (hi & 1) ? (wh & 0xFFFF0000u) : (wh << 16);
                const h16x2 mul = {(h16)(float)(1 << (Tr::kPmax - Tr::pos(j, 2 * pr))),
                                   (h16)(float)(1 << (Tr::kPmax - Tr::pos(j, 2 * pr + 1)))};
                w[pr] = as_u32(as_h2(l16 | h16b) * mul);
            }
            out[j * 4 + g] = make_uint4(w[0], w[1], w[2], w[3]);
        }
    // (times 2^(pmax - 24), which the matrix products carry and the zero-point term is subtracted under)
#pragma unroll
    for (int k = 0; k < kGroups; ++k) gsum[((size_t)t * units + U) * kGroups + k] = sum[k] * (1.0f / kScaleBack);
}

template <int BITS, bool G32, int NT>
__global__ __launch_bounds__(kUpThreads) void up_wide_kernel(const WideGroup* __restrict__ groups,
                                                             const int32_t* __restrict__ n_groups, const int32_t* __restrict__ order,
                                                             const uint4* __restrict__ frag, const float* __restrict__ gsum,
                                                             const float* __restrict__ back, int slots, float* __restrict__ v,
                                                             const float* __restrict__ task_tau, uint32_t* __restrict__ mask_words,
                                                             int d, int f, int parts) {
    using Tr = MfmaTraits<BITS, G32>;
    constexpr int kTok = 16 * NT;
    constexpr int kGroups = G32 ? 2 : 1;                       // quantization groups per unit
    constexpr int kPieces = kSliceUnits * 8;                   // 16-byte pieces of a token per slice
    constexpr int kRounds = (kTok * kPieces + kUpThreads - 1) / kUpThreads;
    constexpr int kSums = kSliceUnits * kGroups;               // group sums of a token per slice
    constexpr int kSuperScales = 16;                           // scales per channel that sit in LDS at a time ...
    constexpr int kSuper = kSuperScales / kSums;               // ... those of so many slices
    __shared__ uint4 xs[2][kTok * kPieces];                    // [token][piece ^ (token & 15)]
    __shared__ __align__(16) float xg[2][kSums * kTok];        // [sum][token]
    __shared__ uint32_t meta[2][kSuperScales * kUpWgChan];  // [scale index][channel of the workgroup] (scale, zero)
    __shared__ int s_task[kTok];
    __shared__ float s_tau[kTok], s_back[kTok];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int c = lane & 15, g4 = lane >> 4;
    const int units = d >> 6, ns = units / kSliceUnits;        // an even number of slices (d % 512 == 0)
    const int blocks = (f + kUpChan - 1) / kUpChan;            // of 32 channels, per group
    const int total = n_groups[0] * parts * blocks;
    const int piece = wide_piece(gridDim.x);
    int pos = wide_cut(total, gridDim.x, piece);
    const int end = wide_cut(total, gridDim.x, piece + 1);
    const int nwords = mask_words_per_task(f);

    while (pos < end) {
        const int gi = __builtin_amdgcn_readfirstlane(pos / blocks);
        const int b0 = pos - gi * blocks;
        const int len = min(blocks - b0, end - pos);
        pos += len;
        const WideGroup grp = groups[gi / parts];
        // a group of more tokens than the accumulators take is cut into `parts`
        const int part_len = (grp.n + parts - 1) / parts;
        const int tok_first = (gi % parts) * part_len, n_tok = min(part_len, grp.n - tok_first);
        if (n_tok <= 0) continue;
        const unsigned char* codes = scalar_ptr(grp.e.codes);
        const unsigned char* scale = scalar_ptr(grp.e.scale);
        const unsigned char* zero = scalar_ptr(grp.e.zero);
        __syncthreads();  // the previous part's arrays are no longer read
        if (tid < kTok) {
            const int task = order[grp.first + tok_first + (tid < n_tok ? tid : 0)];  // dead token rows repeat the first one
            s_task[tid] = task;
            s_tau[tid] = task_tau ? task_tau[task] : 0.0f;
            s_back[tid] = back[task / slots];
        }
        __syncthreads();
        // byte offsets of this thread's pieces of a slice (T * d * 2 <= 64 MiB) and of its group sums: (token, unit of the slice)
        uint32_t xo[kRounds];
#pragma unroll
        for (int r = 0; r < kRounds; ++r)
            xo[r] = ((uint32_t)(s_task[min((tid + r * kUpThreads) / kPieces, kTok - 1)] / slots) * (uint32_t)units * 8u + tid % kPieces) * 16u;
        const int sum_tok = min(tid / kSliceUnits, kTok - 1), sum_u = tid % kSliceUnits;
        const uint32_t so = ((uint32_t)(s_task[sum_tok] / slots) * (uint32_t)units + sum_u) * (4u * kGroups);
        const unsigned char* frag8 = reinterpret_cast<const unsigned char*>(frag);
        const unsigned char* gsum8 = reinterpret_cast<const unsigned char*>(gsum);

        const int np = (len + kUpWaves - 1) / kUpWaves;
        const int per = (len + np - 1) / np;
        for (int p0 = 0; p0 < len; p0 += per) {
            const bool active = wave < per && p0 + wave < len;
            const int ch0 = (b0 + p0 + wave) * kUpChan;
            // Waves without channels repeat the last active one's requests (they are served by the cache): with their own,
            // a launch of few blocks read the codes and scales of its neighbours' channels eight times over (one expert,
            // 24 tokens, d 4096 f 14336: 36 -> 32 us).
            const int n_active = min(per, len - p0);
            const int load0 = (b0 + p0 + min(wave, n_active - 1)) * kUpChan;
            uint4 xq[kRounds];
            float sq[kGroups];
            // (requests are unconditional - past the end they repeat the last slice - so that the compiler can count them)
            auto load_x = [&](int s) {
                const int ss = min(s, ns - 1);
#pragma unroll
                for (int r = 0; r < kRounds; ++r) xq[r] = gload16(frag8 + (xo[r] + (uint32_t)ss * (kPieces * 16)));
#pragma unroll
                for (int k = 0; k < kGroups; ++k) sq[k] = gloadf(gsum8 + (so + (uint32_t)(ss * kSums + k) * 4u));
            };
            auto store_x = [&](int buf) {
#pragma unroll
                for (int r = 0; r < kRounds; ++r) {
                    const int i = tid + r * kUpThreads, tok = i / kPieces;
                    if (tok < kTok) xs[buf][tok * kPieces + ((i % kPieces) ^ (tok & 15))] = xq[r];
                }
                if (tid < kTok * kSliceUnits) {
#pragma unroll
                    for (int k = 0; k < kGroups; ++k) xg[buf][(sum_u * kGroups + k) * kTok + sum_tok] = sq[k];
                }
            };
            uint32_t co[kUpTiles];  // byte offsets of this lane's channels (f <= 65536 rows of at most 4 KiB)
#pragma unroll
            for (int t = 0; t < kUpTiles; ++t)
                co[t] = (uint32_t)min(load0 + 16 * t + c, f - 1) * (uint32_t)(units * BITS * 8) + g4 * (BITS * 8);  // clamped lanes never store
            // scales (lower half of the threads) and zeros (upper half): a thread brings in those of one channel
            const int m_ch = tid % kUpWgChan, m_half = tid / kUpWgChan;
            static_assert(kUpThreads == 2 * kUpWgChan, "a thread per channel for the scales and one for the zeros");
            const uint32_t mo = (uint32_t)min((b0 + p0) * kUpChan + min(m_ch, n_active * kUpChan - 1), f - 1) * (uint32_t)(units * kGroups * 2);
            const unsigned char* msrc = m_half ? zero : scale;
            uint4 mq[2];
            auto load_meta = [&](int super) {
                const uint32_t o = mo + (uint32_t)min(super * kSuperScales, units * kGroups - 8) * 2u;
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    mq[h] = gload16(msrc + (o + (super * kSuperScales + 8 * h < units * kGroups ? 16u * h : 0u)));
            };
            auto store_meta = [&](int buf) {
                uint16_t* m16 = reinterpret_cast<uint16_t*>(&meta[buf][m_ch]) + m_half;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint32_t w[4] = {mq[h].x, mq[h].y, mq[h].z, mq[h].w};
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        m16[(8 * h + 2 * k) * 2 * kUpWgChan] = (uint16_t)w[k];
                        m16[(8 * h + 2 * k + 1) * 2 * kUpWgChan] = (uint16_t)(w[k] >> 16);
                    }
                }
            };
            CodeSlice<BITS> cs[kUpTiles];
            auto load_c = [&](int s) {
                const uint32_t o = (uint32_t)min(s, ns - 1) * (kSliceUnits * BITS * 8);
#pragma unroll
                for (int t = 0; t < kUpTiles; ++t) cs[t].load(codes, co[t] + o);
            };
            load_meta(0);
            load_x(0);
            __builtin_amdgcn_sched_barrier(0);  // the waits of the loop count the requests in this order
            load_c(0);
            __builtin_amdgcn_sched_barrier(0);
            store_meta(0);
            store_x(0);
            load_x(1);
            __syncthreads();
            f32x4 acc[kUpTiles][NT];
#pragma unroll
            for (int t = 0; t < kUpTiles; ++t)
#pragma unroll
                for (int n = 0; n < NT; ++n) acc[t][n] = f32x4{0.f, 0.f, 0.f, 0.f};

            auto slice = [&](int s, int in_super, int mbuf) {
                const int buf = s & 1;
                // operand words of the four units: wd[t][u][k]
                uint32_t wd[kUpTiles][kSliceUnits][CodeSlice<BITS>::kLaneWords];
#pragma unroll
                for (int t = 0; t < kUpTiles; ++t) cs[t].deal(wd[t]);
                load_c(s + 1);
                store_x(buf ^ 1);
                load_x(s + 2);
                __builtin_amdgcn_sched_barrier(0);
                if (active) {
#pragma unroll
                for (int u = 0; u < kSliceUnits; ++u) {
                    {
                        // scale and zero of the unit's group(s).  Widened once per tile and unit, and kept so: left as halves they
                        // go into mixed-precision FMAs, which issue at half the rate of plain ones.
                        float sc[kUpTiles][2], zr[kUpTiles][2];
                        uint32_t r0[kUpTiles][4], r1[kUpTiles][4];
#pragma unroll
                        for (int tt = 0; tt < kUpTiles; ++tt) {
                            const int t = tt;
                            const uint32_t* mp = &meta[mbuf][(in_super * kSums + u * kGroups) * kUpWgChan + wave * kUpChan + 16 * t + c];
#pragma unroll
                            for (int k = 0; k < kGroups; ++k) {
                                const h16x2 m = as_h2(mp[k * kUpWgChan]);
                                sc[tt][k] = (float)m.x;
                                zr[tt][k] = (float)m.y;
                                asm volatile("" : "+v"(sc[tt][k]), "+v"(zr[tt][k]));
                            }
                            weight_frag24<BITS, G32>(wd[t][u], 0, r0[tt]);
                            weight_frag24<BITS, G32>(wd[t][u], 1, r1[tt]);
                        }
#pragma unroll
                        for (int n = 0; n < NT; ++n) {
                            if (n > 0 && 16 * n >= n_tok) break;  // token tiles without tokens (the same for the whole workgroup)
                            const h16x8 x0 = __builtin_bit_cast(h16x8, xs[buf][(16 * n + c) * kPieces + ((8 * u + g4) ^ c)]);
                            const h16x8 x1 = __builtin_bit_cast(h16x8, xs[buf][(16 * n + c) * kPieces + ((8 * u + 4 + g4) ^ c)]);
                            const f32x4 sg0 = *reinterpret_cast<const f32x4*>(&xg[buf][(u * kGroups) * kTok + 16 * n + 4 * g4]);
                            const f32x4 sg1 = *reinterpret_cast<const f32x4*>(&xg[buf][(u * kGroups + kGroups - 1) * kTok + 16 * n + 4 * g4]);
                            const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                            for (int tt = 0; tt < kUpTiles; ++tt) {
                                f32x4& ac = acc[tt][n];
                                if constexpr (G32) {
                                    const f32x4 c0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(x0, as_h8(r0[tt]), zero4, 0, 0, 0);
                                    const f32x4 c1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(x1, as_h8(r1[tt]), zero4, 0, 0, 0);
#pragma unroll
                                    for (int i = 0; i < 4; ++i) {
                                        const float t0 = fmaf(-zr[tt][0], sg0[i], c0[i]);
                                        const float t1 = fmaf(-zr[tt][kGroups - 1], sg1[i], c1[i]);
                                        ac[i] = fmaf(sc[tt][kGroups - 1], t1, fmaf(sc[tt][0], t0, ac[i]));
                                    }
                                } else {
                                    f32x4 cc = __builtin_amdgcn_mfma_f32_16x16x32_f16(x0, as_h8(r0[tt]), zero4, 0, 0, 0);
                                    cc = __builtin_amdgcn_mfma_f32_16x16x32_f16(x1, as_h8(r1[tt]), cc, 0, 0, 0);
#pragma unroll
                                    for (int i = 0; i < 4; ++i) ac[i] = fmaf(sc[tt][0], fmaf(-zr[tt][0], sg0[i], cc[i]), ac[i]);
                                }
                                asm volatile("" : "+v"(ac));  // here, not later: the products of a whole slice would wait in registers
                            }
                        }
                    }
                }
                }
                __syncthreads();
            };
            for (int s0 = 0, mbuf = 0; s0 < ns; s0 += kSuper, mbuf ^= 1) {
                load_meta(s0 / kSuper + 1);
                const int n_in = min(kSuper, ns - s0);
#pragma unroll 1
                for (int k = 0; k < n_in; ++k) slice(s0 + k, k, mbuf);
                store_meta(mbuf ^ 1);
                __syncthreads();
            }
            if (!active) continue;
            // lane (c, g4) holds channel ch0 + 16 t + c for tokens 16 n + 4 g4 + i
            int tok0 = 4 * g4;
            asm volatile("" : "+v"(tok0));  // or the addresses below are formed ahead of the loop and held across it
#pragma unroll
            for (int n = 0; n < NT; ++n)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int tok = 16 * n + tok0 + i;
                    const bool live = tok < n_tok;
                    const int task = s_task[tok];
                    const float bk = s_back[tok], tau = s_tau[tok];
                    float* vt = v + (size_t)task * f;
                    uint32_t w = 0u;
#pragma unroll
                    for (int t = 0; t < kUpTiles; ++t) {
                        const int ch = ch0 + 16 * t + c;
                        const float val = acc[t][n][i] * bk;
                        if (live && ch < f) vt[ch] = val;
                        const uint64_t m = __ballot(live && ch < f && fabsf(val) > tau);
                        w |= ((uint32_t)(m >> (16 * g4)) & 0xFFFFu) << (16 * t);
                    }
                    if (mask_words && live && c == 0) mask_words[(size_t)task * nwords + ch0 / 32] = w;
                }
        }
    }
}

size_t up_wide_scratch_bytes(int T, int d, int group) {
    return (size_t)T * d * 2 + (size_t)T * (d / 64) * (group == 32 ? 2 : 1) * 4 + (size_t)T * 4;
}

template <int BITS, bool G32, int NT>
static void launch_nt(const UpWideArgs& a, uint4* frag, float* gsum, float* back, hipStream_t stream) {
    up_wide_kernel<BITS, G32, NT><<<dim3(a.workgroups), dim3(kUpThreads), 0, stream>>>(
        a.groups, a.n_groups, a.order, frag, gsum, back, a.slots, a.v, a.task_tau, a.mask_words, a.d, a.f, a.parts);
}
template <int BITS, bool G32>
static hipError_t launch_bits(const UpWideArgs& a, hipStream_t stream) {
    uint4* frag = static_cast<uint4*>(a.scratch);
    float* gsum = reinterpret_cast<float*>(frag + (size_t)a.T * a.d / 8);
    float* back = gsum + (size_t)a.T * (a.d / 64) * (G32 ? 2 : 1);
    x_frag_kernel<BITS, G32><<<dim3(a.T), dim3(128), 0, stream>>>(a.x, a.d, frag, gsum, back);
    switch (a.nt) {
        case 1: launch_nt<BITS, G32, 1>(a, frag, gsum, back, stream); break;
        case 2: launch_nt<BITS, G32, 2>(a, frag, gsum, back, stream); break;
        case 3: launch_nt<BITS, G32, 3>(a, frag, gsum, back, stream); break;
        case 4:
            if constexpr (BITS == 2) {
                launch_nt<BITS, G32, 4>(a, frag, gsum, back, stream);
                break;
            }
            return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_up_wide(UpWideArgs a, int bits, int group, hipStream_t stream) {
    if (!up_wide_shape(a.d, a.f, bits, group)) return hipErrorInvalidValue;
    if (a.single) {
        const hipError_t rc = launch_wide_single(*a.single, a.n_tasks, a.chunk, const_cast<WideGroup*>(a.groups),
                                                 const_cast<int32_t*>(a.n_groups), const_cast<int32_t*>(a.order), stream);
        if (rc != hipSuccess) return rc;
    }
    // token tiles that the registers take beside the codes: four for INT2, three for the wider codes
    const int max_tiles = bits == 2 ? 4 : 3;
    a.parts = (a.nt + max_tiles - 1) / max_tiles;
    a.nt = (a.nt + a.parts - 1) / a.parts;
    const long long blocks = (long long)a.est_groups * a.parts * ((a.f + kUpChan - 1) / kUpChan);
    a.workgroups = (int)(blocks < num_cus() ? blocks : num_cus());
    if (a.workgroups > 8) a.workgroups &= ~7;  // (see wide_piece)
    const bool g32 = group == 32;
    if (bits == 2) return launch_bits<2, false>(a, stream);
    if (bits == 3) return g32 ? launch_bits<3, true>(a, stream) : launch_bits<3, false>(a, stream);
    return g32 ? launch_bits<4, true>(a, stream) : launch_bits<4, false>(a, stream);
}

}  // namespace floe
