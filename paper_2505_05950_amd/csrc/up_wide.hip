// S2 for batches in which an expert sees many tokens: V = X . W_up^Q on the matrix cores (Alg. 1 line 2; the paper itself is
// batch-1, each token keeps its own threshold, mask and result).  The arithmetic is that of up_gemv_mfma.hip: codes masked
// in place as fp16 subnormals, activations scaled by powers of two, scale and zero applied per quantization group in fp32.
//
//   up_wide_kernel  a wave takes two channel tiles of 16 for up to nine token tiles (INT3, INT4: five); the eight waves of a
//                   workgroup share the activations, which travel from memory straight into a ring of four slots in LDS, two
//                   units (128 columns) each, in operand order (x_operand_kernel in up_split.hip).  Codes, scales and zeros of
//                   eight units go to registers, half of eight units ahead.
//
// What bounds it: vector instructions (per unit and wave 24 to mask codes and widen scale and zero, 16 per token tile to apply them)
// and matrix products (four per token tile), which share the issue of the SIMD's two waves; the order in the loop deals products and
// multiply-adds one to four.  8 experts d 4096 f 14336 INT2, 512 tokens: 286 -> 224 us (before: sixteen waves, four token tiles, the
// codes unpacked three times); of that 8 to find the work, and per pass of 256 channels 6 until the ring is full and 8 for the
// results.  Tried: four channel tiles and up to four token tiles 297; pieces that do not end where groups end 266; operands fetched
// three items ahead (the same).
//
// Division of work: channel blocks of 32; each part of a group is cut into equal pieces, one workgroup each.
#include <atomic>
#include <type_traits>

#include "floe_dev.h"
#include "launch.h"
#include "mfma_codes.h"

namespace floe {

constexpr int kUpWaves = 8;
constexpr int kUpThreads = kUpWaves * 64;
constexpr int kUpSlotUnits = 2;

template <int BITS, bool G32, int NT>
__global__ __launch_bounds__(kUpThreads) void up_wide_kernel(const WideGroup* __restrict__ groups, int32_t* __restrict__ shares, const int32_t* __restrict__ n_groups,
                                                             int max_groups, const uint4* __restrict__ frag, const float* __restrict__ gsum,
                                                             const float* __restrict__ back, float* __restrict__ v,
                                                             const float* __restrict__ tau, uint32_t* __restrict__ mask_words,
                                                             int d, int f) {
    constexpr int CT = 2;                                // channel tiles of 16 per wave: one mask word
    constexpr int kTok = 16 * NT;
    constexpr int kGroups = G32 ? 2 : 1;                 // quantization groups per unit
    constexpr int kVec = BITS;                           // 16-byte vectors of codes per lane and tile: two units of eight
    constexpr int kMetaLoads = (CT * 2 * kGroups + 3) / 4;
    constexpr int kLaneWords = BITS == 2 ? 1 : 2;        // operand words per unit
    constexpr int kCh = 16 * CT;                         // channels per wave
    constexpr int kXVecs = kUpSlotUnits * 2 * NT * 64;   // per slot: activations, and behind them the group sums
    constexpr int kSumVecs = (kUpSlotUnits * kGroups * NT * 4 + 63) / 64 * 64;
    __shared__ uint4 x0[kXVecs + kSumVecs], x1[kXVecs + kSumVecs], x2[kXVecs + kSumVecs], x3[kXVecs + kSumVecs];
    __shared__ __align__(16) float s_tau[kTok], s_back[kTok];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int c = lane & 15, g4 = lane >> 4;
    const int units = d >> 6;
    const int blocks = (f + kCh - 1) / kCh;              // per part of a group
    const int nwords = mask_words_per_task(f);
    // A block of channels costs as much as it has token tiles to do, and two more for its codes; a group of more than NT tiles comes in
    // parts of equal size.
    const int ng = n_groups[0];
    auto parts_of = [](int n) { return (n + kTok - 1) / kTok; };
    auto part_tiles = [&](int n) { return (wide_tiles(n) + parts_of(n) - 1) / parts_of(n); };
    auto weight = [&](int n) { return part_tiles(n) + 2; };
    struct Share { int parts, part_weight; };
    const int n_here = groups[min(lane, max_groups - 1)].n;  // (the first 64 groups are asked for once)
    auto share_of = [&](int g0) {  // lane's group (the load does not wait for ng)
        const int n = g0 == 0 ? n_here : groups[min(g0 + lane, max_groups - 1)].n;
        return g0 + lane < ng ? Share{parts_of(n), weight(n) * blocks} : Share{0, 0};
    };
    int total = 0, n_parts = 0;
    for (int g0 = 0; g0 < ng; g0 += kWave) {
        const Share sh = share_of(g0);
        total += wave_sum(sh.parts * sh.part_weight);
        n_parts += wave_sum(sh.parts);
    }
    const int W = gridDim.x, piece = wide_piece(W);
    // Pieces end where parts end: a pass of the workgroup takes as long with one wave at work as with eight, so a piece that holds the
    // ends of two parts takes a pass more than its share, and the launch waits for it (512 tokens: 266 us, the mean piece 182).  Each
    // part is cut into as few equal pieces of at most `most` as it takes, `most` the smallest that leaves no more than W pieces.
    const bool whole = n_parts <= W;
    int most = max((total + W - 1) / W, 1);
    while (whole) {
        int sum = 0;
        for (int g0 = 0; g0 < ng; g0 += kWave) {
            const Share sh = share_of(g0);
            sum += wave_sum(sh.parts * ((sh.part_weight + most - 1) / most));
        }
        if (sum <= W) break;  // (at the largest part at the latest: a piece each)
        most += (most + 31) / 32;
    }
    int pos = whole ? piece : wide_cut(total, W, piece);
    const int end = whole ? piece + 1 : wide_cut(total, W, piece + 1);

    while (pos < end) {
        // the group that `pos` - a piece of the parts, or a share of the total cost - lies in, and where it begins
        int g = -1, base = 0;
        for (int g0 = 0; g0 < ng; g0 += kWave) {
            const Share sh = share_of(g0);
            const int w = sh.parts * (whole ? (sh.part_weight + most - 1) / most : sh.part_weight);
            const int inc = wave_inclusive_scan(w);
            const unsigned long long past = __ballot(base + inc > pos);
            if (past) {
                const int l = __ffsll((long long)past) - 1;
                g = g0 + l;
                base += __builtin_amdgcn_readlane(inc - w, l);
                break;
            }
            base += __builtin_amdgcn_readlane(inc, kWave - 1);
        }
        if (g < 0) break;  // fewer pieces than workgroups
        g = __builtin_amdgcn_readfirstlane(g);
        const WideGroup grp = wide_group_less_share(groups, g);
        const int wgt = weight(grp.n), part_weight = wgt * blocks;
        const int in_part = whole ? (part_weight + most - 1) / most : part_weight;
        const int part = __builtin_amdgcn_readfirstlane((pos - base) / in_part);
        const int at = base + part * in_part;
        int b0, len;
        if (whole) {
            b0 = blocks * (pos - at) / in_part;
            len = blocks * (pos - at + 1) / in_part - b0;
        } else {  // block k of a part belongs to the piece that holds the start of its share, k * wgt behind the part's
            b0 = (pos - at + wgt - 1) / wgt;
            len = min(blocks, max(end - at + wgt - 1, 0) / wgt) - b0;
        }
        b0 = __builtin_amdgcn_readfirstlane(b0);
        len = __builtin_amdgcn_readfirstlane(len);
        pos = whole ? end : at + part_weight;  // the next part, or past the end
        const int tile0 = part * part_tiles(grp.n), tok_first = 16 * tile0;
        const int n_tok = min(16 * part_tiles(grp.n), grp.n - tok_first);
        if (len <= 0 || n_tok <= 0) continue;
        const int tiles = wide_tiles(n_tok);
        const unsigned char* codes = scalar_ptr(grp.e.codes);
        const unsigned char* scale = scalar_ptr(grp.e.scale);
        const unsigned char* zero = scalar_ptr(grp.e.zero);
        const unsigned char* xsrc = scalar_ptr(frag + (size_t)(grp.tile + tile0) * units * 128);
        const unsigned char* ssrc = scalar_ptr(gsum + (size_t)(grp.tile + tile0) * units * (16 * kGroups));
        __syncthreads();  // the previous part's arrays are no longer read
        if (tid < kTok) {
            const int row = tok_first + (tid < n_tok ? tid : 0);  // dead token rows repeat the first one
            s_tau[tid] = tau[grp.first + row];
            s_back[tid] = back[grp.tile * 16 + row];
        }
        const int np = (len + kUpWaves - 1) / kUpWaves;
        const int per = (len + np - 1) / np;

        int selected = 0;  // channels of this part's first 16 tokens that this wave found above their thresholds
        // live: token tiles that this part has, of NT at most
        auto run = [&](auto live) __attribute__((always_inline)) {
            constexpr int NL = decltype(live)::value;
            constexpr int kPieces = kUpSlotUnits * 2 * NL, kSumPieces = (kUpSlotUnits * kGroups * NL * 4 + 63) / 64;
            constexpr int kReq = (kPieces + kSumPieces + kUpWaves - 1) / kUpWaves;  // a wave's share of a slot
            constexpr int kRegLoads = CT * kVec + kMetaLoads;
            // where a lane's four sums are: [unit][group][tile][token quarter] in LDS, [tile][unit][group][16] in memory
            auto sum_at = [&](int i) {
                i = min(i, kUpSlotUnits * kGroups * NL * 4 - 1);
                return (uint32_t)(min(i / 4 % NL, tiles - 1) * units * kGroups + i / (4 * NL)) * 64u + 16u * (uint32_t)(i & 3);
            };
            const uint32_t sum_off = sum_at(lane), sum_off2 = sum_at(64 + lane);
            const int slots = units / kUpSlotUnits;  // a multiple of four (d % 512 == 0)
            // slot s (past the last one: the last one again)
            auto load_x = [&](uint4* x, int s) __attribute__((always_inline)) {
                const int u0 = min(s, slots - 1) * kUpSlotUnits;
#pragma unroll
                for (int k = 0; k < kReq; ++k) {
                    const int it = min(wave + kUpWaves * k, kPieces + kSumPieces - 1);
                    // piece it: 1 KB of (unit, tile, instruction of the unit), or behind them four sums per lane
                    const int u = it / (2 * NL), n = it / 2 % NL, j = it & 1;
                    const uint32_t xo = (uint32_t)((min(n, tiles - 1) * units + u0 + u) * 2 + j) * 1024u;
                    if constexpr (kSumPieces == 1) {
                        const bool sums = it == kPieces;
                        dma16((sums ? ssrc + (uint32_t)u0 * (64u * kGroups) : xsrc + xo) + (sums ? sum_off : 16u * lane), x + (sums ? kXVecs : it * 64));
                    } else {
                        const bool sums = it >= kPieces;
                        dma16((sums ? ssrc + (uint32_t)u0 * (64u * kGroups) : xsrc + xo) + (sums ? (it == kPieces ? sum_off : sum_off2) : 16u * lane),
                              x + (sums ? kXVecs + (it - kPieces) * 64 : it * 64));
                    }
                }
            };
            for (int p0 = 0; p0 < len; p0 += per) {
                const bool active = wave < per && p0 + wave < len;
                const int ch0 = (b0 + p0 + wave) * kCh;
                __syncthreads();  // the slots are no longer read
                if (!active) {  // the same barriers as the waves below
                    load_x(x0, 0);
                    load_x(x1, 1);
                    load_x(x2, 2);
                    auto step = [&](uint4* next, int s) __attribute__((always_inline)) {
                        wait_requests_all_but<2 * kReq>();
                        meet();
                        load_x(next, s + 3);
                    };
#pragma unroll 1
                    for (int s = 0; s < slots; s += 4) {
                        step(x3, s);
                        step(x0, s + 1);
                        step(x1, s + 2);
                        step(x2, s + 3);
                    }
                    continue;
                }
                // codes: quarter g of a channel's four lanes brings in units 2 g and 2 g + 1 of eight, and one vector of its scales and
                // zeros (clamped lanes never store)
                uint4 cq[CT][kVec], mq[kMetaLoads];
                auto row_of = [&](int t) { return (uint32_t)min(ch0 + 16 * t + c, f - 1) * (uint32_t)units; };
                auto load_codes = [&](int s) __attribute__((always_inline)) {  // of the eight units from slot s on
                    const uint32_t u0 = (uint32_t)min(s, slots - 4) * kUpSlotUnits;
#pragma unroll
                    for (int k = 0; k < kMetaLoads; ++k) {
                        // vector 4 k + g of [tile][scales, zeros][kGroups]
                        const int vec = min(4 * k + g4, CT * 2 * kGroups - 1), part_ = vec % kGroups;
                        mq[k] = gload16((vec / kGroups & 1 ? zero : scale) + ((row_of(vec / (2 * kGroups)) + u0) * (2u * kGroups) + 16 * part_));
                    }
#pragma unroll
                    for (int t = 0; t < CT; ++t)
#pragma unroll
                        for (int k = 0; k < kVec; ++k) cq[t][k] = gload16(codes + ((row_of(t) + u0 + 2 * g4) * (uint32_t)(BITS * 8) + 16 * k));
                };
                load_x(x0, 0);
                __builtin_amdgcn_sched_barrier(0);
                load_codes(0);
                __builtin_amdgcn_sched_barrier(0);
                load_x(x1, 1);
                load_x(x2, 2);
                f32x4 acc[CT][NL];
#pragma unroll
                for (int t = 0; t < CT; ++t)
#pragma unroll
                    for (int n = 0; n < NL; ++n) acc[t][n] = f32x4{0.f, 0.f, 0.f, 0.f};
                // The codes of the coming four slots are here, the two slots requested behind them may still be under way.  (Said by
                // hand, here and at the end of the loop: with requests to LDS among them the compiler waits for all of them.  No call
                // got faster by it, the slots are long enough: 512 tokens on 8 experts 737 us either way.)
                wait_requests_all_but<2 * kReq>();
#pragma unroll 1
                for (int s = 0; s < slots; s += 4) {
                    uint32_t wd[CT][2][4][kLaneWords];
#pragma unroll
                    for (int t = 0; t < CT; ++t)
#pragma unroll
                        for (int p = 0; p < 2; ++p) deal_units<BITS>(cq[t], p, wd[t][p]);
                    uint4 mc[kMetaLoads];
#pragma unroll
                    for (int k = 0; k < kMetaLoads; ++k) {
                        mc[k] = mq[k];
                        asm volatile("" : "+v"(mc[k].x), "+v"(mc[k].y), "+v"(mc[k].z), "+v"(mc[k].w));  // a copy: mq is loaded again below
                    }
                    auto step = [&](auto slot, const uint4* x, uint4* next) __attribute__((always_inline)) {
                        constexpr int k = decltype(slot)::value;
                        // slot k is here: younger are the requests of two slots and, for the last one, those of the codes
                        wait_requests_all_but<2 * kReq + (k == 3 ? kRegLoads : 0)>();
                        meet();
                        if constexpr (k == 2) load_codes(s + 4);  // (not sooner: half of the operand words make room for them)
                        __builtin_amdgcn_sched_barrier(0);
                        load_x(next, s + k + 3);
                        __builtin_amdgcn_sched_barrier(0);
                        // scales and zeros of the slot's units, to all quarters: word k (groups of 64), or words 2 (k & 1) + u of vector k / 2
                        uint32_t sz[kMetaLoads * 4][kGroups];
#pragma unroll
                        for (int m = 0; m < kMetaLoads; ++m) {
                            const uint32_t w[4] = {mc[m].x, mc[m].y, mc[m].z, mc[m].w};
#pragma unroll
                            for (int h = 0; h < kGroups; ++h) {
                                const uint32_t word = kGroups == 1 ? w[k] : w[2 * (k & 1) + h];
                                quarters_to_all(word, sz[4 * m][h], sz[4 * m + 1][h], sz[4 * m + 2][h], sz[4 * m + 3][h]);
                            }
                        }
                        // Step i of the slot is token tile i % NL of unit i / NL.  Three of them are under way: the operands of a
                        // later one come from LDS, the products of one are formed, the scales of the one before are applied, product by
                        // product (a product takes the matrix unit as long as four of the multiply-adds take the vector unit).
                        constexpr int kItems = kUpSlotUnits * NL, kAhead = 2;
                        const f32x4* sums = reinterpret_cast<const f32x4*>(x + kXVecs);
                        uint4 xf[kAhead + 1][2];
                        f32x4 sg[kAhead + 1][kGroups];
                        auto fetch = [&](int i) __attribute__((always_inline)) {
                            const int u = i / NL, n = i % NL;
#pragma unroll
                            for (int j = 0; j < 2; ++j) xf[i % (kAhead + 1)][j] = x[(i * 2 + j) * 64 + lane];
#pragma unroll
                            for (int h = 0; h < kGroups; ++h) sg[i % (kAhead + 1)][h] = sums[((u * kGroups + h) * NL + n) * 4 + g4];
                        };
                        float sc[2][CT][kGroups], zr[2][CT][kGroups];  // of the unit of the products, and of the one before
                        uint32_t r0[CT][4], r1[CT][4];
                        auto unpack = [&](int u) __attribute__((always_inline)) {
#pragma unroll
                            for (int t = 0; t < CT; ++t) {
#pragma unroll
                                for (int h = 0; h < kGroups; ++h) {
                                    // groups of 64: vectors [tile][scale, zero], half u of the word; groups of 32: vectors
                                    // [tile][scale, zero][k / 2], word u, half h
                                    const int vs = kGroups == 1 ? 2 * t : 4 * t + k / 2, vz = vs + kGroups;
                                    const h16x2 s2 = as_h2(sz[vs][kGroups == 1 ? 0 : u]), z2 = as_h2(sz[vz][kGroups == 1 ? 0 : u]);
                                    const bool hi = kGroups == 1 ? u : h;
                                    sc[u][t][h] = (float)(hi ? s2.y : s2.x);
                                    zr[u][t][h] = (float)(hi ? z2.y : z2.x);
                                    asm volatile("" : "+v"(sc[u][t][h]), "+v"(zr[u][t][h]));  // widened once; as halves they make mixed FMAs, at half the rate
                                }
                                weight_frag24<BITS, G32>(wd[t][u][k], 0, r0[t]);
                                weight_frag24<BITS, G32>(wd[t][u][k], 1, r1[t]);
                            }
                        };
                        f32x4 cc[2][CT][kGroups];  // products of this item and of the one before
                        // quarter q of the multiply-adds of item i
                        auto apply = [&](int i, int q) __attribute__((always_inline)) {
                            const int u = i / NL, n = i % NL, t = q >> 1;
                            f32x4& ac = acc[t][n];
#pragma unroll
                            for (int e = 2 * (q & 1); e < 2 * (q & 1) + 2; ++e) {
                                float v0 = ac[e];
#pragma unroll
                                for (int h = 0; h < kGroups; ++h)
                                    v0 = fmaf(sc[u][t][h], fmaf(-zr[u][t][h], sg[i % (kAhead + 1)][h][e], cc[i & 1][t][h][e]), v0);
                                asm volatile("" : "+v"(v0));  // here, not later: the products of a whole slot would wait in registers
                                ac[e] = v0;
                            }
                        };
                        auto product = [&](int i, int q) __attribute__((always_inline)) {  // q: first then second instruction of both tiles
                            const int t = q & 1, j = q >> 1;
                            const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
                            const h16x8 xa = __builtin_bit_cast(h16x8, xf[i % (kAhead + 1)][j]);
                            const h16x8 w = j ? as_h8(r1[t]) : as_h8(r0[t]);
                            f32x4& c0 = cc[i & 1][t][G32 ? j : 0];
                            c0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(xa, w, G32 || j == 0 ? zero4 : c0, 0, 0, 0);
                        };
#pragma unroll
                        for (int i = 0; i < kAhead; ++i) fetch(i);
                        unpack(0);
#pragma unroll
                        for (int i = 0; i < kItems + 1; ++i) {
                            if (i == NL) {
                                unpack(1);
                                __builtin_amdgcn_sched_barrier(0);
                            }
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                if (i < kItems) product(i, q);
                                if (i > 0) apply(i - 1, q);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                            if (i + kAhead < kItems) fetch(i + kAhead);
                        }
                    };
                    step(std::integral_constant<int, 0>{}, x0, x3);
                    step(std::integral_constant<int, 1>{}, x1, x0);
                    step(std::integral_constant<int, 2>{}, x2, x1);
                    step(std::integral_constant<int, 3>{}, x3, x2);
                    wait_requests_all_but<2 * kReq>();
                }
                // lane (c, g4) holds channel ch0 + 16 t + c for tokens 16 n + 4 g4 + i
                int tok0 = 4 * g4;
                asm volatile("" : "+v"(tok0));  // or the addresses below are formed ahead of the loop and held across it
#pragma unroll
                for (int n = 0; n < NL; ++n) {
                    const float4 tau4 = *reinterpret_cast<const float4*>(&s_tau[16 * n + tok0]);
                    const float4 back4 = *reinterpret_cast<const float4*>(&s_back[16 * n + tok0]);
                    const int pos0 = grp.first + tok_first + 16 * n + tok0;
                    const float limit[4] = {tau4.x, tau4.y, tau4.z, tau4.w}, bk[4] = {back4.x, back4.y, back4.z, back4.w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const bool used = 16 * n + tok0 + i < n_tok;
                        float* vt = v + (size_t)(pos0 + i) * f;
#pragma unroll
                        for (int t2 = 0; t2 < CT / 2; ++t2) {
                            uint32_t w = 0u;
#pragma unroll
                            for (int h = 0; h < 2; ++h) {
                                const int t = 2 * t2 + h, ch = ch0 + 16 * t + c;
                                const float val = acc[t][n][i] * bk[i];
                                if (used && ch < f) vt[ch] = val;
                                const uint64_t m = __ballot(used && ch < f && fabsf(val) > limit[i]);
                                if (n == 0) selected += __builtin_amdgcn_readfirstlane(__popcll(m));
                                w |= ((uint32_t)(m >> (16 * g4)) & 0xFFFFu) << (16 * h);
                            }
                            const int word = ch0 / 32 + t2;
                            if (mask_words && used && c == 0 && word < nwords) mask_words[(size_t)(pos0 + i) * nwords + word] = w;
                        }
                    }
                }
            }
        };
        with_live_tiles<NT>(tiles, run);
        // a group's share from the workgroup that has its first channels (from all of them it would be 256 additions to one place)
        if (part == 0 && b0 == 0 && lane == 0 && selected)
            atomicAdd(shares + g * kWideGroupWords, wide_selected_share(selected, min(len * 16 * CT, f) * min(n_tok, 16)));
    }
}

template <int BITS, bool G32, int NT>
static hipError_t launch_nt(const UpWideArgs& a, hipStream_t stream) {
    const long long blocks = (long long)a.est_groups * ((a.f + 31) / 32);
    int wgs = (int)(blocks < num_cus() ? blocks : num_cus());
    if (wgs > 8) wgs &= ~7;  // (see wide_piece)
    XOperand x;
    const hipError_t rc = launch_x_operand(a, BITS, G32 ? 32 : 64, x, stream);
    if (rc != hipSuccess) return rc;
    up_wide_kernel<BITS, G32, NT><<<dim3(wgs), dim3(kUpThreads), 0, stream>>>(a.groups, &a.groups->share, a.n_groups, a.max_groups, x.frag, x.gsum,
                                                                               x.back, a.v, a.prep.tau, a.mask_words, a.d, a.f);
    return hipGetLastError();
}
template <int BITS, bool G32>
static hipError_t launch_bits(const UpWideArgs& a, hipStream_t stream) {
    switch (a.nt) {
        case 1:
        case 2: return launch_nt<BITS, G32, 2>(a, stream);
        case 3: return launch_nt<BITS, G32, 3>(a, stream);
        case 4: return launch_nt<BITS, G32, 4>(a, stream);
        case 5: return launch_nt<BITS, G32, 5>(a, stream);
        case 10:  // nine tiles fit the ring, and the registers of INT2
            if constexpr (BITS == 2) return launch_nt<BITS, G32, 9>(a, stream);
            else return launch_nt<BITS, G32, 5>(a, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_up_wide(const UpWideArgs& a, int bits, int group, hipStream_t stream) {
    if (!up_wide_shape(a.d, a.f, bits, group)) return hipErrorInvalidValue;
    const bool g32 = group == 32;
    if (bits == 2) return launch_bits<2, false>(a, stream);
    if (bits == 3) return g32 ? launch_bits<3, true>(a, stream) : launch_bits<3, false>(a, stream);
    return g32 ? launch_bits<4, true>(a, stream) : launch_bits<4, false>(a, stream);
}

}  // namespace floe
