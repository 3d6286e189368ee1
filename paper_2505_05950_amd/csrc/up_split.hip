// S2 for token groups of up to 32 tokens, larger ones in parts of 32: V = X . W_up^Q on the matrix cores with the columns split over the waves of a
// workgroup (Alg. 1 line 2; the paper itself is batch-1, each token keeps its own threshold, mask and result).  The arithmetic
// is that of up_gemv_mfma.hip: codes masked in place as fp16 subnormals, activations scaled by powers of two, scale and zero
// applied per quantization group in fp32.
//
//   x_operand_kernel  per task, once: the activations in operand order, their group sums, the factor that undoes the scaling.
//   up_split_kernel   a wave owns 512 columns (eight units) of every channel its workgroup works on.  The activations that meet
//                     them are loaded once per group and stay in the wave's registers (64 per token tile; half of the second
//                     tile's lie in LDS), so that nothing but codes, scales and zeros moves in the loop over channel blocks; those
//                     of the next block are requested as the vectors of this one are used up, half a block at a time, and all of them are
//                     waited for at its top (the compiler copies them there).  The partial sums of the waves meet in LDS, two buffers in
//                     turn, one barrier per block.
//
// What bounds it: vector instructions (12 per unit and channel tile to mask codes and widen scale and zero, 8 per token tile to
// apply them), before them the cache's accesses: lanes that read 16 bytes each from rows of their own cost one access apiece whatever
// they use, so a lane brings in two whole units, and the quarters of a channel's lanes one vector of scales or zeros each, handed around by
// lane exchanges.  Measured, the kernels traced one by one, this one and x_operand in front of it (grouped or wide kernel, with what
// prepared its activations / the two, us): one expert d 4096 f 14336 INT2, 24 tokens 34 / 15.8 + 3.7 (256 workgroups of up_wide.hip had two
// of sixteen waves at work); 8 such experts, 64 tokens 72 / 61.6 + 6.0; 64 + 2 experts d 2048 f 1408 INT3 g32, 128 tokens 79 / 44.3 + 8.4.
// Tried: one token tile and half the registers, so that four waves share a SIMD (64 tokens 116 us: twice the accesses); the four reducing
// waves of a block in turn (the same).
//
// Division of work: the channel blocks of all groups form one sequence that is cut into pieces of equal cost, one workgroup each.
#include <atomic>
#include <type_traits>

#include "floe_dev.h"
#include "launch.h"
#include "mfma_codes.h"
#include "wide_layout.h"

namespace floe {

constexpr int kSpWaveUnits = 8;   // units of 64 columns that a wave owns
constexpr int kSpParked = 4 * 2 * 64;  // vectors per wave: the second token tile's activations of four units lie in LDS

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

// The activations of every task as the operand of the matrix instruction, [token tile][unit][instruction of the unit][lane],
// their sums per quantization group and the factor that undoes the scaling.  One task per workgroup, one unit per thread (d <= 8192).  (Every
// workgroup of the kernel below would otherwise gather them for itself, 16 bytes per lane from as many rows: 11 of its first 15 us.)
// In front of that the grouping, where nobody has done it: every workgroup counts the tasks of each expert for itself (a few hundred
// numbers; a kernel of one workgroup in front took 5 to 10 us).
struct XOperandArgs {
    const h16* x;
    int32_t slots, d, max_groups, n_tasks, chunk, n_all;
    WideGroup* groups;
    int32_t* n_groups;
    int32_t* order;
    const int32_t* task_expert;
    const DevExpert* table;
    DevExpert e;
    uint4* frag;
    float* gsum;
    float* back;
    WidePrep prep;
};
enum class Grouping { kReady, kSingle, kHere };  // the tables are there; all tasks belong to one expert; from the tasks' experts
template <int BITS, bool G32, Grouping HOW>
__global__ __launch_bounds__(128) void x_operand_kernel(XOperandArgs a) {
    using Tr = MfmaTraits<BITS, G32>;
    constexpr int kGroups = G32 ? 2 : 1;
    constexpr float kScaleBack = (float)(1 << (24 - Tr::kPmax));
    __shared__ float wave_max[2];
    const int i = blockIdx.x, U = threadIdx.x, lane = U & 63, units = a.d >> 6;
    int task = i, pos = i, row = 0;  // row: of the token tiles
    const bool live = U < units;
    if constexpr (HOW == Grouping::kReady) task = a.order[i];
    uint4 q[8];
    const uint4* xr = reinterpret_cast<const uint4*>(a.x + (size_t)(task / a.slots) * a.d) + (live ? U : 0) * 8;
#pragma unroll
    for (int r = 0; r < 8; ++r) q[r] = xr[r];
    if constexpr (HOW == Grouping::kSingle) {
        const int len = wide_single_len(a.n_tasks, a.chunk), g = i / len;
        row = ((i + 15 * g - (i - g * len)) >> 4) * 16 + (i - g * len);
        if (U == 0) {
            a.order[i] = i;
            if (i < wide_single_groups(a.n_tasks, a.chunk)) a.groups[i] = wide_single_group(a.e, a.n_tasks, a.chunk, i);
            if (i == 0) a.n_groups[0] = wide_single_groups(a.n_tasks, a.chunk);
        }
    } else if constexpr (HOW == Grouping::kHere) {
        // workgroup i is task i; groups of equal size per expert, tasks of a group ascending.  (Every task has an expert of the table: the routers pick
        // among n_all whatever the logits are, and every task is in a group.)
        __shared__ int tasks_of[1024 + 64];
        __shared__ int sums_of[2][4];  // tasks before this one in its expert; tasks and groups of the experts before; groups
        const int e = a.task_expert[i], threads = blockDim.x;
        for (int k = U; k < a.n_all; k += threads) tasks_of[k] = 0;
        __syncthreads();
        int before = 0;
        for (int j0 = U; j0 < a.n_tasks; j0 += 8 * threads) {
            int ej[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) ej[k] = j0 + k * threads < a.n_tasks ? a.task_expert[j0 + k * threads] : -1;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                if (ej[k] >= 0) atomicAdd(&tasks_of[ej[k]], 1);  // (sums of integers: in any order)
                before += ej[k] == e && j0 + k * threads < i;
            }
        }
        __syncthreads();
        int tasks = 0, groups = 0, all = 0;
        const float per_chunk = 1.0f / (float)a.chunk;
        for (int k = U; k < a.n_all; k += threads) {
            const int n = tasks_of[k], ng = small_quotient(n + a.chunk - 1, per_chunk);
            tasks += k < e ? n : 0;
            groups += k < e ? ng : 0;
            all += ng;
        }
        int sum[4] = {wave_sum(before), wave_sum(tasks), wave_sum(groups), wave_sum(all)};
        if (threads > kWave) {
            if (lane == 0) {
#pragma unroll
                for (int k = 0; k < 4; ++k) sums_of[U >> 6][k] = sum[k];
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < 4; ++k) sum[k] = sums_of[0][k] + sums_of[1][k];
        }
        const int n = tasks_of[e], ng = small_quotient(n + a.chunk - 1, per_chunk), len = small_quotient(n + ng - 1, 1.0f / (float)ng);
        const int gl = small_quotient(sum[0], 1.0f / (float)len), g = sum[2] + gl, first = sum[1] + gl * len, tile = (first + 15 * g) >> 4;
        pos = sum[1] + sum[0];
        row = tile * 16 + sum[0] - gl * len;
        if (U == 0) {
            a.order[pos] = i;
            if (sum[0] == gl * len) a.groups[g] = WideGroup{0, min(len, n - gl * len), first, tile, a.table[e]};
            if (i == 0) a.n_groups[0] = sum[3];
        }
    } else {
        int g;
        row = wide_token_row(a.groups, a.n_groups[0], a.max_groups, i, lane, g);
    }
    const int d = a.d;
    uint4* __restrict__ frag = a.frag;
    float* __restrict__ gsum = a.gsum;
    if (U == 0) wide_clear(a.prep, pos, task, a.n_tasks);
    u16x2 top2 = {0, 0};
    uint32_t xv[32];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        xv[4 * r] = q[r].x; xv[4 * r + 1] = q[r].y; xv[4 * r + 2] = q[r].z; xv[4 * r + 3] = q[r].w;
    }
    // the largest magnitude, as the bits of a half (those of non-negative numbers order like integers; a NaN lands on top)
#pragma unroll
    for (int k = 0; k < 32; ++k) top2 = __builtin_elementwise_max(top2, __builtin_bit_cast(u16x2, xv[k] & 0x7FFF7FFFu));
    float amax = wave_allreduce_max_nonneg((float)__builtin_bit_cast(h16, (uint16_t)max((uint32_t)top2.x, (uint32_t)top2.y)));
    if (blockDim.x > kWave) {  // (more than 64 units)
        if (lane == 0) wave_max[U >> 6] = amax;
        __syncthreads();
        amax = fmaxf(wave_max[0], wave_max[1]);
    }
    const int down = (amax >= 512.0f && amax < 3.0e38f) ? ilogbf(amax) - 8 : 0;  // |x'| < 512: 2^(pmax - p) x' stays finite
    if (U == 0) a.back[row] = ldexpf(1.0f, down) * kScaleBack;
    if (!live) return;
    const h16 ps = (h16)ldexpf(1.0f, -down);
    const h16x2 ps2 = {ps, ps};
    const int tile = row >> 4, c = row & 15;
    uint4* xop = a.prep.xop + ((size_t)tile * (d / 32) + 2 * U) * 64 + c;
#pragma unroll
    for (int r = 0; r < 8; ++r) xop[(r >> 2) * 64 + (r & 3) * 16] = q[r];
    uint4* out = frag + ((size_t)tile * units + U) * 128 + c;
    float sum[2] = {0.0f, 0.0f};
#pragma unroll
    for (int k = 0; k < 32; ++k) sum[G32 ? (k >> 4) : 0] = __builtin_amdgcn_fdot2(as_h2(xv[k]), ps2, sum[G32 ? (k >> 4) : 0], false);
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
                w[pr] = as_u32(as_h2(l16 | h16b) * (mul * ps2));
            }
            out[j * 64 + g * 16] = make_uint4(w[0], w[1], w[2], w[3]);
        }
    // (times 2^(pmax - 24), which the matrix products carry and the zero-point term is subtracted under)
#pragma unroll
    for (int k = 0; k < kGroups; ++k) gsum[(((size_t)tile * units + U) * kGroups + k) * 16 + c] = sum[k] * (1.0f / kScaleBack);
}

template <int BITS, bool G32, int NT, int TILES>
__global__ __launch_bounds__(512) void up_split_kernel(const WideGroup* __restrict__ groups, int32_t* __restrict__ shares, const int32_t* __restrict__ n_groups,
                                                       int max_groups, const uint4* __restrict__ frag,
                                                       const float* __restrict__ gsum, const float* __restrict__ back,
                                                       float* __restrict__ v, const float* __restrict__ tau,
                                                       uint32_t* __restrict__ mask_words, int d, int f) {
    constexpr int kTok = 16 * NT;
    constexpr int kGroups = G32 ? 2 : 1;                 // quantization groups per unit
    constexpr int kVec = BITS;                           // 16-byte vectors of codes per lane and tile: two units
    constexpr int kMetaLoads = (TILES * 2 * kGroups + 3) / 4;
    constexpr int kLaneWords = BITS == 2 ? 1 : 2;        // operand words per unit
    constexpr int kCh = 16 * TILES;
    extern __shared__ __align__(16) unsigned char lds[];
    const int nw = blockDim.x >> 6;                      // d / 512
    float2* red = reinterpret_cast<float2*>(lds);        // [2][nw][TILES * NT * 2][64]
    uint4* park = reinterpret_cast<uint4*>(red + (size_t)2 * nw * (TILES * NT * 2 * 64));  // [nw][4][2][64] where NT == 2
    float* xg = reinterpret_cast<float*>(park + (NT == 2 ? nw * kSpParked : 0));  // [nw][NT][8 * kGroups][16]
    __shared__ __align__(8) float s_tau[kTok], s_back[kTok];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int c = lane & 15, g4 = lane >> 4;
    const int units = d >> 6;
    const int nwords = mask_words_per_task(f);
    const int blocks = (32 * nwords + kCh - 1) / kCh;    // whole mask words
    FLOE_TL(0);
    // Equal pieces by what a block costs with one and with two token tiles and by what the start of a part costs.  INT2 with two channel
    // tiles per block: vector instructions, 20 and 28 per unit and channel tile, and the rest alike: 3 to 4.  The wider codes have one channel
    // tile and more to unpack, 7 to 8 (us with 3 to 4 / 7 to 8, 8 experts d 4096 f 14336 INT4 g64, 150 tokens 544 / 534; g32 552 / 545; INT3 g64,
    // 6 experts, 130 tokens 425 / 420); INT3 with groups of 32 again 3 to 4 (64 + 2 experts d 2048 f 1408, 128 tokens 240 / 243).
    const int ng = n_groups[0];
    constexpr int kStart = 12;
    auto weight = [](int n) { return n > 16 ? 8 : (BITS == 2 || (BITS == 3 && G32) ? 6 : 7); };
    // a group of more than 32 tokens comes in parts of 32 and a last one of the rest: what the last one and a full one weigh
    auto parts_of = [](int n) { return (n + 31) >> 5; };
    const int full_weight = weight(32) * blocks + kStart;
    auto last_weight = [&](int n) { return weight(n - 32 * (parts_of(n) - 1)) * blocks + kStart; };
    const int n_head = groups[min(lane, max_groups - 1)].n;  // (the first 64 groups are asked for once, without waiting for their number)
    auto tokens_of = [&](int g0) { return g0 == 0 ? n_head : groups[min(g0 + lane, max_groups - 1)].n; };
    auto group_weight = [&](int g0) {  // of lane's group
        const int n = tokens_of(g0);
        return g0 + lane < ng ? (parts_of(n) - 1) * full_weight + last_weight(n) : 0;
    };
    int total = 0;
    for (int g0 = 0; g0 < ng; g0 += kWave) total += wave_sum(group_weight(g0));
    const int piece = wide_piece(gridDim.x);
    int pos = wide_cut(total, gridDim.x, piece);
    const int end = wide_cut(total, gridDim.x, piece + 1);
    uint16_t* mask16 = reinterpret_cast<uint16_t*>(mask_words);
    uint4* my_park = park + wave * kSpParked + lane;
    float* my_xg = xg + wave * (kSpWaveUnits * kGroups * kTok);

    while (pos < end) {
        int g = ng - 1, base = 0;  // the group that `pos` lies in and where it begins
        for (int g0 = 0; g0 < ng; g0 += kWave) {
            const int w = group_weight(g0);
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
        g = __builtin_amdgcn_readfirstlane(g);
        const WideGroup grp = wide_group_less_share(groups, g);
        const int part = __builtin_amdgcn_readfirstlane(min((pos - base) / full_weight, parts_of(grp.n) - 1));
        const int tok_first = 32 * part, n_tok = min(32, grp.n - tok_first);
        // block k of a part belongs to the piece that holds the start of its share, kStart + k * wgt behind the part's
        const int wgt = weight(n_tok), at = base + part * full_weight + kStart;
        const int b0 = __builtin_amdgcn_readfirstlane(max(pos - at + wgt - 1, 0) / wgt);
        const int len = __builtin_amdgcn_readfirstlane(min(blocks, max(end - at + wgt - 1, 0) / wgt)) - b0;
        pos = at + blocks * wgt;  // the next part, or past the end
        if (len <= 0) continue;
        const unsigned char* codes = scalar_ptr(grp.e.codes);
        const unsigned char* scale = scalar_ptr(grp.e.scale);
        const unsigned char* zero = scalar_ptr(grp.e.zero);

        // ---- requests: block i's codes, scales and zeros (past the end the last block again: unconditional, so that the
        // compiler can count what is in flight).  Quarter g of a channel's four lanes brings in units 2 g and 2 g + 1 of the
        // wave's eight, and one vector of its scales and zeros.
        uint4 cq[TILES][kVec], mq[kMetaLoads];
        auto row_of = [&](int i, int t) { return (uint32_t)min((b0 + min(i, len - 1)) * kCh + 16 * t + c, f - 1); };  // clamped lanes never store
        auto load_codes = [&](int i, int t, int k) {
            cq[t][k] = gload16(codes + (row_of(i, t) * (uint32_t)(units * BITS * 8) + (uint32_t)((wave * kSpWaveUnits + 2 * g4) * (BITS * 8) + 16 * k)));
        };
        auto load_meta = [&](int i) {
#pragma unroll
            for (int k = 0; k < kMetaLoads; ++k) {
                // vector 4 k + g of [tile][scales, zeros][kGroups]
                const int vec = min(4 * k + g4, TILES * 2 * kGroups - 1), t = vec / (2 * kGroups), part = vec % kGroups;
                const uint32_t o = (row_of(i, t) * (uint32_t)units + wave * kSpWaveUnits) * (2u * kGroups) + 16 * part;
                mq[k] = gload16((vec / kGroups & 1 ? zero : scale) + o);
            }
        };
        load_meta(0);
#pragma unroll
        for (int k = 0; k < kVec; ++k)
#pragma unroll
            for (int t = 0; t < TILES; ++t) load_codes(0, t, k);
        __builtin_amdgcn_sched_barrier(0);  // the waits of the loop count the requests in this order
        // ---- the activations of the wave's units: tile n, lane (c, g4)
        const int tile0 = grp.tile + 2 * part;
        uint4 xr[NT][kSpWaveUnits][2];
#pragma unroll
        for (int n = 0; n < NT; ++n) {
            // (a second tile that the group does not have repeats the first: tiles past the last one do not exist)
            const uint4* xt = frag + ((size_t)(tile0 + (16 * n < n_tok ? n : 0)) * units + wave * kSpWaveUnits) * 128 + lane;
#pragma unroll
            for (int u = 0; u < kSpWaveUnits; ++u)
#pragma unroll
                for (int j = 0; j < 2; ++j) xr[n][u][j] = xt[u * 128 + j * 64];
        }
        FLOE_TL(1);
        __syncthreads();  // the previous group's arrays are no longer read
        if (tid < kTok) {
            const int row = tid < n_tok ? tid : 0;  // dead token rows repeat the first one
            s_tau[tid] = tau[grp.first + tok_first + row];
            s_back[tid] = back[tile0 * 16 + row];
        }
#pragma unroll
        for (int n = 0; n < NT; ++n)  // the wave's group sums of a tile: 8 * kGroups * 16 numbers
#pragma unroll
            for (int k = 0; k < 2 * kGroups; ++k)
                my_xg[(n * 2 * kGroups + k) * 64 + lane] =
                    gsum[((size_t)(tile0 + (16 * n < n_tok ? n : 0)) * units + wave * kSpWaveUnits) * (16 * kGroups) + k * 64 + lane];
        if constexpr (NT == 2) {
#pragma unroll
            for (int u = 4; u < kSpWaveUnits; ++u)
#pragma unroll
                for (int j = 0; j < 2; ++j) my_park[(u - 4) * 128 + j * 64] = xr[1][u][j];
        }
        FLOE_TL(2);
        __syncthreads();  // the group sums and s_back are complete
        FLOE_TL(3);
        int selected = 0;  // channels of this part's tokens that this wave found above their thresholds
        // live: token tiles that hold tokens
        auto body = [&](auto live, int i) __attribute__((always_inline)) {
            constexpr int NL = decltype(live)::value;
            f32x4 acc[TILES][NL];
#pragma unroll
            for (int t = 0; t < TILES; ++t)
#pragma unroll
                for (int n = 0; n < NL; ++n) acc[t][n] = f32x4{0.f, 0.f, 0.f, 0.f};
            f32x4 sg[2][NL][kGroups];  // group sums of this unit and, on their way, of the next
            auto sums_at = [](int u) { return (u >> 1) & 1; };  // (units in the order 0 2 4 6 1 3 5 7)
            auto load_sums = [&](int u) __attribute__((always_inline)) {
#pragma unroll
                for (int n = 0; n < NL; ++n)
#pragma unroll
                    for (int k = 0; k < kGroups; ++k)
                        sg[sums_at(u)][n][k] = *reinterpret_cast<const f32x4*>(&my_xg[((n * kSpWaveUnits + u) * kGroups + k) * 16 + 4 * g4]);
            };
            load_sums(0);
            // scales and zeros of the wave's eight units, to all four quarters of a channel
            uint32_t meta[kMetaLoads * 4][4];  // [vector][word]
#pragma unroll
            for (int k = 0; k < kMetaLoads; ++k) {
                const uint32_t w[4] = {mq[k].x, mq[k].y, mq[k].z, mq[k].w};
#pragma unroll
                for (int j = 0; j < 4; ++j) quarters_to_all(w[j], meta[4 * k][j], meta[4 * k + 1][j], meta[4 * k + 2][j], meta[4 * k + 3][j]);
            }
            load_meta(i + 1);
#pragma unroll
            for (int p = 0; p < 2; ++p) {  // units p, p + 2, p + 4, p + 6
                uint32_t wd[TILES][4][kLaneWords];
#pragma unroll
                for (int t = 0; t < TILES; ++t) deal_units<BITS>(cq[t], p, wd[t]);
                // vectors that are used up
#pragma unroll
                for (int k = 0; k < kVec; ++k)
                    if ((p == 0) == (k < BITS / 2)) {
#pragma unroll
                        for (int t = 0; t < TILES; ++t) load_codes(i + 1, t, k);
                    }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int us = 0; us < 4; ++us) {
                    const int u = 2 * us + p, un = us < 3 ? u + 2 : 1;
                    if (u != 7) load_sums(un);
                    uint4 xf[NL][2];
#pragma unroll
                    for (int n = 0; n < NL; ++n)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            xf[n][j] = n == 1 && u >= 4 ? my_park[(u - 4) * 128 + 64 * j]
                                                        : xr[n][u][j];
#pragma unroll
                    for (int t = 0; t < TILES; ++t) {
                        float sc[kGroups], zr[kGroups];
#pragma unroll
                        for (int k = 0; k < kGroups; ++k) {
                            const int m = u * kGroups + k, vec = t * 2 * kGroups + m / 8;  // (zeros: kGroups vectors on)
                            const h16x2 s2 = as_h2(meta[vec][(m & 7) >> 1]), z2 = as_h2(meta[vec + kGroups][(m & 7) >> 1]);
                            sc[k] = (float)((m & 1) ? s2.y : s2.x);
                            zr[k] = (float)((m & 1) ? z2.y : z2.x);
                            asm volatile("" : "+v"(sc[k]), "+v"(zr[k]));  // widened once; as halves they make mixed FMAs, at half the rate
                        }
                        uint32_t r0[4], r1[4];
                        weight_frag24<BITS, G32>(wd[t][us], 0, r0);
                        weight_frag24<BITS, G32>(wd[t][us], 1, r1);
#pragma unroll
                        for (int n = 0; n < NL; ++n) {
                            const h16x8 x0 = __builtin_bit_cast(h16x8, xf[n][0]), x1 = __builtin_bit_cast(h16x8, xf[n][1]);
                            const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
                            f32x4& ac = acc[t][n];
                            if constexpr (G32) {
                                const f32x4 c0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(x0, as_h8(r0), zero4, 0, 0, 0);
                                const f32x4 c1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(x1, as_h8(r1), zero4, 0, 0, 0);
#pragma unroll
                                for (int e = 0; e < 4; ++e) {
                                    const float t0 = fmaf(-zr[0], sg[sums_at(u)][n][0][e], c0[e]);
                                    const float t1 = fmaf(-zr[kGroups - 1], sg[sums_at(u)][n][kGroups - 1][e], c1[e]);
                                    ac[e] = fmaf(sc[kGroups - 1], t1, fmaf(sc[0], t0, ac[e]));
                                }
                            } else {
                                f32x4 cc = __builtin_amdgcn_mfma_f32_16x16x32_f16(x0, as_h8(r0), zero4, 0, 0, 0);
                                cc = __builtin_amdgcn_mfma_f32_16x16x32_f16(x1, as_h8(r1), cc, 0, 0, 0);
#pragma unroll
                                for (int e = 0; e < 4; ++e) ac[e] = fmaf(sc[0], fmaf(-zr[0], sg[sums_at(u)][n][0][e], cc[e]), ac[e]);
                            }
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);  // or the operands of later units pile up in registers
                }
            }
            // ---- the waves' shares meet: item (tile, token tile, half of the four tokens) of every lane
            float2* mine = red + ((size_t)(i & 1) * nw + wave) * (TILES * NL * 2 * 64);
#pragma unroll
            for (int t = 0; t < TILES; ++t)
#pragma unroll
                for (int n = 0; n < NL; ++n)
#pragma unroll
                    for (int h = 0; h < 2; ++h) mine[((t * NL + n) * 2 + h) * 64 + lane] = make_float2(acc[t][n][2 * h], acc[t][n][2 * h + 1]);
            __syncthreads();
            const float2* all = red + (size_t)(i & 1) * nw * (TILES * NL * 2 * 64);
            for (int it = wave; it < TILES * NL * 2; it += nw) {
                const int t = it / (NL * 2), n = (it >> 1) % NL, h = it & 1;
                const int tok0 = 16 * n + 4 * g4 + 2 * h;
                const float2 tau2 = *reinterpret_cast<const float2*>(&s_tau[tok0]), back2 = *reinterpret_cast<const float2*>(&s_back[tok0]);
                float2 r = make_float2(0.f, 0.f);
                for (int w0 = 0; w0 < nw; w0 += 4) {  // four reads under way at a time
                    float2 a[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) a[k] = all[((size_t)min(w0 + k, nw - 1) * (TILES * NL * 2) + it) * 64 + lane];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        r.x += w0 + k < nw ? a[k].x : 0.f;
                        r.y += w0 + k < nw ? a[k].y : 0.f;
                    }
                }
                const int base = (b0 + i) * kCh + 16 * t, ch = base + c;
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const bool live = tok0 + e < n_tok;
                    const int task = grp.first + tok_first + tok0 + e;
                    const float val = e ? r.y * back2.y : r.x * back2.x;
                    if (live && ch < f) v[(size_t)task * f + ch] = val;
                    const uint64_t m = __ballot(live && ch < f && fabsf(val) > (e ? tau2.y : tau2.x));
                    selected += __builtin_amdgcn_readfirstlane(__popcll(m));
                    if (mask16 && live && c == 0 && base < 32 * nwords)
                        mask16[(size_t)task * nwords * 2 + (base >> 4)] = (uint16_t)(m >> (16 * g4));
                }
            }
        };
        auto walk = [&](auto live) __attribute__((always_inline)) {
#pragma unroll 1
            for (int i = 0; i < len; ++i) {
                body(live, i);
                if (i == 0) FLOE_TL(4);
            }
        };
        if (NT > 1 && n_tok <= 16) walk(std::integral_constant<int, 1>{});
        else walk(std::integral_constant<int, NT>{});
        // a group's share from the workgroup that has its first channels (from all of them it would be 256 additions to one place)
        if (part == 0 && b0 == 0 && lane == 0 && selected)
            atomicAdd(shares + g * kWideGroupWords, wide_selected_share(selected, min(len * kCh, f) * n_tok));
    }
    FLOE_TL(5);
}

#ifdef FLOE_TIMELINE
extern "C" int floe_debug_set_timeline_up_split(unsigned long long* p) {
    return (int)hipMemcpyToSymbol(HIP_SYMBOL(g_timeline), &p, sizeof(p));
}
#endif

size_t x_operand_sum_bytes(int tiles, int d, int group) { return (size_t)tiles * 16 * ((size_t)(d / 64) * (group == 32 ? 2 : 1) * 4 + 4); }

template <int BITS, bool G32>
static hipError_t operand_bits(const UpWideArgs& a, const XOperand& x, hipStream_t stream) {
    const bool here = !a.single && a.task_expert && a.n_tasks <= kOperandGroups;
    const XOperandArgs p{a.x, a.slots, a.d, a.max_groups, a.n_tasks, a.chunk, a.n_all, a.groups,
                         const_cast<int32_t*>(a.n_groups), const_cast<int32_t*>(a.order), a.task_expert, a.table,
                         a.single ? *a.single : DevExpert{}, x.frag, x.gsum, x.back, a.prep};
    const dim3 grid(a.n_tasks), block(a.d > 4096 ? 128 : 64);
    if (a.single) x_operand_kernel<BITS, G32, Grouping::kSingle><<<grid, block, 0, stream>>>(p);
    else if (here) x_operand_kernel<BITS, G32, Grouping::kHere><<<grid, block, 0, stream>>>(p);
    else x_operand_kernel<BITS, G32, Grouping::kReady><<<grid, block, 0, stream>>>(p);
    return hipGetLastError();
}
hipError_t launch_x_operand(const UpWideArgs& a, int bits, int group, XOperand& x, hipStream_t stream) {
    const size_t tiles = (size_t)(a.n_tasks + 15 * a.max_groups) / 16;  // that the groups can have together
    x.frag = static_cast<uint4*>(a.x_frag);
    x.gsum = static_cast<float*>(a.x_sums);
    x.back = x.gsum + tiles * (a.d / 64) * (group == 32 ? 32 : 16);
    if (bits == 2) return operand_bits<2, false>(a, x, stream);
    if (bits == 3) return group == 32 ? operand_bits<3, true>(a, x, stream) : operand_bits<3, false>(a, x, stream);
    return group == 32 ? operand_bits<4, true>(a, x, stream) : operand_bits<4, false>(a, x, stream);
}

template <int BITS, bool G32, int NT>
static hipError_t launch_split(const UpWideArgs& a, hipStream_t stream) {
    // channel tiles per block: what the registers take beside the activations (64 per token tile)
    constexpr int TILES = (BITS == 2 ? 4 : 2) / NT;
    constexpr int kGroups = G32 ? 2 : 1;
    const int nw = a.d / 512;
    const size_t lds = (size_t)2 * nw * (TILES * NT * 2 * 64) * sizeof(float2) + (NT == 2 ? nw * kSpParked * sizeof(uint4) : 0) +
                       (size_t)nw * kSpWaveUnits * kGroups * 16 * NT * sizeof(float);
    // the attribute belongs to the function on one device: set once per device, from whichever thread comes first
    constexpr int kMaxDevices = 64;
    static std::atomic<bool> attr_set[kMaxDevices];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    const auto kernel = &up_split_kernel<BITS, G32, NT, TILES>;
    if (!attr_set[dev].load(std::memory_order_acquire)) {
        const hipError_t rc = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 152 * 1024);
        if (rc != hipSuccess) return rc;
        attr_set[dev].store(true, std::memory_order_release);
    }
    const long long blocks = (long long)a.est_groups * ((a.nt + 1) / 2) * ((32 * mask_words_per_task(a.f) + 16 * TILES - 1) / (16 * TILES));
    const int room = num_cus() * (8 / nw > 1 ? 8 / nw : 1);  // workgroups that the registers hold at a time (eight waves per compute unit)
    int wgs = (int)(blocks < room ? blocks : room);
    if (wgs > 8) wgs &= ~7;  // (see wide_piece)
    XOperand x;
    const hipError_t rc = launch_x_operand(a, BITS, G32 ? 32 : 64, x, stream);
    if (rc != hipSuccess) return rc;
    kernel<<<dim3(wgs), dim3(64 * nw), lds, stream>>>(a.groups, &a.groups->share, a.n_groups, a.max_groups, x.frag, x.gsum, x.back, a.v, a.prep.tau,
                                                    a.mask_words, a.d, a.f);
    return hipGetLastError();
}

hipError_t launch_up_split(const UpWideArgs& a, int bits, int group, hipStream_t stream) {
    if (!up_split_shape(a.d, a.f, bits, group)) return hipErrorInvalidValue;
    const bool g32 = group == 32, two = a.nt > 1;
    if (bits == 2) return two ? launch_split<2, false, 2>(a, stream) : launch_split<2, false, 1>(a, stream);
    if (bits == 3) {
        if (g32) return two ? launch_split<3, true, 2>(a, stream) : launch_split<3, true, 1>(a, stream);
        return two ? launch_split<3, false, 2>(a, stream) : launch_split<3, false, 1>(a, stream);
    }
    if (g32) return two ? launch_split<4, true, 2>(a, stream) : launch_split<4, true, 1>(a, stream);
    return two ? launch_split<4, false, 2>(a, stream) : launch_split<4, false, 1>(a, stream);
}

}  // namespace floe
