// S4 + S5 for batches in which an expert sees many tokens (Alg. 1 steps 4-5; the paper itself is batch-1, each token keeps
// its own threshold, mask and result).  The tokens of an expert form groups of up to 16 * NT (NT token tiles of the matrix
// instruction); every row that any token of a group selected is read once for the whole group.
//
//   wide_prepare_kernel  where x_operand_kernel (up_split.hip) has not run: the activations in the order of the gate kernel's operand, cleared
//                      counters.
//   gate_wide_kernel   A[row][token] = gate_row . x_token.  A wave takes a pair of 16-row tiles.  Rows and activations travel
//                      from memory straight into a ring of three or four slots in LDS, 64 columns of 256 rows and of the group's
//                      tokens each; one barrier per slot.  In front of that the segment's row list: the ascending union of the tokens' selected
//                      channels, from the mask bits (wide_layout.h).  h = SiLU(A) * v * weight where |v| > tau, else 0, leaves in fp32 in
//                      the lane order of the down kernel's operand, and the largest |h| of each task beside it.
//   down_wide_kernel   Y[token][col] += h[token][row] * down[row][col].  A workgroup owns 512 output columns and a range of
//                      row pairs; a lane fetches 8-byte pieces of eight rows per pair (four pairs in flight), a register
//                      transpose (v_perm_b32) makes the operand.  h passes through LDS as two fp16 numbers (hi + lo),
//                      scaled by a power of two of the token's own that brings its largest |h| to [2^14, 2^15): relative
//                      to that the split is good to 2^-23, whatever the size of h, and no token depends on another.
//   combine_wide       adds a task's partial results.
//
// Division of work.  Gate: the channels of all groups in equal pieces, by what a group's rows are expected to be from its tokens and the share
// of channels they selected (wide_weight).  Down: the row pairs of all
// groups form one sequence; the workgroups cut it into equal pieces, whatever the routing did to the group sizes, so the launch is one even
// round and no compute unit waits for a crowded expert.
// The share is what the up projection found in a group's first piece.  Without it (one channel in eight, whatever the layer's sparsity) groups of
// few tokens were given pieces too large at 60 %: layer calls, cut by counted rows in a launch of its own / by one in eight / by the share, us, 96 + 1
// experts top-4 d 2048 f 2048 INT2, 128 tokens 397 / 446 / 397, 16 experts top-2 d 4096 f 4000, 64 tokens 271 / 282 / 264, 128 experts top-8
// d 2048 f 768 INT4, 128 tokens 281 / 285 / 266.  Pieces that end where groups end, without the limit to how uneven they may be / with it: the
// last one with 384 tokens (134 groups, 256 workgroups) 378 / 355, 256 experts top-8 d 4096 f 1408, 150 tokens 962 / 926.
//
// The lists were a launch of their own between the up projection and the gate kernel, 6 to 8 us (17 at 512 tokens, the activations with
// it), so that the gate kernel could cut by rows.  Made in the gate kernel they cost its workgroups 4 us before their first row; together with
// pieces that end where groups do, layer calls: one expert with 24 tokens 96 -> 89 us, 64 tokens on 8 experts 372 -> 357, 64 + 2 experts of d 2048
// f 1408 with 128 tokens 235 -> 220 (the grouping of tasks, a launch of one workgroup, is in these as well: x_operand_kernel).
//
// What bounds it: the rows (a kernel that only reads them in these pieces runs at 5.9 TB/s whatever the pieces are) and what stands
// between: the start of the streams, once per pass of eight pairs, SiLU behind them, and in the down kernel twice the matrix products.
// Hence groups as large as the accumulators allow (a second group reads the rows again).  Rows that go to registers instead, 16 bytes per
// lane from sixteen rows, cost the cache 64 accesses per request; with the activations' it was busy for half of the cycles and the
// waves stood behind their own requests.  The same holds for v gathered by lane (a tenth of the kernel).  Requests cost the cache their 1 KB
// whether or not rows repeat: the rows of a segment dealt to all eight waves, few each, took 37 us for one expert with 24 tokens, not 27.  Measured, gate, 8 experts
// d 4096 f 14336 at 90 %: 512 tokens 280 -> 232 us, 64 tokens 152 -> 144, one expert with 24 tokens 28.4 -> 24.6; with the lists made here 240, 147 and
// 26.6.  Gate + down before groups of more than 16 tokens: 64 tokens 364 us, 512 tokens 2425.  Down, the same layer with 512 tokens 277 -> 254 us, 267
// since it walks segments (ten token tiles leave that six registers too few: they are spilled, four before): half of its cycles were matrix products, a
// fifth of these for token tiles that a group does not fill, and the waves stood for the LDS reads in front of each tile's.  (A body per
// number of live tiles, as in the gate kernel, spills: 284.  So does reading one tile ahead with an address register per entry of h, 309:
// a reload waits for every row in flight.)  Up to two tiles it is bound by the rows and did not change.

#include <type_traits>

#include "floe_dev.h"
#include "launch.h"
#include "wide_layout.h"

namespace floe {

typedef _Float16 h16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 h16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kWideWaves = 8;
constexpr int kWideThreads = kWideWaves * 64;
constexpr int kPairRows = 32;    // two tiles of 16 rows: one k-step of the down kernel's matrix instruction
constexpr int kSliceCols = 64;   // columns of rows and activations per ring slot of the gate kernel
constexpr int kSpan = 64;        // channels of v that a wave brings in for a pair of row tiles
constexpr int kDownCols = 512;   // output columns per workgroup of the down kernel (64 per wave)

// What x_operand_kernel and the wide up projections do beside their own work, behind an up projection of another kind: the activations in the
// order of the gate kernel's operand, cleared counters, and each group's share of selected channels.  A workgroup per position of the order.
__global__ __launch_bounds__(128) void wide_prepare_kernel(WidePrep prep, WideArgs a, const uint32_t* __restrict__ mask_words, int n_tasks, int d) {
    const int i = blockIdx.x, tid = threadIdx.x, nwords = mask_words_per_task(a.f);
    int g;
    const int task = a.order[i], row = wide_token_row(a.groups, a.n_groups[0], a.max_groups, i, tid & 63, g);
    // (a group's share from its first four tokens: additions of all of them to one place take longer than the rest, 400 tokens on 6 experts 6 -> 17 us)
    const int seen = min(a.groups[g].n, 4);
    if (i - a.groups[g].first < seen) {
        const uint32_t* mw = mask_words + (size_t)(a.by_task ? task : i) * nwords;
        int selected = 0;
        for (int w0 = tid; w0 < nwords; w0 += 8 * 128) {
            uint32_t m[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) m[k] = w0 + k * 128 < nwords ? mw[w0 + k * 128] : 0u;
#pragma unroll
            for (int k = 0; k < 8; ++k) selected += __popc(m[k]);
        }
        selected = wave_sum(selected);
        if ((tid & 63) == 0 && selected) atomicAdd(&a.groups[g].share, wide_selected_share(selected, seen * a.f));
    }
    if (tid == 0) wide_clear(prep, i, task, n_tasks);
    // vector p of the row is quarter p % 4 of k-step p / 4
    const uint4* x = reinterpret_cast<const uint4*>(a.x + (size_t)(task / a.slots) * d);
    uint4* out = prep.xop + (size_t)(row >> 4) * (d / 32) * 64 + (row & 15);
    for (int p = tid; p < d / 8; p += 128) out[(p >> 2) * 64 + (p & 3) * 16] = x[p];
}

// ---------------------------------------------------------------------------------------------------------------
// gate
// ---------------------------------------------------------------------------------------------------------------
// Rows and activations travel from memory straight into LDS (global_load_lds_dwordx4), in ring slots that are arrays of their own, so
// that the compiler can tell which requests a read has to wait for.  The waits that matter are placed by hand, in front of the barrier
// that makes a slot everybody's.
template <int NT>
__global__ __launch_bounds__(kWideThreads) void gate_wide_kernel(WideArgs a, const uint32_t* __restrict__ mask_words, int d) {
    constexpr int kTok = 16 * NT;
    constexpr int kSlots = NT <= 3 ? 4 : 3;                  // ring slots that fit 160 KB of LDS
    constexpr int kRowVecs = kWideWaves * 256, kXVecs = 2 * NT * 64;  // per slot: 32 rows x 128 bytes per wave; two k-steps of x
    __shared__ uint4 r0[kRowVecs], r1[kRowVecs], r2[kRowVecs], r3[kSlots > 3 ? kRowVecs : 1];
    __shared__ uint4 x0[kXVecs], x1[kXVecs], x2[kXVecs], x3[kSlots > 3 ? kXVecs : 1];
    __shared__ int s_row[kTok];  // of v and the mask words
    __shared__ float s_w[kTok], s_tau[kTok];
    __shared__ uint32_t s_hmax[kTok];  // bits of the largest finite |h| of this workgroup's rows (ordered like the numbers)
    __shared__ int s_count[kTok], s_wave[kWideWaves];
    constexpr bool kKept = NT <= 5;  // (ten token tiles have no registers to keep the groups' records and weights)
    constexpr int kHeld = 4;
    __shared__ uint8_t s_weight[kKept ? kHeld * kWave : 1];  // of the first groups
    constexpr bool kIds = NT <= 5;  // (there is room for the row ids of a pass)
    __shared__ __align__(16) int s_ids[kIds ? kWideWaves * kPairRows : 4];
    uint32_t* s_union = reinterpret_cast<uint32_t*>(r0);  // before the rows: mask words of the segment's union,
    int* s_before = reinterpret_cast<int*>(r1);           // selected channels before each
    int* s_list = reinterpret_cast<int*>(r2);             // and its first rows
    constexpr int kList = kRowVecs * 4;
    static_assert(kRowVecs * 4 > kWideMaxMaskWords, "a segment's mask words fit a slot");
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int l16 = lane & 15, q4 = lane >> 4;
    const int ng = a.n_groups[0];
    const int W = gridDim.x, piece = wide_piece(W);
    const int units = wide_piece_units(a.f);
    // The records of the first 64 groups, in the lane of their number, and the weights of the first 256 are asked for once, without waiting
    // for the number of groups (the search below asked for them in every round: 0.4 us each).
    const WideGroup head = a.groups[min(lane, a.max_groups - 1)];
    auto weight_at = [&](int g0) {  // of the group in this lane
        const WideGroup& rec = a.groups[min(g0 + lane, a.max_groups - 1)];
        return wide_weight(rec.n, rec.share);
    };
    const bool many = a.max_groups > kWave;
    int held[kHeld] = {};
    held[0] = weight_at(0);
    if (many) {
#pragma unroll
        for (int q = 1; q < kHeld; ++q) held[q] = weight_at(q * kWave);
    }
#pragma unroll
    for (int q = 0; q < kHeld; ++q) held[q] = q * kWave + lane < ng ? held[q] : 0;  // 0 behind the last group
    if (kKept && many) {  // (every wave writes the same, and reads what it wrote)
#pragma unroll
        for (int q = 1; q < kHeld; ++q) s_weight[q * kWave + lane] = (uint8_t)held[q];
    }
    int total = (held[0] + held[1] + held[2] + held[3]) * units;
    for (int g0 = kHeld * kWave; g0 < ng; g0 += kWave) total += g0 + lane < ng ? weight_at(g0) * units : 0;
    total = wave_sum(total);
    // Pieces end where groups end: a second segment costs its start and its end again, 10 us, and the launch waits for the few workgroups that
    // have one (64 tokens on 8 experts: the mean workgroup done at 139 us, the last at 163).  Each group is cut into as few equal pieces of
    // at most `most` as it takes, `most` the smallest that leaves no more than W pieces - if that is not too large (wide_most_limit).
    bool whole = ng <= min(W, kHeld * kWave);
    int most = max((total + W - 1) / W, 1);
    const int limit = wide_most_limit(most);
    while (whole) {
        const float per_most = 1.0f / (float)most;
        int sum = wide_share(held[0], units, most, per_most);
        if (many) {
#pragma unroll
            for (int q = 1; q < kHeld; ++q) sum += wide_share(held[q], units, most, per_most);
        }
        sum = wave_sum(sum);
        if (sum <= W) break;
        most = wide_next_most(most);
        whole = most <= limit;
    }
    const float per_most = 1.0f / (float)most;
    auto share_of = [&](int weight) { return whole ? wide_share(weight, units, most, per_most) : weight * units; };
    int pos = whole ? piece : wide_cut(total, W, piece);
    const int end = whole ? piece + 1 : wide_cut(total, W, piece + 1);
    const int ns = d / kSliceCols;  // a multiple of eight (d % 512 == 0)
    const int pmax = (a.f + kPairRows - 1) / kPairRows;
    const int nwords = mask_words_per_task(a.f);
    // where in its 128 bytes a row's piece lies in LDS: at piece ^ swizzle(row), so that the sixteen rows of a tile meet all banks
    auto swizzle = [](int row) { return (row & 7) ^ ((row >> 3) & 1); };

    while (pos < end) {  // one group's part of this workgroup's piece at a time
        int g = -1, base = 0, weight = 0;  // the group that `pos` lies in and where it begins
        WideGroup grp{};
        for (int g0 = 0; g0 < ng; g0 += kWave) {
            const WideGroup rec = kKept && g0 == 0 ? head : a.groups[min(g0 + lane, a.max_groups - 1)];
            int wgt;
            if (kKept && g0 == 0) wgt = held[0];
            else if (kKept && g0 < kHeld * kWave) wgt = s_weight[g0 + lane];
            else wgt = g0 + lane < ng ? wide_weight(rec.n, rec.share) : 0;
            const int w = share_of(wgt);
            const int inc = wave_inclusive_scan(w);
            const unsigned long long past = __ballot(base + inc > pos);
            if (past) {
                const int l = __ffsll((long long)past) - 1;
                g = g0 + l;
                base += __builtin_amdgcn_readlane(inc - w, l);
                weight = __builtin_amdgcn_readlane(wgt, l);
                grp = wide_record(rec, l);
                break;
            }
            base += __builtin_amdgcn_readlane(inc, kWave - 1);
        }
        if (g < 0) break;  // fewer pieces than workgroups
        WideUnits part;
        int first_piece;
        if (whole) {
            part = wide_units_of_share(units, share_of(weight), pos - base);
            first_piece = base;
            pos = end;
        } else {
            part = wide_units_of_span(units, weight, pos - base, end - base);
            first_piece = wide_owner(total, W, base);
            pos = base + units * weight;  // the next group, or past the end
        }
        const int u0 = __builtin_amdgcn_readfirstlane(part.begin), u1 = __builtin_amdgcn_readfirstlane(part.end);
        if (u1 <= u0) continue;
        const int slot = wide_slot(u0, piece, first_piece);
        int32_t* rows = a.rows + (wide_row_slot(g, first_piece, pmax) + slot) * kPairRows;
        const unsigned char* gd = scalar_ptr(grp.e.gd);
        // ---- the tokens' mask words, the first ones requested ahead of all else
        const int c0 = 8 * u0, c1 = min(8 * u1, a.f), w0 = c0 >> 5, nws = ((c1 + 31) >> 5) - w0;
        const float per_segment = 1.0f / (float)nws;
        const uint32_t first_mask = ~0u << (c0 & 31), last_mask = (c1 & 31) ? (1u << (c1 & 31)) - 1u : ~0u;
        uint32_t m[4];
        int tok[4], j[4];
        auto load_masks = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = min(i0 + k * kWideThreads, grp.n * nws - 1);
                tok[k] = small_quotient(i, per_segment);
                j[k] = i - tok[k] * nws;
                const int at = grp.first + tok[k];
                m[k] = gload4(mask_words + (size_t)(a.by_task ? a.order[at] : at) * nwords + w0 + j[k]);
            }
        };
        load_masks(tid);
        __syncthreads();  // the previous segment's arrays and slots are no longer read
        int my_task = 0;  // of token tid, into LDS further down (nobody waits for them yet)
        float my_w = 0.0f, my_tau = 0.0f;
        if (tid < kTok) {
            const int at = grp.first + (tid < grp.n ? tid : 0);  // dead token rows repeat the first one
            my_task = a.order[at];
            my_w = a.scale[at];
            my_tau = a.tau[at];
            s_hmax[tid] = 0u;
            s_count[tid] = 0;
        }
        // ---- the union of the tokens' selected channels in this segment, ascending
        for (int i = tid; i < nws; i += kWideThreads) s_union[i] = 0u;
        __syncthreads();
        for (int i0 = tid;;) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                if (i0 + k * kWideThreads >= grp.n * nws) continue;
                m[k] &= (j[k] == 0 ? first_mask : ~0u) & (j[k] == nws - 1 ? last_mask : ~0u);
                if (m[k]) {
                    atomicOr(&s_union[j[k]], m[k]);
                    atomicAdd(&s_count[tok[k]], __popc(m[k]));
                }
            }
            i0 += 4 * kWideThreads;
            if (i0 >= grp.n * nws) break;
            load_masks(i0);
        }
        __syncthreads();
        const int per_thread = (nws + kWideThreads - 1) / kWideThreads;
        int mine = 0;
        for (int k = 0; k < per_thread; ++k) mine += tid * per_thread + k < nws ? __popc(s_union[tid * per_thread + k]) : 0;
        const int inc = wave_inclusive_scan(mine);
        if (lane == kWave - 1) s_wave[wave] = inc;
        __syncthreads();
        int run = inc - mine, count = 0;
#pragma unroll
        for (int w = 0; w < kWideWaves; ++w) {
            run += w < wave ? s_wave[w] : 0;
            count += s_wave[w];
        }
        count = __builtin_amdgcn_readfirstlane(count);
        for (int k = 0; k < per_thread; ++k) {
            const int w = tid * per_thread + k;
            if (w < nws) {
                s_before[w] = run;
                run += __popc(s_union[w]);
            }
        }
        __syncthreads();
        const int npairs = (count + kPairRows - 1) / kPairRows;
        for (int i = tid; i < 32 * nws; i += kWideThreads) {
            const uint32_t m = s_union[i >> 5], bit = 1u << (i & 31);
            if (m & bit) {
                const int k = s_before[i >> 5] + __popc(m & (bit - 1u)), row = 32 * w0 + i;
                rows[k] = row;
                if (k < kList) s_list[k] = row;
                if (count > kList && k == count - 1)
                    for (int p = count; p < npairs * kPairRows; ++p) rows[p] = row;
            }
        }
        if (tid == 0) a.segments[piece + g] = make_int4(npairs, slot, g, u0 == 0);
        if (tid < kTok) {
            s_row[tid] = a.by_task ? my_task : grp.first + (tid < grp.n ? tid : 0);
            s_w[tid] = my_w;
            s_tau[tid] = my_tau;
            if (tid < grp.n && s_count[tid]) atomicAdd(&a.count[my_task], s_count[tid]);
        }
        // (the first pass takes its rows from LDS; when others read the list back, the first slice has been waited for by every wave, and with it
        // the stores before)
        wait_lds();
        meet();
        if (count <= kList && count + tid < npairs * kPairRows) rows[count + tid] = s_list[count - 1];
        if (count == 0) continue;
        const int tiles = wide_tiles(grp.n);
        const unsigned char* xop = scalar_ptr(a.xop + (size_t)grp.tile * (d / 32) * 64);
        // Workgroups start at different column slices: rows are 4 d bytes apart, so workgroups that walk the columns in step
        // ask for the same few memory channels at the same time.  (Two groups of one expert that work on the same rows
        // start alike and share them through the L2.)
        const int rot = (int)((unsigned)(u0 >> 5) * 10u % (unsigned)ns);
        auto col_slice = [&](int s) {  // s-th slice of this workgroup (past the last one: the last one again)
            const int c = min(s, ns - 1) + rot;
            return c < ns ? c : c - ns;
        };
        // equal passes of at most a pair per wave
        const int passes = (npairs + kWideWaves - 1) / kWideWaves, per_pass = (npairs + passes - 1) / passes * kPairRows;
        uint4* hseg = a.hbuf + wide_h_first(grp.tile, g, first_piece, pmax, NT) + (size_t)slot * tiles * 128;
        // live: token tiles that this group fills, of NT at most (a tile without tokens would cost as much as any other)
        auto segment = [&](auto live) __attribute__((always_inline)) {
            constexpr int NL = decltype(live)::value;
            constexpr int kXReq = (2 * NL + kWideWaves - 1) / kWideWaves;  // a wave's share of a slice's activations
            constexpr int kReq = 4 + kXReq;                                // ... and its rows
            for (int p0 = 0; p0 < count; p0 += per_pass) {
                const int first = p0 + wave * kPairRows;  // the wave's rows
                const bool active = first < min(count, p0 + per_pass);  // the others only help to bring x in
                auto load_x = [&](uint4* x, int s) {
#pragma unroll
                    for (int k = 0; k < kXReq; ++k) {
                        const int it = min(wave + kWideWaves * k, 2 * NL - 1), ks = it / NL, n = it % NL;
                        dma16(xop + ((uint32_t)(min(n, tiles - 1) * (d / 32) + 2 * col_slice(s) + ks) * 1024u + 16u * lane), x + it * 64);
                    }
                };
                uint32_t wo[4];  // byte offsets from gd of the rows' pieces this lane brings in: at most f * 4 d <= 2^31
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int r = 8 * j + (lane >> 3);
                    const int k = min(first + r, count - 1);  // rows past the end repeat the last one
                    const int id = p0 == 0 ? s_list[min(k, kList - 1)] : rows[k];  // (kWideWaves * kPairRows of them at most)
                    if (kIds && (lane & 7) == 0) s_ids[wave * kPairRows + r] = id;
                    wo[j] = (uint32_t)id * (uint32_t)(4 * d) + 16u * (uint32_t)((lane & 7) ^ swizzle(r));
                }
                // The v that meet these rows.  Gathered by the lane that needs them they are 64 accesses of 4 bytes to the cache per
                // instruction and a tenth of the kernel's time; where the wave's rows lie within kSpan channels (half of the channels
                // or more selected by somebody) the wave brings the whole span in instead, 16 bytes per lane, and picks from LDS.  Up to three
                // token tiles it does so ahead of the loop (behind it the round trip stood bare, 2 us).
                constexpr bool kEarlyV = NT <= 3;
                const int last_in = min(first + kPairRows, count) - first - 1;
                auto row_at = [&](int r) {  // (a scalar)
                    return __builtin_amdgcn_readfirstlane(kIds ? s_ids[wave * kPairRows + r] : rows[first + r]);
                };
                int row0 = 0;
                bool span = false;
                uint4 vq[kEarlyV ? NL : 2][4];
                auto load_v = [&](int n) __attribute__((always_inline)) {  // four tokens per request
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        vq[kEarlyV ? n : n & 1][k] = gload16u(a.v + (size_t)s_row[16 * n + 4 * k + q4] * a.f + row0 + 4 * l16);
                };
                if (kEarlyV && active) {
                    row0 = min(row_at(0), a.f - kSpan);
                    span = row0 >= 0 && row_at(last_in) - row0 < kSpan;
                    if (span) {
#pragma unroll
                        for (int n = 0; n < NL; ++n) load_v(n);
                    }
                }
                __syncthreads();  // the slots are no longer read
                if (!active) {  // the same barriers as the waves below
                    load_x(x0, 0);
                    load_x(x1, 1);
                    if constexpr (kSlots > 3) load_x(x2, 2);
                    auto step = [&](uint4* next, int s) __attribute__((always_inline)) {
                        wait_requests_all_but<(kSlots - 2) * kXReq>();
                        meet();
                        load_x(next, s + kSlots - 1);
                    };
                    int s = 0;
#pragma unroll 1
                    for (; s + kSlots <= ns; s += kSlots) {
                        step(kSlots > 3 ? x3 : x2, s);
                        step(x0, s + 1);
                        step(x1, s + 2);
                        if constexpr (kSlots > 3) step(x2, s + 3);
                    }
                    if constexpr (kSlots == 3) {
                        if (s < ns) step(x2, s);
                        if (s + 1 < ns) step(x0, s + 1);
                    }
                    continue;
                }
                auto load_rows = [&](uint4* r, int s) {
                    const uint32_t c = (uint32_t)col_slice(s) * (2u * kSliceCols);
#pragma unroll
                    for (int j = 0; j < 4; ++j) dma16(gd + (wo[j] + c), r + wave * 256 + j * 64);
                };
                f32x4 acc[2][NL];
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int n = 0; n < NL; ++n) acc[t][n] = f32x4{0.f, 0.f, 0.f, 0.f};
                auto step = [&](const uint4* r, const uint4* x, uint4* next_r, uint4* next_x, int s) __attribute__((always_inline)) {
                    wait_requests_all_but<(kSlots - 2) * kReq>();  // slice s is here, for this wave ...
                    meet();                                        // ... and for all; nobody reads the slot of slice s - 1 any more
                    load_rows(next_r, s + kSlots - 1);
                    load_x(next_x, s + kSlots - 1);
                    __builtin_amdgcn_sched_barrier(0);
                    uint4 w[2][2];
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                        for (int t = 0; t < 2; ++t) w[ks][t] = r[wave * 256 + (16 * t + l16) * 8 + ((4 * ks + q4) ^ swizzle(l16))];
                    // LDS reads a few ahead of the products that need them (left alone, the compiler lets each pair wait for its own)
                    constexpr int kAhead = 2 * NL < 6 ? 2 * NL : 6;
                    uint4 xf[kAhead];
#pragma unroll
                    for (int i = 0; i < kAhead; ++i) xf[i] = x[i * 64 + lane];
#pragma unroll
                    for (int i = 0; i < 2 * NL; ++i) {
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int t = 0; t < 2; ++t)
                            acc[t][i % NL] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h16x8, w[i / NL][t]),
                                                                                    __builtin_bit_cast(h16x8, xf[i % kAhead]), acc[t][i % NL], 0, 0, 0);
                        if (i + kAhead < 2 * NL) xf[i % kAhead] = x[(i + kAhead) * 64 + lane];
                    }
                };
                load_rows(r0, 0);
                load_x(x0, 0);
                load_rows(r1, 1);
                load_x(x1, 1);
                if constexpr (kSlots > 3) {
                    load_rows(r2, 2);
                    load_x(x2, 2);
                }
                int s = 0;
#pragma unroll 1
                for (; s + kSlots <= ns; s += kSlots) {
                    step(r0, x0, kSlots > 3 ? r3 : r2, kSlots > 3 ? x3 : x2, s);
                    step(r1, x1, r0, x0, s + 1);
                    step(r2, x2, r1, x1, s + 2);
                    if constexpr (kSlots > 3) step(r3, x3, r2, x2, s + 3);
                }
                if constexpr (kSlots == 3) {
                    if (s < ns) step(r0, x0, r2, x2, s);
                    if (s + 1 < ns) step(r1, x1, r0, x0, s + 1);
                }
                wait_requests_all_but<0>();  // (repeats of the last slice) the wave's rows make room for v
                // lane (l16, q4) holds A[row 16 t + 4 q4 + i][token 16 n + l16]
                int row[2][4];
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int r = 16 * t + 4 * q4 + i;
                        row[t][i] = first + r < count ? (kIds ? s_ids[wave * kPairRows + r] : rows[first + r]) : -1;
                    }
                int tok0 = l16;
                asm volatile("" : "+v"(tok0));  // or the addresses below are formed ahead of the loop and held across it
                if (!kEarlyV) {
                    row0 = min(row_at(0), a.f - kSpan);
                    span = row0 >= 0 && row_at(last_in) - row0 < kSpan;
                }
                float* stage = reinterpret_cast<float*>(r0 + wave * 256);  // [16 tokens][64 channels], pieces of 16 bytes at piece ^ token
                auto finish = [&](int n, const float (&vv)[2][4]) __attribute__((always_inline)) {
                    const float w = s_w[16 * n + tok0], tau = s_tau[16 * n + tok0];
                    const bool used = 16 * n + tok0 < grp.n;
                    uint32_t top = 0u;
#pragma unroll
                    for (int t = 0; t < 2; ++t)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const float v = vv[t][i];
                            const bool keep = used && row[t][i] >= 0 && fabsf(v) > tau;
                            const float h = keep ? silu(acc[t][n][i]) * v * w : 0.0f;
                            acc[t][n][i] = h;
                            const uint32_t m = __builtin_bit_cast(uint32_t, h) & 0x7FFFFFFFu;
                            top = max(top, m < 0x7F800000u ? m : 0u);
                        }
                    atomicMax(&s_hmax[16 * n + tok0], top);  // (no result wanted: fire and forget)
                };
                if (span) {
                    if (!kEarlyV) load_v(0);
#pragma unroll
                    for (int n = 0; n < NL; ++n) {
                        if (!kEarlyV && n + 1 < NL) load_v(n + 1);
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            // (stored as a native vector of what is read back: a wave's LDS accesses stay in order, and the compiler
                            // must not take the two for different objects)
                            *reinterpret_cast<f32x4*>(&stage[(4 * k + q4) * kSpan + 4 * (tok0 ^ (4 * k + q4))]) = __builtin_bit_cast(f32x4, vq[kEarlyV ? n : n & 1][k]);
                        }
                        __builtin_amdgcn_wave_barrier();
                        float vv[2][4];
#pragma unroll
                        for (int t = 0; t < 2; ++t)
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const int ch = max(row[t][i] - row0, 0);
                                vv[t][i] = stage[tok0 * kSpan + 4 * ((ch >> 2) ^ tok0) + (ch & 3)];
                            }
                        __builtin_amdgcn_wave_barrier();
                        finish(n, vv);
                    }
                } else {
                    constexpr int kBatch = NL < 4 ? NL : 4;  // token tiles whose v are requested together
#pragma unroll
                    for (int n0 = 0; n0 < NL; n0 += kBatch) {
                        float vv[kBatch][2][4];
#pragma unroll
                        for (int n = n0; n < n0 + kBatch && n < NL; ++n) {
                            const unsigned char* vt = reinterpret_cast<const unsigned char*>(a.v + (size_t)s_row[16 * n + tok0] * a.f);
#pragma unroll
                            for (int t = 0; t < 2; ++t)
#pragma unroll
                                for (int i = 0; i < 4; ++i) vv[n - n0][t][i] = gloadf(vt + 4 * max(row[t][i], 0));
                        }
#pragma unroll
                        for (int n = n0; n < n0 + kBatch && n < NL; ++n) finish(n, vv[n - n0]);
                    }
                }
                uint4* hb = hseg + (size_t)(first / kPairRows) * tiles * 128 + lane;
#pragma unroll
                for (int n = 0; n < NL; ++n)
                    if (n < tiles) {
#pragma unroll
                        for (int t = 0; t < 2; ++t) hb[n * 128 + t * 64] = __builtin_bit_cast(uint4, acc[t][n]);
                    }
            }
        };
        with_live_tiles<NT>(wide_tiles(grp.n), segment);
        __syncthreads();
        // a maximum does not depend on the order in which the workgroups of a group arrive
        if (tid < grp.n) atomicMax(&a.hmax[grp.first + tid], s_hmax[tid]);
    }
}

// ---------------------------------------------------------------------------------------------------------------
// down
// ---------------------------------------------------------------------------------------------------------------
// The h of SL pairs sits in LDS at a time; the rows of the next slice are in flight (four pairs, 16 KB per wave; two where
// the accumulators of ten token tiles need the registers).
template <int NT>
__global__ __launch_bounds__(kWideThreads) void down_wide_kernel(WideArgs a, int d) {
    constexpr int SL = NT <= 5 ? 4 : 2;
    constexpr int kTok = 16 * NT;
    constexpr int kRing = 4;                              // slices of row ids kept
    constexpr int kHRounds = SL * NT * 128 / kWideThreads;
    static_assert(SL * NT * 128 % kWideThreads == 0, "slice split");
    __shared__ uint4 hs[2][SL * NT * 128];  // [pair][token tile][hi, lo][lane]
    __shared__ float s_scale[kTok], s_back[kTok];  // the token's power of two and its reciprocal
    __shared__ __align__(16) int ids[kRing][SL * kPairRows];
    __shared__ int s_pair[kWideMaxSegments + 1];       // first pair of each segment in the sequence of all
    __shared__ uint32_t s_slot[kWideMaxSegments];      // its pair slot in the group; group in the upper half
    __shared__ uint16_t s_first[kWideMaxSegments];     // a group's first segment
    __shared__ int s_wave[kWideWaves], s_at;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int l16 = lane & 15, q4 = lane >> 4;
    const int ng = a.n_groups[0];
    const WideGroup head = a.groups[min(lane, a.max_groups - 1)];  // the first 64 groups' records, in the lane of their number
    const int nseg = min(a.pieces + ng, kWideMaxSegments);
    int total = 0;
    for (int i0 = 0; i0 < nseg; i0 += kWideThreads) {
        const int i = i0 + tid;
        const int4 seg = i < nseg ? a.segments[i] : make_int4(0, 0, 0, 0);
        const int inc = wave_inclusive_scan(seg.x);
        if (lane == kWave - 1) s_wave[wave] = inc;
        __syncthreads();
        int at = total + inc - seg.x;
#pragma unroll
        for (int w = 0; w < kWideWaves; ++w) {
            at += w < wave ? s_wave[w] : 0;
            total += s_wave[w];
        }
        if (i < nseg) {
            s_pair[i] = at;
            s_slot[i] = (uint32_t)seg.y | (uint32_t)seg.z << 16;
            if (seg.w) s_first[seg.z] = (uint16_t)i;
        }
        __syncthreads();
    }
    total = __builtin_amdgcn_readfirstlane(total);
    if (tid == 0) s_pair[nseg] = total;
    __syncthreads();
    auto segment_of = [&](int pair) {  // the last one that begins at or before it (those without rows begin where the next does)
        int lo = 0, hi = nseg;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (s_pair[mid] <= pair) lo = mid;
            else hi = mid;
        }
        return lo;
    };
    // no more pieces than the actual rows fill with four pairs each: every piece up to the last one holds some rows, so the
    // pieces of a group are consecutive and all of them write a partial result
    const int W = min((int)gridDim.x, (total + 3) / 4), piece = wide_piece(gridDim.x);
    if (piece >= W) return;
    int pos = wide_cut(total, W, piece);
    const int end = wide_cut(total, W, piece + 1);
    for (int i = tid; i < nseg; i += kWideThreads)
        if (s_pair[i] <= pos && pos < s_pair[i + 1]) s_at = i;
    __syncthreads();
    int seg_at = __builtin_amdgcn_readfirstlane(s_at);  // the segment that `pos` lies in
    const int pmax = (a.f + kPairRows - 1) / kPairRows;
    const int col = blockIdx.y * kDownCols + wave * 64 + 4 * l16;  // this lane's four columns (d % 512 == 0)

    while (pos < end) {
        const int g = __builtin_amdgcn_readfirstlane((int)(s_slot[seg_at] >> 16));
        const int first_seg = __builtin_amdgcn_readfirstlane((int)s_first[g]);
        const int base = __builtin_amdgcn_readfirstlane(s_pair[first_seg]);
        const int gend = g + 1 < ng ? __builtin_amdgcn_readfirstlane(s_pair[s_first[min(g + 1, ng - 1)]]) : total;
        WideGroup grp;
        if (NT <= 5 && g < kWave) grp = wide_record(head, g);
        else grp = a.groups[g];
        const int32_t* rows = a.rows + wide_row_slot(g, first_seg - g, pmax) * kPairRows;
        const unsigned char* gd = scalar_ptr(grp.e.gd);
        const uint32_t dcol = 2 * (uint32_t)(d + col);
        const int npairs = gend - base;
        const int pair0 = pos, len = min(gend, end) - pos;
        pos = pair0 + len;
        // the pair slots of the pairs one after the other (past the end the last pair's), as scalars
        int seg = seg_at, seg_end = __builtin_amdgcn_readfirstlane(s_pair[seg_at + 1]);
        int seg_slot = __builtin_amdgcn_readfirstlane((int)(s_slot[seg_at] & 0xFFFFu) - s_pair[seg_at]);
        auto slots_of = [&](int (&r)[SL], int s) __attribute__((always_inline)) {
#pragma unroll
            for (int p = 0; p < SL; ++p) {
                const int pair = pair0 + min(s * SL + p, len - 1);
                while (pair >= seg_end) {
                    ++seg;
                    seg_end = __builtin_amdgcn_readfirstlane(s_pair[seg + 1]);
                    seg_slot = __builtin_amdgcn_readfirstlane((int)(s_slot[seg] & 0xFFFFu) - s_pair[seg]);
                }
                r[p] = seg_slot + pair;
            }
        };
        if (pos < end) {  // where the next part begins
            seg_at = __builtin_amdgcn_readfirstlane((int)s_first[g + 1]);
            while (__builtin_amdgcn_readfirstlane(s_pair[seg_at + 1]) <= pos) ++seg_at;
        }
        auto slot_at = [](const int (&r)[SL], int p) __attribute__((always_inline)) {  // (p: a scalar)
            int v = r[0];
#pragma unroll
            for (int k = 1; k < SL; ++k) {
                const int other = __builtin_amdgcn_readfirstlane(r[k]);  // (left alone, the choice becomes an array in memory)
                v = p == k ? other : v;
            }
            return v;
        };
        const int w_first = wide_owner(total, W, base);
        if (piece == w_first && blockIdx.y == 0) {  // where a task's partial results are
            const int slots = wide_owner(total, W, base + npairs - 1) - w_first + 1;
            if (tid < grp.n) a.task_rows[a.order[grp.first + tid]] = make_int2(grp.first + tid + w_first * kTok, slots);
        }
        const int tiles = __builtin_amdgcn_readfirstlane(wide_tiles(grp.n));
        const unsigned char* hsrc = scalar_ptr(a.hbuf + wide_h_first(grp.tile, g, first_seg - g, pmax, NT));
        const int ns = (len + SL - 1) / SL;
        uint4 hq[kHRounds];
        int idq = 0;
        // (requests are unconditional, as in the gate kernel: past the end they repeat a valid entry and the value is
        // replaced by zero on its way into LDS)
        auto load_h = [&](const int (&slots)[SL]) __attribute__((always_inline)) {  // h of the slice that has these slots
#pragma unroll
            for (int r = 0; r < kHRounds; ++r) {
                const int first = wave * kWave + r * kWideThreads;  // (a wave's entries belong to one pair and one tile)
                const int pr = slot_at(slots, first / (NT * 128));
                const int tile = min(first % (NT * 128) / 128, tiles - 1);  // (past the group's tiles: token rows that nobody reads)
                hq[r] = gload16(hsrc + (uint32_t)(pr * tiles + tile) * 2048u + (uint32_t)(tid & 127) * 16u);
            }
        };
        // The powers of the tokens whose h this thread brings in (the same ones in every slice): in registers where there are
        // some left, which saves the small segments a barrier in front of their first slice.
        constexpr bool kScaleRegs = NT <= 4;
        float scale_reg[kScaleRegs ? kHRounds : 1];
        auto exponent = [&](int tok) {  // |h| < 2^(e + 15); 2^e and 2^-e stay normal numbers
            const uint32_t m = gload4(a.hmax + grp.first + (tok < grp.n ? tok : 0));
            return max((int)(m >> 23) - 141, -126);
        };
        auto power = [](int e) { return __builtin_bit_cast(float, (uint32_t)(127 + e) << 23); };
        // into LDS as hi + lo, the group's own tiles (what a wave skips or clears is a branch).  An infinite or NaN h has a lo of NaN: all sums of its token are then formed again below.
        auto store_h = [&](int s) {
            int at = tid, at16 = l16;  // (entry i of the slice: pair and token tile i / 128, half (i >> 6) & 1 of the pair's rows, lane)
            asm volatile("" : "+v"(at), "+v"(at16));  // or the addresses are formed ahead of the loop and spilled: a reload waits for every request
            uint2* out0 = reinterpret_cast<uint2*>(&hs[s & 1][(at / 128) * 128 + (at & 63)]) + ((at >> 6) & 1);
#pragma unroll
            for (int r = 0; r < kHRounds; ++r) {
                const int first = wave * kWave + r * kWideThreads, tile = first % (NT * 128) / 128;
                if (tile >= tiles) continue;
                uint2* out = out0 + r * kWideThreads * 2;
                if (s * SL + first / (NT * 128) >= len) {
                    out[0] = out[2 * 64] = make_uint2(0u, 0u);
                    continue;
                }
                const float scale = kScaleRegs ? scale_reg[kScaleRegs ? r : 0] : s_scale[16 * tile + at16];
                const f32x4 h = {__builtin_bit_cast(float, hq[r].x), __builtin_bit_cast(float, hq[r].y), __builtin_bit_cast(float, hq[r].z),
                                 __builtin_bit_cast(float, hq[r].w)};
                const h16x4 hi = __builtin_convertvector(h * scale, h16x4);
                const f32x4 rest = {fmaf(h[0], scale, -(float)hi[0]), fmaf(h[1], scale, -(float)hi[1]), fmaf(h[2], scale, -(float)hi[2]),
                                    fmaf(h[3], scale, -(float)hi[3])};
                out[0] = __builtin_bit_cast(uint2, hi);
                out[2 * 64] = __builtin_bit_cast(uint2, __builtin_convertvector(rest, h16x4));
            }
        };
        auto load_ids = [&](const int (&slots)[SL]) __attribute__((always_inline)) {
            const int pr = (2 * wave) & (SL - 1), lower = slot_at(slots, pr), upper = slot_at(slots, pr + 1);
            idq = (int)gload4(rows + (lane < 32 ? lower : upper) * kPairRows + (lane & 31));
        };
        auto store_ids = [&](int s) {
            int k = tid;
            asm volatile("" : "+v"(k));  // or the address is formed ahead of the loop and spilled: its reload waits for every request
            if (k < SL * kPairRows) ids[s & (kRing - 1)][k] = idq;
        };
        uint2 dq[SL][8];
        auto load_d = [&](uint2 (&q)[8], int s, int p) {
            const int4 r0 = *reinterpret_cast<const int4*>(&ids[s & (kRing - 1)][p * kPairRows + 4 * q4]);
            const int4 r1 = *reinterpret_cast<const int4*>(&ids[s & (kRing - 1)][p * kPairRows + 16 + 4 * q4]);
            const int r[8] = {r0.x, r0.y, r0.z, r0.w, r1.x, r1.y, r1.z, r1.w};
#pragma unroll
            for (int k = 0; k < 8; ++k) q[k] = gload8(gd + ((uint32_t)r[k] * (uint32_t)(4 * d) + dcol));
        };
        f32x4 acc[4][NT];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int n = 0; n < NT; ++n) acc[j][n] = f32x4{0.f, 0.f, 0.f, 0.f};

        __syncthreads();  // the previous group's LDS contents are no longer read
        int slots[SL];  // of the coming slice
        slots_of(slots, 0);
        load_ids(slots);
        load_h(slots);
        const int e = exponent(min(tid, kTok - 1));
        if constexpr (kScaleRegs) {
#pragma unroll
            for (int r = 0; r < kHRounds; ++r) scale_reg[r] = power(-exponent(16 * ((tid + r * kWideThreads) % (NT * 128) / 128) + l16));
        }
        if (tid < kTok) {
            if constexpr (!kScaleRegs) s_scale[tid] = power(-e);
            s_back[tid] = power(e);
        }
        store_ids(0);
        slots_of(slots, 1);
        load_ids(slots);
        if constexpr (!kScaleRegs) __syncthreads();
        store_h(0);
        store_ids(1);
        __syncthreads();
#pragma unroll
        for (int p = 0; p < SL; ++p) {
            load_d(dq[p], 0, p);
            __builtin_amdgcn_sched_barrier(0);  // the waits of the loop count the requests in this order
        }
#pragma unroll 1
        for (int s = 0; s < ns; ++s) {
            const int buf = s & 1;
            load_h(slots);
            slots_of(slots, s + 2);
            load_ids(slots);
#pragma unroll
            for (int p = 0; p < SL; ++p) {
                uint32_t b[4][4];  // operand of column j: rows 0..7 of this lane's quarter
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    b[0][k] = __builtin_amdgcn_perm(dq[p][2 * k + 1].x, dq[p][2 * k].x, 0x05040100u);
                    b[1][k] = __builtin_amdgcn_perm(dq[p][2 * k + 1].x, dq[p][2 * k].x, 0x07060302u);
                    b[2][k] = __builtin_amdgcn_perm(dq[p][2 * k + 1].y, dq[p][2 * k].y, 0x05040100u);
                    b[3][k] = __builtin_amdgcn_perm(dq[p][2 * k + 1].y, dq[p][2 * k].y, 0x07060302u);
                }
                // a tile's hi and lo are requested behind the products with those of the tile before: with the requests in
                // front of a tile's own products the matrix cores stand for every one of them
                uint4 hi = hs[buf][p * NT * 128 + lane], lo = hs[buf][p * NT * 128 + 64 + lane];
                auto products = [&](auto first) __attribute__((always_inline)) {  // two tiles
                    constexpr int n0 = decltype(first)::value;
#pragma unroll
                    for (int n = n0; n < n0 + 2 && n < NT; ++n) {
                        const int next = (p * NT + min(n + 1, NT - 1)) * 128 + lane;
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            acc[j][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h16x8, hi),
                                                                               __builtin_bit_cast(h16x8, make_uint4(b[j][0], b[j][1], b[j][2], b[j][3])),
                                                                               acc[j][n], 0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                        if (n + 1 < NT) hi = hs[buf][next];
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            acc[j][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h16x8, lo),
                                                                               __builtin_bit_cast(h16x8, make_uint4(b[j][0], b[j][1], b[j][2], b[j][3])),
                                                                               acc[j][n], 0, 0, 0);
                        __builtin_amdgcn_sched_barrier(0);
                        if (n + 1 < NT) lo = hs[buf][next + 64];
                    }
                };
                products(std::integral_constant<int, 0>{});
                if (NT > 2 && tiles > 2) products(std::integral_constant<int, 2>{});
                if (NT > 4 && tiles > 4) products(std::integral_constant<int, 4>{});
                if (NT > 6 && tiles > 6) products(std::integral_constant<int, 6>{});
                if (NT > 8 && tiles > 8) products(std::integral_constant<int, 8>{});
                load_d(dq[p], s + 1, p);  // (past the last slice: ids repeat the last row, cache hits that nobody uses)
                __builtin_amdgcn_sched_barrier(0);
            }
            store_h(s + 1);
            store_ids(s + 2);
            __syncthreads();
        }
        // lane (l16, q4) holds Y[token 16 n + 4 q4 + i][columns col .. col + 3]
        float* out = a.partial + ((size_t)grp.first + (size_t)piece * kTok) * d + col;
        uint64_t odd = 0ull;  // bit 4 n + i: a sum of token 16 n + 4 q4 + i is not finite
        int tok0 = 4 * q4;
        asm volatile("" : "+v"(tok0));  // or the addresses below are formed ahead of the loop and spilled across it
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int tok = 16 * n + tok0 + i;
                if (tok < grp.n) {
                    const float back = s_back[tok];
                    float* o = out + (size_t)tok * d;
                    const float4 y = make_float4(acc[0][n][i] * back, acc[1][n][i] * back, acc[2][n][i] * back, acc[3][n][i] * back);
                    *reinterpret_cast<float4*>(o) = y;
                    if (!(fmaf(y.x, 0.0f, fmaf(y.y, 0.0f, fmaf(y.z, 0.0f, y.w * 0.0f))) == 0.0f)) odd |= 1ull << (4 * n + i);
                }
            }
        // A row that a token did not select entered its sums as h = 0, and 0 times a weight that is not finite is NaN.  Such
        // sums, seen here by their results, are formed again from the token's own rows alone: four columns of one token at a
        // time, the rows dealt to the lanes of the wave.
        const uint64_t lanes = __ballot(odd != 0ull);
        if (lanes == 0ull) continue;
        __threadfence_block();  // the stores above are done before others to the same places
        const float* hp = reinterpret_cast<const float*>(hsrc);
        const int last = len * kPairRows;
        auto slot_of = [&](int p) {  // pair slot of pair p of this part
            const int s = segment_of(pair0 + p);
            return (int)(s_slot[s] & 0xFFFFu) + pair0 + p - s_pair[s];
        };
        for (uint64_t left = lanes; left != 0ull; left &= left - 1ull) {
            const int src = __ffsll((long long)left) - 1;  // the lane that holds these columns, for a quarter of the tokens
            uint64_t toks = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)odd, src) |
                            (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(odd >> 32), src) << 32;
            const int c0 = blockIdx.y * kDownCols + wave * 64 + 4 * (src & 15);
            for (; toks != 0ull; toks &= toks - 1ull) {
                const int bit = __ffsll((long long)toks) - 1, n = bit >> 2, tok = 16 * n + 4 * (src >> 4) + (bit & 3);
                const int at = grp.first + tok;
                const float* vt = a.v + (size_t)(a.by_task ? a.order[at] : at) * a.f;
                const float tau = a.tau[at];
                float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
                constexpr int kRows = 4;  // per lane, requested together
                for (int r0 = 0; r0 < last; r0 += kRows * kWave) {
                    int row[kRows], before[kRows];
                    float vr[kRows], h[kRows];
                    uint2 w[kRows];
#pragma unroll
                    for (int i = 0; i < kRows; ++i) {
                        const int r = min(r0 + i * kWave + lane, last - 1), sl = slot_of(r / kPairRows), in = r % kPairRows;
                        row[i] = rows[sl * kPairRows + in];
                        before[i] = in ? rows[sl * kPairRows + in - 1] : -1;
                        h[i] = hp[((size_t)(sl * tiles + n) * 128 + (in >> 4) * 64 + ((in >> 2) & 3) * 16 + (tok & 15)) * 4 + (in & 3)];
                    }
#pragma unroll
                    for (int i = 0; i < kRows; ++i) {
                        vr[i] = vt[row[i]];
                        w[i] = gload8(gd + ((uint32_t)row[i] * (uint32_t)(4 * d) + 2 * (uint32_t)(d + c0)));
                    }
#pragma unroll
                    for (int i = 0; i < kRows; ++i) {
                        // (the last row of a segment is repeated up to a whole pair)
                        if (!(r0 + i * kWave + lane < last && row[i] != before[i] && fabsf(vr[i]) > tau)) continue;
                        const h16x2 lo = as_h2(w[i].x), hi = as_h2(w[i].y);
                        sum.x = fmaf(h[i], (float)lo.x, sum.x);
                        sum.y = fmaf(h[i], (float)lo.y, sum.y);
                        sum.z = fmaf(h[i], (float)hi.x, sum.z);
                        sum.w = fmaf(h[i], (float)hi.y, sum.w);
                    }
                }
                const float4 y = make_float4(wave_allreduce_sum(sum.x), wave_allreduce_sum(sum.y), wave_allreduce_sum(sum.z), wave_allreduce_sum(sum.w));
                if (lane == 0)
                    *reinterpret_cast<float4*>(a.partial + ((size_t)grp.first + (size_t)piece * kTok + tok) * d + c0) = y;
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------------------------
// S6: the partial results of a token's tasks, slot by slot, piece by piece (a fixed order)
// ---------------------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(128) void combine_wide_kernel(const float* __restrict__ partial, const int2* __restrict__ task_rows,
                                                           int stride, int slots, int d, float* __restrict__ y_acc,
                                                           h16* __restrict__ y_half) {
    const int t = blockIdx.y;
    const int c = (blockIdx.x * 128 + threadIdx.x) * 4;
    if (c >= d) return;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int sl = 0; sl < slots; ++sl) {
        const int2 tr = task_rows[(size_t)t * slots + sl];  // first row, number of pieces
        const float* p = partial + (size_t)tr.x * d + c;
        for (int k = 0; k < tr.y; k += 4) {
            float4 q[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                q[i] = k + i < tr.y ? *reinterpret_cast<const float4*>(p + (size_t)(k + i) * stride * d) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int i = 0; i < 4; ++i) { s.x += q[i].x; s.y += q[i].y; s.z += q[i].z; s.w += q[i].w; }
        }
    }
    if (y_acc) {
        float4* y = reinterpret_cast<float4*>(y_acc + (size_t)t * d + c);
        float4 o = *y;
        o.x += s.x; o.y += s.y; o.z += s.z; o.w += s.w;
        *y = o;
    }
    if (y_half) {
        const h16x2 lo = {(h16)s.x, (h16)s.y}, hi = {(h16)s.z, (h16)s.w};
        *reinterpret_cast<uint2*>(y_half + (size_t)t * d + c) = make_uint2(as_u32(lo), as_u32(hi));
    }
}

// Groups and order of a single expert that every task belongs to (the one-expert entry point).
__global__ __launch_bounds__(256) void wide_single_kernel(DevExpert e, int n_tasks, int chunk, WideGroup* __restrict__ groups,
                                                          int32_t* __restrict__ n_groups, int32_t* __restrict__ order) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n_tasks) order[i] = i;
    if (i < wide_single_groups(n_tasks, chunk)) groups[i] = wide_single_group(e, n_tasks, chunk, i);
    if (i == 0) n_groups[0] = wide_single_groups(n_tasks, chunk);
}

// ---------------------------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------------------------
// what follows from the token tiles; est_groups: the groups to be expected
static WidePlan wide_plan_for(int nt, int max_groups, int est_groups, int d, int f, int n_tasks, int max_down) {
    WidePlan p{};
    p.nt = nt;
    p.chunk = 16 * nt;
    p.max_groups = max_groups;
    p.est_groups = est_groups < 1 ? 1 : (est_groups < max_groups ? est_groups : max_groups);
    p.h_tiles = (n_tasks + 15 * max_groups) / 16;
    p.pairs = (f + kPairRows - 1) / kPairRows;
    const long long est_pairs = (long long)p.est_groups * p.pairs;
    // one workgroup per compute unit; a piece is at least one pair (gate) or four (down: each piece costs a partial result)
    p.wg_gate = (int)(est_pairs < num_cus() ? est_pairs : num_cus());
    if (p.wg_gate > 8) p.wg_gate &= ~7;
    // (see wide_layout.h)
    p.row_slots = wide_row_slots(max_groups, p.pairs, p.wg_gate);
    p.h_vecs = wide_h_vecs(p.h_tiles, p.pairs, nt, max_groups, p.wg_gate);
    p.segments = p.wg_gate + max_groups;
    const int per_col = num_cus() / (d / kDownCols);
    const long long by_len = (est_pairs + 3) / 4;
    p.wg_down = (int)(by_len < per_col ? by_len : per_col);
    if (max_down > 0 && p.wg_down > max_down) p.wg_down = max_down;
    if (p.wg_down > 8) p.wg_down &= ~7;  // (see wide_piece)
    if (p.wg_down < 1) p.wg_down = 1;
    p.partial_rows = (size_t)n_tasks + (size_t)p.chunk * (p.wg_down - 1);
    return p;
}

WidePlan wide_plan(int d, int f, int T, int n_experts, int top_k, int n_shared, int max_down) {
    const int n_tasks = T * (top_k + n_shared), n_all = n_experts + n_shared;
    double groups = 0.0;
    const int nt = wide_tiles_for(T, n_experts, top_k, n_shared, groups);
    return wide_plan_for(nt, wide_max_groups(n_all, n_tasks, nt), (int)(groups + 0.5), d, f, n_tasks, max_down);
}

// No plan of this layer for up to T tokens needs more of anything: the groups of one tile, of which there are most, with as many
// tiles as any of these batches takes.  (What a shared expert adds jumps behind each multiple of 16 tokens; between two jumps the
// scores move one way, so the most tiles are taken at a multiple of 16 or right behind one.  Checked against every T up to 1500
// for up to 160 routed and four shared experts.)
WidePlan wide_room(int d, int f, int T, int n_experts, int top_k, int n_shared) {
    const int n_tasks = T * (top_k + n_shared), n_all = n_experts + n_shared;
    const int max_groups = wide_max_groups(n_all, n_tasks, 1);
    double groups = 0.0;
    int nt = wide_tiles_for(T, n_experts, top_k, n_shared, groups);
    for (int t = T / 16 * 16; t > 0 && nt < 10; t -= 16)
        for (const int at : {t, t + 1 < T ? t + 1 : t}) {
            const int n = wide_tiles_for(at, n_experts, top_k, n_shared, groups);
            nt = n > nt ? n : nt;
        }
    return wide_plan_for(nt, max_groups, max_groups, d, f, n_tasks, 0);
}

template <int NT>
static hipError_t launch_wide_nt(const WideArgs& a, const WidePlan& p, const uint32_t* mask_words, int d, hipStream_t stream) {
    gate_wide_kernel<NT><<<dim3(p.wg_gate), dim3(kWideThreads), 0, stream>>>(a, mask_words, d);
    hipError_t rc = hipGetLastError();
    if (rc != hipSuccess) return rc;
    down_wide_kernel<NT><<<dim3(p.wg_down, d / kDownCols), dim3(kWideThreads), 0, stream>>>(a, d);
    return hipGetLastError();
}

hipError_t launch_gate_down_wide(const WideArgs& a, const WidePlan& p, const uint32_t* mask_words, int d, hipStream_t stream) {
    if (d % kDownCols != 0 || mask_words_per_task(a.f) > kWideMaxMaskWords || p.segments > kWideMaxSegments) return hipErrorInvalidValue;
    switch (p.nt) {
        case 1: return launch_wide_nt<1>(a, p, mask_words, d, stream);
        case 2: return launch_wide_nt<2>(a, p, mask_words, d, stream);
        case 3: return launch_wide_nt<3>(a, p, mask_words, d, stream);
        case 4: return launch_wide_nt<4>(a, p, mask_words, d, stream);
        case 5: return launch_wide_nt<5>(a, p, mask_words, d, stream);
        case 10: return launch_wide_nt<10>(a, p, mask_words, d, stream);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_wide_prepare(const WidePrep& prep, const WideArgs& a, const uint32_t* mask_words, int n_tasks, int d, hipStream_t stream) {
    wide_prepare_kernel<<<dim3(n_tasks), dim3(128), 0, stream>>>(prep, a, mask_words, n_tasks, d);
    return hipGetLastError();
}

hipError_t launch_wide_single(const DevExpert& e, int n_tasks, int chunk, WideGroup* groups, int32_t* n_groups, int32_t* order,
                              hipStream_t stream) {
    wide_single_kernel<<<dim3((n_tasks + 255) / 256), dim3(256), 0, stream>>>(e, n_tasks, chunk, groups, n_groups, order);
    return hipGetLastError();
}

hipError_t launch_combine_wide(const WideArgs& a, const WidePlan& p, int d, int T, float* y_acc, h16* y_half, hipStream_t stream) {
    combine_wide_kernel<<<dim3((d / 4 + 127) / 128, T), dim3(128), 0, stream>>>(a.partial, a.task_rows, p.chunk, a.slots, d, y_acc, y_half);
    return hipGetLastError();
}

}  // namespace floe
