// S4 + S5 for batches in which an expert sees many tokens (Alg. 1 steps 4-5; the paper itself is batch-1, each token keeps
// its own threshold, mask and result).  The tokens of an expert form groups of up to 16 * NT (NT token tiles of the matrix
// instruction); every row that any token of a group selected is read once for the whole group.
//
//   wide_rows_kernel   per group: ascending list of the union of the tokens' selected channels (from the mask bits), the
//                      selected counts of its tasks.  Beside that the activations in the order of the gate kernel's operand.
//   gate_wide_kernel   A[row][token] = gate_row . x_token.  A wave takes a pair of 16-row tiles.  Rows and activations travel
//                      from memory straight into a ring of three or four slots in LDS, 64 columns of 256 rows and of the group's
//                      tokens each; one barrier per slot.  h = SiLU(A) * v * weight where |v| > tau, else 0, leaves in fp32 in
//                      the lane order of the down kernel's operand, and the largest |h| of each task beside it.
//   down_wide_kernel   Y[token][col] += h[token][row] * down[row][col].  A workgroup owns 512 output columns and a range of
//                      row pairs; a lane fetches 8-byte pieces of eight rows per pair (four pairs in flight), a register
//                      transpose (v_perm_b32) makes the operand.  h passes through LDS as two fp16 numbers (hi + lo),
//                      scaled by a power of two of the token's own that brings its largest |h| to [2^14, 2^15): relative
//                      to that the split is good to 2^-23, whatever the size of h, and no token depends on another.
//   combine_wide       adds a task's partial results.
//
// Division of work: the row pairs of all groups form one sequence; the workgroups cut it into equal pieces, whatever the
// routing did to the group sizes, so the launch is one even round and no compute unit waits for a crowded expert.
//
// What bounds it: the rows (a kernel that only reads them in these pieces runs at 5.9 TB/s whatever the pieces are) and what stands
// between: the start of the streams, once per pass of eight pairs, SiLU behind them, and in the down kernel twice the matrix products.
// Hence groups as large as the accumulators allow (a second group reads the rows again).  Rows that go to registers instead, 16 bytes per
// lane from sixteen rows, cost the cache 64 accesses per request; with the activations' it was busy for half of the cycles and the
// waves stood behind their own requests.  The same holds for v gathered by lane (a tenth of the kernel).  Measured, gate, 8 experts
// d 4096 f 14336 at 90 %: 512 tokens 280 -> 232 us, 64 tokens 152 -> 144, one expert with 24 tokens 28.4 -> 24.6.  Gate + down before
// groups of more than 16 tokens: 64 tokens 364 us, 512 tokens 2425.  Tried: pieces that end where groups end (one expert with 24 tokens
// 24.6 -> 27.8, the others the same).  Down, the same layer with 512 tokens 277 -> 254 us: half of its cycles were matrix products, a
// fifth of these for token tiles that a group does not fill, and the waves stood for the LDS reads in front of each tile's.  (A body per
// number of live tiles, as in the gate kernel, spills: 284.  So does reading one tile ahead with an address register per entry of h, 309:
// a reload waits for every row in flight.)  Up to two tiles it is bound by the rows and did not change.

#include <type_traits>

#include "floe_dev.h"
#include "launch.h"

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

// pairs of union rows of group g
__device__ __forceinline__ int wide_pairs(const int32_t* ucount, int g) { return (ucount[g] + kPairRows - 1) / kPairRows; }

// h of a group lies in [pair][token tile][half of the pair's rows][lane], the group's own tiles only, from this entry on.
__device__ __forceinline__ size_t wide_h_first(const WideGroup& g, int pmax) { return (size_t)g.tile * pmax * 128; }

__device__ __forceinline__ int wide_total(const WideArgs& a, int ng, int lane) {
    int total = 0;
    for (int g0 = 0; g0 < ng; g0 += kWave) {
        const int p = g0 + lane < ng ? wide_pairs(a.ucount, g0 + lane) : 0;
        total += __builtin_amdgcn_readlane(wave_inclusive_scan(p, lane), kWave - 1);
    }
    return total;
}
// the group that holds pair `pos` of the sequence (pos < total) and the position of its first pair; every lane the same
__device__ __forceinline__ void wide_find(const WideArgs& a, int ng, int lane, int pos, int& g, int& base) {
    int run = 0;
    for (int g0 = 0; g0 < ng; g0 += kWave) {
        const int p = g0 + lane < ng ? wide_pairs(a.ucount, g0 + lane) : 0;
        const int inc = wave_inclusive_scan(p, lane);
        const unsigned long long past = __ballot(run + inc > pos);
        if (past) {
            const int l = __ffsll((long long)past) - 1;
            g = g0 + l;
            base = run + __builtin_amdgcn_readlane(inc - p, l);
            return;
        }
        run += __builtin_amdgcn_readlane(inc, kWave - 1);
    }
    g = ng - 1;  // not reached for pos < total
    base = pos;
}
// pair p belongs to piece ((p + 1) * W - 1) / total (see wide_cut)
__device__ __forceinline__ int wide_owner(int total, int W, int p) { return (int)(((long long)(p + 1) * W - 1) / total); }

// ---------------------------------------------------------------------------------------------------------------
// union lists
// ---------------------------------------------------------------------------------------------------------------
// The activations of a token tile in the order of the matrix instruction's operand, [k-step of 32 columns][lane]: what the gate kernel
// copies into LDS as it is.  A wave per token, one block per 2048 columns.  (Beside the lists in one launch: neither needs the other.)
constexpr int kOperandCols = 2048;
__device__ __forceinline__ void operand_tile(const WideArgs& a, int tile, int col0, int max_groups, int d) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int ng = a.n_groups[0];
    int first = 0, n = 0;
    for (int g0 = 0; g0 < ng; g0 += kWave) {
        const WideGroup* mine = a.groups + min(g0 + lane, max_groups - 1);
        const int t0 = mine->tile, len = mine->n, f0 = mine->first;
        const unsigned long long m = __ballot(g0 + lane < ng && tile >= t0 && tile < t0 + wide_tiles(len));
        if (m) {
            const int l = __ffsll((long long)m) - 1;
            first = __builtin_amdgcn_readlane(f0 + 16 * (tile - t0), l);
            n = __builtin_amdgcn_readlane(len - 16 * (tile - t0), l);
            break;
        }
    }
    if (wave >= n) return;  // no such token: nobody looks at its results
    // pieces of 16 bytes: piece p is quarter p % 4 of k-step p / 4; 64 of them per 512 columns
    const uint4* x = reinterpret_cast<const uint4*>(a.x + (size_t)(a.order[first + wave] / a.slots) * d + col0) + lane;
    uint4* out = a.xop + ((size_t)tile * (d / 32) + col0 / 32 + (lane >> 2)) * 64 + (lane & 3) * 16 + wave;
    const int last = min(d - col0, kOperandCols) / 512 - 1;
    const uint4 q0 = x[0], q1 = x[min(1, last) * kWave], q2 = x[min(2, last) * kWave], q3 = x[min(3, last) * kWave];
    out[0] = q0;  // (past the last one the last one again: the same bytes)
    out[min(1, last) * 1024] = q1;
    out[min(2, last) * 1024] = q2;
    out[min(3, last) * 1024] = q3;
}

__global__ __launch_bounds__(1024) void wide_rows_kernel(WideArgs a, const uint32_t* __restrict__ mask_words, int max_groups, int d) {
    constexpr int kWaves = 16;
    __shared__ uint32_t u[kWideMaxMaskWords];
    __shared__ int before[kWideMaxMaskWords];
    __shared__ int wave_tot[kWaves];
    const int parts = (d + kOperandCols - 1) / kOperandCols, op = (int)blockIdx.x - max_groups;
    if (op >= 0) return operand_tile(a, op / parts, op % parts * kOperandCols, max_groups, d);
    const int g = blockIdx.x;
    if (g >= a.n_groups[0]) return;  // the grid is sized for the worst case
    const WideGroup grp = a.groups[g];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int nwords = mask_words_per_task(a.f);
    for (int w = tid; w < nwords; w += 1024) u[w] = 0u;
    __syncthreads();
    for (int i = wave; i < grp.n; i += kWaves) {  // a wave per task
        const int task = a.order[grp.first + i];
        const uint32_t* mw = mask_words + (size_t)task * nwords;
        int c = 0;
        for (int w0 = lane; w0 < nwords; w0 += 8 * kWave) {
            uint32_t m[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) m[q] = w0 + q * kWave < nwords ? mw[w0 + q * kWave] : 0u;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                c += __popc(m[q]);
                if (m[q]) atomicOr(&u[w0 + q * kWave], m[q]);
            }
        }
        c = __builtin_amdgcn_readlane(wave_inclusive_scan(c, lane), kWave - 1);
        if (lane == 0) {
            a.count[task] = c;
            a.hmax[grp.first + i] = 0u;
            a.task_rows[task] = make_int2(0, 0);  // filled in by the down kernel unless the group has no rows at all
        }
    }
    __syncthreads();
    // exclusive prefix of the words' populations; a thread owns two consecutive words
    const int w2 = 2 * tid;
    const int c0 = w2 < nwords ? __popc(u[w2]) : 0, c1 = w2 + 1 < nwords ? __popc(u[w2 + 1]) : 0;
    const int inc = wave_inclusive_scan(c0 + c1, lane);
    if (lane == kWave - 1) wave_tot[wave] = inc;
    __syncthreads();
    int run = inc - c0 - c1, all = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        run += w < wave ? wave_tot[w] : 0;
        all += wave_tot[w];
    }
    if (w2 < nwords) before[w2] = run;
    if (w2 + 1 < nwords) before[w2 + 1] = run + c0;
    if (tid == 0) a.ucount[g] = all;
    __syncthreads();
    int32_t* out = a.urow + (size_t)g * a.f;
    for (int w0 = 2 * wave; w0 < nwords; w0 += 2 * kWaves) {  // two words per wave, a lane per bit
        const int w = w0 + (lane >> 5), b = lane & 31;
        if (w < nwords) {
            const uint32_t m = u[w];
            if ((m >> b) & 1u) out[before[w] + __popc(m & ((1u << b) - 1u))] = w * 32 + b;
        }
    }
}

// ---------------------------------------------------------------------------------------------------------------
// gate
// ---------------------------------------------------------------------------------------------------------------
// Rows and activations travel from memory straight into LDS (global_load_lds_dwordx4), in ring slots that are arrays of their own, so
// that the compiler can tell which requests a read has to wait for.  The waits that matter are placed by hand, in front of the barrier
// that makes a slot everybody's.
template <int NT>
__global__ __launch_bounds__(kWideThreads) void gate_wide_kernel(WideArgs a, int d) {
    constexpr int kTok = 16 * NT;
    constexpr int kSlots = NT <= 3 ? 4 : 3;                  // ring slots that fit 160 KB of LDS
    constexpr int kRowVecs = kWideWaves * 256, kXVecs = 2 * NT * 64;  // per slot: 32 rows x 128 bytes per wave; two k-steps of x
    __shared__ uint4 r0[kRowVecs], r1[kRowVecs], r2[kRowVecs], r3[kSlots > 3 ? kRowVecs : 1];
    __shared__ uint4 x0[kXVecs], x1[kXVecs], x2[kXVecs], x3[kSlots > 3 ? kXVecs : 1];
    __shared__ int s_task[kTok];
    __shared__ float s_w[kTok], s_tau[kTok];
    __shared__ uint32_t s_hmax[kTok];  // bits of the largest finite |h| of this workgroup's rows (ordered like the numbers)
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int l16 = lane & 15, q4 = lane >> 4;
    const int ng = a.n_groups[0];
    const int total = wide_total(a, ng, lane);
    const int W = gridDim.x, piece = wide_piece(W);
    int pos = wide_cut(total, W, piece);
    const int end = wide_cut(total, W, piece + 1);
    const int ns = d / kSliceCols;  // a multiple of eight (d % 512 == 0)
    const int pmax = (a.f + kPairRows - 1) / kPairRows;
    // where in its 128 bytes a row's piece lies in LDS: at piece ^ swizzle(row), so that the sixteen rows of a tile meet all banks
    auto swizzle = [](int row) { return (row & 7) ^ ((row >> 3) & 1); };

    while (pos < end) {  // one group's part of this workgroup's piece at a time
        int g, base;
        wide_find(a, ng, lane, pos, g, base);
        g = __builtin_amdgcn_readfirstlane(g);
        base = __builtin_amdgcn_readfirstlane(base);
        const WideGroup grp = a.groups[g];
        const int count = a.ucount[g];
        const int32_t* rows = a.urow + (size_t)g * a.f;
        const unsigned char* gd = scalar_ptr(grp.e.gd);
        const int seg0 = pos - base, seg1 = min((count + kPairRows - 1) / kPairRows, end - base);
        pos = base + seg1;
        __syncthreads();  // the previous group's task arrays are no longer read
        if (tid < kTok) {
            const int task = a.order[grp.first + (tid < grp.n ? tid : 0)];  // dead token rows repeat the first one
            s_task[tid] = task;
            s_w[tid] = a.task_scale ? a.task_scale[task] : 1.0f;
            s_tau[tid] = a.task_tau[task];
            s_hmax[tid] = 0u;
        }
        const int tiles = wide_tiles(grp.n);
        const unsigned char* xop = scalar_ptr(a.xop + (size_t)grp.tile * (d / 32) * 64);
        // Workgroups start at different column slices: rows are 4 d bytes apart, so workgroups that walk the columns in step
        // ask for the same few memory channels at the same time.  (Two groups of one expert that work on the same rows
        // start alike and share them through the L2.)
        const int rot = (int)((unsigned)(seg0 / 8) * 10u % (unsigned)ns);
        auto col_slice = [&](int s) {  // s-th slice of this workgroup (past the last one: the last one again)
            const int c = min(s, ns - 1) + rot;
            return c < ns ? c : c - ns;
        };
        // equal passes of at most one pair per wave
        const int len = seg1 - seg0;
        const int np = (len + kWideWaves - 1) / kWideWaves;
        const int per = (len + np - 1) / np;
        // live: token tiles that this group fills, of NT at most (a tile without tokens would cost as much as any other)
        auto segment = [&](auto live) __attribute__((always_inline)) {
            constexpr int NL = decltype(live)::value;
            constexpr int kXReq = (2 * NL + kWideWaves - 1) / kWideWaves;  // a wave's share of a slice's activations
            constexpr int kReq = 4 + kXReq;                                // ... and its rows
            for (int p0 = seg0; p0 < seg1; p0 += per) {
                const int pair = p0 + wave;
                const bool active = wave < per && pair < seg1;  // the others only help to bring x in
                auto load_x = [&](uint4* x, int s) {
#pragma unroll
                    for (int k = 0; k < kXReq; ++k) {
                        const int it = min(wave + kWideWaves * k, 2 * NL - 1), ks = it / NL, n = it % NL;
                        dma16(xop + ((uint32_t)(min(n, tiles - 1) * (d / 32) + 2 * col_slice(s) + ks) * 1024u + 16u * lane), x + it * 64);
                    }
                };
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
                uint32_t wo[4];  // byte offsets from gd of the rows' pieces this lane brings in: at most f * 4 d <= 2^31
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int r = 8 * j + (lane >> 3);
                    const int k = min(pair * kPairRows + r, count - 1);  // rows past the end repeat the last one
                    wo[j] = (uint32_t)rows[k] * (uint32_t)(4 * d) + 16u * (uint32_t)((lane & 7) ^ swizzle(r));
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
                        const int k = pair * kPairRows + 16 * t + 4 * q4 + i;
                        row[t][i] = k < count ? rows[k] : -1;
                    }
                int tok0 = l16;
                asm volatile("" : "+v"(tok0));  // or the addresses below are formed ahead of the loop and held across it
                // The v that meet these rows.  Gathered by the lane that needs them they are 64 accesses of 4 bytes to the cache per
                // instruction and a tenth of the kernel's time; where the pair's rows lie within kSpan channels (half of the channels
                // or more selected by somebody) the wave brings the whole span in instead, 16 bytes per lane, and picks from LDS.
                const int last_row = __builtin_amdgcn_readfirstlane(rows[min((pair + 1) * kPairRows, count) - 1]);
                const int row0 = min(__builtin_amdgcn_readfirstlane(rows[pair * kPairRows]), a.f - kSpan);
                const bool span = row0 >= 0 && last_row - row0 < kSpan;
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
                    uint4 vq[2][4];
                    auto load_v = [&](int n) {  // four tokens per request
#pragma unroll
                        for (int k = 0; k < 4; ++k)
                            vq[n & 1][k] = gload16u(a.v + (size_t)s_task[16 * n + 4 * k + q4] * a.f + row0 + 4 * tok0);
                    };
                    load_v(0);
#pragma unroll
                    for (int n = 0; n < NL; ++n) {
                        if (n + 1 < NL) load_v(n + 1);
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            // (stored as a native vector of what is read back: a wave's LDS accesses stay in order, and the compiler
                            // must not take the two for different objects)
                            *reinterpret_cast<f32x4*>(&stage[(4 * k + q4) * kSpan + 4 * (tok0 ^ (4 * k + q4))]) = __builtin_bit_cast(f32x4, vq[n & 1][k]);
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
                            const unsigned char* vt = reinterpret_cast<const unsigned char*>(a.v + (size_t)s_task[16 * n + tok0] * a.f);
#pragma unroll
                            for (int t = 0; t < 2; ++t)
#pragma unroll
                                for (int i = 0; i < 4; ++i) vv[n - n0][t][i] = gloadf(vt + 4 * max(row[t][i], 0));
                        }
#pragma unroll
                        for (int n = n0; n < n0 + kBatch && n < NL; ++n) finish(n, vv[n - n0]);
                    }
                }
                uint4* hb = a.hbuf + wide_h_first(grp, pmax) + (size_t)pair * tiles * 128 + lane;
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
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int l16 = lane & 15, q4 = lane >> 4;
    const int ng = a.n_groups[0];
    const int total = wide_total(a, ng, lane);
    // no more pieces than the actual rows fill with four pairs each: every piece up to the last one holds some rows, so the
    // pieces of a group are consecutive and all of them write a partial result
    const int W = min((int)gridDim.x, (total + 3) / 4), piece = wide_piece(gridDim.x);
    if (piece >= W) return;
    int pos = wide_cut(total, W, piece);
    const int end = wide_cut(total, W, piece + 1);
    const int pmax = (a.f + kPairRows - 1) / kPairRows;
    const int col = blockIdx.y * kDownCols + wave * 64 + 4 * l16;  // this lane's four columns (d % 512 == 0)

    while (pos < end) {
        int g, base;
        wide_find(a, ng, lane, pos, g, base);
        g = __builtin_amdgcn_readfirstlane(g);
        base = __builtin_amdgcn_readfirstlane(base);
        const WideGroup grp = a.groups[g];
        const int count = a.ucount[g];
        const int32_t* rows = a.urow + (size_t)g * a.f;
        const unsigned char* gd = scalar_ptr(grp.e.gd);
        const uint32_t dcol = 2 * (uint32_t)(d + col);
        const int npairs = (count + kPairRows - 1) / kPairRows;
        const int seg0 = pos - base, seg1 = min(npairs, end - base);
        const int len = seg1 - seg0;
        pos = base + seg1;
        const int w_first = wide_owner(total, W, base);
        if (piece == w_first && blockIdx.y == 0) {  // where a task's partial results are
            const int slots = wide_owner(total, W, base + npairs - 1) - w_first + 1;
            if (tid < grp.n) a.task_rows[a.order[grp.first + tid]] = make_int2(grp.first + tid + w_first * kTok, slots);
        }
        const int tiles = __builtin_amdgcn_readfirstlane(wide_tiles(grp.n));
        const unsigned char* hsrc = scalar_ptr(a.hbuf + wide_h_first(grp, pmax) + (size_t)seg0 * tiles * 128);
        const int ns = (len + SL - 1) / SL;
        uint4 hq[kHRounds];
        int idq = 0;
        // (requests are unconditional, as in the gate kernel: past the end they repeat a valid entry and the value is
        // replaced by zero on its way into LDS)
        auto load_h = [&](int s) {  // h of slice s
#pragma unroll
            for (int r = 0; r < kHRounds; ++r) {
                const int first = wave * kWave + r * kWideThreads;  // (a wave's entries belong to one pair and one tile)
                const int pr = min(s * SL + first / (NT * 128), len - 1);
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
        auto load_ids = [&](int s) {
            idq = (int)gload4(rows + min((seg0 + s * SL) * kPairRows + (tid & (SL * kPairRows - 1)), count - 1));
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
        load_ids(0);
        load_h(0);
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
        load_ids(1);
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
            load_h(s + 1);
            load_ids(s + 2);
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
        const int first = seg0 * kPairRows, last = min(count, seg1 * kPairRows);
        for (uint64_t left = lanes; left != 0ull; left &= left - 1ull) {
            const int src = __ffsll((long long)left) - 1;  // the lane that holds these columns, for a quarter of the tokens
            uint64_t toks = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)odd, src) |
                            (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(odd >> 32), src) << 32;
            const int c0 = blockIdx.y * kDownCols + wave * 64 + 4 * (src & 15);
            for (; toks != 0ull; toks &= toks - 1ull) {
                const int bit = __ffsll((long long)toks) - 1, n = bit >> 2, tok = 16 * n + 4 * (src >> 4) + (bit & 3);
                const int task = a.order[grp.first + tok];
                const float* vt = a.v + (size_t)task * a.f;
                const float tau = a.task_tau[task];
                float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
                constexpr int kRows = 4;  // per lane, requested together
                for (int r0 = first; r0 < last; r0 += kRows * kWave) {
                    int row[kRows];
                    float vr[kRows], h[kRows];
                    uint2 w[kRows];
#pragma unroll
                    for (int i = 0; i < kRows; ++i) row[i] = rows[min(r0 + i * kWave + lane, last - 1)];
#pragma unroll
                    for (int i = 0; i < kRows; ++i) {
                        const int r = min(r0 + i * kWave + lane, last - 1), p = r / kPairRows - seg0, in = r % kPairRows;
                        vr[i] = vt[row[i]];
                        h[i] = hp[((size_t)(p * tiles + n) * 128 + (in >> 4) * 64 + ((in >> 2) & 3) * 16 + (tok & 15)) * 4 + (in & 3)];
                        w[i] = gload8(gd + ((uint32_t)row[i] * (uint32_t)(4 * d) + 2 * (uint32_t)(d + c0)));
                    }
#pragma unroll
                    for (int i = 0; i < kRows; ++i) {
                        if (!(r0 + i * kWave + lane < last && fabsf(vr[i]) > tau)) continue;
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
// Token tiles per group: the fewest expected reads of the experts' rows, weighed by what a read costs.  Calls with each number of
// tiles forced, us: 8 experts d 4096 f 14336 INT2 at 85 %, 56 tokens 410 (one tile) 390 394 404 405 416 (ten), 72 tokens 503 419 421 430 432
// 445, 512 tokens 2611 1663 1342 1126 799 740; 64 + 2 experts d 2048 f 1408 INT3 g32, 148 tokens 272 257 259 265 319 355.  Over 255 calls
// the choice costs 4 % on average against the best of the six.  It misses most where one number holds a group and a smaller one its
// halves: 8 experts, 320 tokens 718 (five, taken) 608 (ten); one expert of the same size, 160 tokens 169 (five) 198 (ten, taken), 200
// tokens 240 (five, taken) 203 (ten).
static int wide_tiles_for(int T, int n_experts, int top_k, int n_shared, double& groups) {
    double best = 0.0;
    int best_nt = 0;
    for (const int nt : {1, 2, 3, 4, 5, 10}) {
        const double g = expected_token_groups(n_experts, T, top_k, 16 * nt) + (double)n_shared * ((T + 16 * nt - 1) / (16 * nt));
        const double score = g * (1.0 + (nt <= 5 ? 0.05 : 0.09) * nt);
        if (best_nt == 0 || score < best) {
            best = score;
            best_nt = nt;
            groups = g;
        }
    }
    return best_nt;
}

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
    const int per_col = num_cus() / (d / kDownCols);
    const long long by_len = (est_pairs + 3) / 4;
    p.wg_down = (int)(by_len < per_col ? by_len : per_col);
    if (max_down > 0 && p.wg_down > max_down) p.wg_down = max_down;
    if (p.wg_down > 8) p.wg_down &= ~7;  // (see wide_piece)
    if (p.wg_down < 1) p.wg_down = 1;
    if (p.wg_gate > 8) p.wg_gate &= ~7;
    p.partial_rows = (size_t)n_tasks + (size_t)p.chunk * (p.wg_down - 1);
    return p;
}

WidePlan wide_plan(int d, int f, int T, int n_experts, int top_k, int n_shared, int max_down) {
    const int n_tasks = T * (top_k + n_shared), n_all = n_experts + n_shared;
    double groups = 0.0;
    const int nt = wide_tiles_for(T, n_experts, top_k, n_shared, groups);
    return wide_plan_for(nt, (n_all < n_tasks ? n_all : n_tasks) + n_tasks / (16 * nt), (int)(groups + 0.5), d, f, n_tasks, max_down);
}

// No plan of this layer for up to T tokens needs more of anything: the groups of one tile, of which there are most, with as many
// tiles as any of these batches takes.  (What a shared expert adds jumps behind each multiple of 16 tokens; between two jumps the
// scores move one way, so the most tiles are taken at a multiple of 16 or right behind one.  Checked against every T up to 1500
// for up to 160 routed and four shared experts.)
WidePlan wide_room(int d, int f, int T, int n_experts, int top_k, int n_shared) {
    const int n_tasks = T * (top_k + n_shared), n_all = n_experts + n_shared;
    const int max_groups = (n_all < n_tasks ? n_all : n_tasks) + n_tasks / 16;
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
static hipError_t launch_wide_nt(const WideArgs& a, const WidePlan& p, int d, hipStream_t stream) {
    gate_wide_kernel<NT><<<dim3(p.wg_gate), dim3(kWideThreads), 0, stream>>>(a, d);
    hipError_t rc = hipGetLastError();
    if (rc != hipSuccess) return rc;
    down_wide_kernel<NT><<<dim3(p.wg_down, d / kDownCols), dim3(kWideThreads), 0, stream>>>(a, d);
    return hipGetLastError();
}

hipError_t launch_gate_down_wide(const WideArgs& a, const WidePlan& p, const uint32_t* mask_words, int d, hipStream_t stream) {
    if (d % kDownCols != 0 || mask_words_per_task(a.f) > kWideMaxMaskWords) return hipErrorInvalidValue;
    wide_rows_kernel<<<dim3(p.max_groups + p.h_tiles * ((d + kOperandCols - 1) / kOperandCols)), dim3(1024), 0, stream>>>(a, mask_words, p.max_groups, d);
    hipError_t rc = hipGetLastError();
    if (rc != hipSuccess) return rc;
    switch (p.nt) {
        case 1: return launch_wide_nt<1>(a, p, d, stream);
        case 2: return launch_wide_nt<2>(a, p, d, stream);
        case 3: return launch_wide_nt<3>(a, p, d, stream);
        case 4: return launch_wide_nt<4>(a, p, d, stream);
        case 5: return launch_wide_nt<5>(a, p, d, stream);
        case 10: return launch_wide_nt<10>(a, p, d, stream);
        default: return hipErrorInvalidValue;
    }
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
