// S4 + S5 for decode batches (Alg. 1 steps 4-5; the paper itself is batch-1, each token keeps its own threshold, mask
// and result): the tokens that were routed to the same expert share ONE read of every [gate | down] chunk
// (Sec. 3.4.2) that any of them selected.  A row of the union serves exactly the tokens whose mask holds it; for the
// others its contribution is an exact zero.
//
// Per expert group (up to 16 tokens of one expert, see group_tokens_kernel) ONE kernel runs gate and down, the rows
// staged through an LDS ring (union_fused_kernel).  Selected by tuning only: the matrix-core kernels of wide_batch.hip are
// faster for the batches where sharing rows pays.
#include <atomic>
#include <cmath>

#include "floe_dev.h"
#include "launch.h"

namespace floe {

// channel range of block b: whole mask words
__device__ __forceinline__ void union_block_words(int nwords, int nblk, int b, int& w0, int& w1) {
    const int per = (nwords + nblk - 1) / nblk;
    w0 = min(nwords, b * per);
    w1 = min(nwords, w0 + per);
}

// The ascending list of a block's union rows with the token bits of every row -> LDS (wave 0: a lane per mask word, 64
// words per round) and memory (for a separate down kernel); per-task selected counts of the block (statistics).
// s_task / s_w must have been filled (tasks of dead token rows: -1).  Ends with a barrier; returns the number of rows.
__device__ __forceinline__ int union_list(const UnionArgs& a, const TokenGroup* grp, int n_tok, int blk, int* lrow,
                                          uint32_t* lbits, const int* s_task, int* s_count) {
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int nwords = mask_words_per_task(a.f);
    int w0, w1;
    union_block_words(nwords, a.nblk, blk, w0, w1);
    if (wave == 0) {
        int base = 0;
        int csum[16];  // per task: selected channels of this block (statistics)
#pragma unroll
        for (int n = 0; n < 16; ++n) csum[n] = 0;
        for (int wb = w0; wb < w1; wb += 64) {
            const int w = wb + lane;
            uint32_t m[16];
            uint32_t u = 0;
            const int wc = w < w1 ? w : w1 - 1;  // every lane loads a valid word; dead lanes and dead tokens are zeroed
#pragma unroll
            for (int n = 0; n < 16; ++n) m[n] = gload4(a.mask_words + (size_t)s_task[n < n_tok ? n : 0] * nwords + wc);
#pragma unroll
            for (int n = 0; n < 16; ++n) {
                m[n] = (n < n_tok && w < w1) ? m[n] : 0u;
                u |= m[n];
            }
#pragma unroll
            for (int n = 0; n < 16; ++n) csum[n] += __popc(m[n]);
            int inc = __popc(u);
            const int mine = inc;
#pragma unroll
            for (int o = 1; o < kWave; o <<= 1) {
                const int up = __shfl_up(inc, o, kWave);
                if (lane >= o) inc += up;
            }
            int k = base + inc - mine;
            while (u) {
                const int b = __ffs(u) - 1;
                u &= u - 1;
                uint32_t bits = 0;
#pragma unroll
                for (int n = 0; n < 16; ++n) bits |= ((m[n] >> b) & 1u) << n;
                lrow[k] = w * 32 + b;
                lbits[k] = bits;
                ++k;
            }
            base += __shfl(inc, kWave - 1, kWave);
        }
        if (lane == 0) *s_count = base;
        if (a.count) {  // every (task, block) entry is written, also by a block without channels
#pragma unroll
            for (int n = 0; n < 16; ++n) {
                if (n < n_tok) {  // wave-uniform
                    int c = csum[n];
#pragma unroll
                    for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o, kWave);
                    if (lane == 0) a.count[(size_t)s_task[n] * a.nblk + blk] = c;
                }
            }
        }
    }
    __syncthreads();
    return *s_count;
}

// tasks and combine weights of the group's token rows -> LDS (followed by a barrier)
__device__ __forceinline__ void union_tasks(const UnionArgs& a, const TokenGroup* grp, int n_tok, int* s_task, float* s_w) {
    const int tid = threadIdx.x;
    if (tid < 16) {
        const int task = tid < n_tok ? grp->task[tid] : -1;
        s_task[tid] = task;
        s_w[tid] = task >= 0 ? (a.task_scale ? a.task_scale[task] : 1.0f) : 0.0f;
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------------------------------------------
// Steps 4-5 of a group in ONE kernel, the rows staged through LDS: workgroup = (group, block of channels), one wave per
// token of the group (16 waves).  The [gate | down] chunks of the block's union rows travel from HBM straight into a
// ring in LDS (global_load_lds_dwordx4: whole chunks, 1 KiB per wave instruction, no register is held in flight),
// two stages of 64 KiB: while one stage is consumed the next one lands.  A wave keeps its token's activations and its
// 4 d bytes of accumulators in registers, looks at the rows of the stage that ITS token selected, and for each of them
// reads the chunk from LDS: gate . x on packed dot products, SiLU, times v and the combine weight, then y += h * down.
// Every row is read from HBM once per group; the arithmetic is that of the (token, row) pairs that were selected, as in
// the one-token kernels, and each token's sum is formed in ascending channel order (reproducible bit for bit).
// The ring is written by the DMA loads and read with hand-placed ds_read_b128 (the compiler would make every LDS read
// wait for all loads in flight): a stage is read only after every wave has waited for its own loads of that stage and
// passed a barrier, and is requested again only after a barrier behind its last read.
// ---------------------------------------------------------------------------------------------------------------
constexpr int kFusedUnionWaves = 16;
constexpr int kStageBytes = 64 * 1024;

__device__ __forceinline__ void dma1k_to_lds(const void* src_lane, void* lds_wave_base) {
    __builtin_amdgcn_global_load_lds((const FLOE_GLOBAL void*)src_lane, (__attribute__((address_space(3))) void*)lds_wave_base, 16,
                                     0, 0);
}
// two 16-byte reads of this lane at lds_addr and lds_addr + 1 KiB, complete on return
__device__ __forceinline__ void lds_read2x16(uint32_t lds_addr, u32x4& q0, u32x4& q1) {
    asm volatile(
        "ds_read_b128 %0, %2\n\t"
        "ds_read_b128 %1, %2 offset:1024\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(q0), "=&v"(q1)
        : "v"(lds_addr)
        : "memory");
}
__device__ __forceinline__ void lds_read1x16(uint32_t lds_addr, u32x4& q0) {
    asm volatile("ds_read_b128 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(q0) : "v"(lds_addr) : "memory");
}
// A list word read from LDS, complete on return.  Inside the ring loop every LDS and memory read is issued by hand:
// for reads that the compiler places itself it charges a wait for ALL loads in flight (it cannot tell the ring's
// direct-to-LDS loads from anything else), which would serialise the ring.
__device__ __forceinline__ uint32_t lds_read_word(uint32_t lds_addr) {
    uint32_t r;
    asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=&v"(r) : "v"(lds_addr) : "memory");
    return r;
}
// A 4-byte load whose arrival the caller waits for itself (wait_vm_le) before settle() hands the value out.
__device__ __forceinline__ void gload4_unwaited(const void* p, uint32_t& r) {
    asm volatile("global_load_dword %0, %1, off" : "=&v"(r) : "v"(p) : "memory");
}
__device__ __forceinline__ void settle(uint32_t& r) { asm volatile("" : "+v"(r) : : "memory"); }

template <int N>
__device__ __forceinline__ void wait_vm_le() {  // s_waitcnt vmcnt(N) only (gfx9 encoding: bits 3:0 and 15:14)
    static_assert(N >= 0 && N < 64, "vmcnt has six bits");
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

template <int NV>  // d = 512 * NV <= 4096
__global__ __launch_bounds__(kFusedUnionWaves * 64) void union_fused_kernel(UnionArgs a) {
    constexpr int d = 512 * NV;
    constexpr int kChunk = 4 * d;                       // bytes of a [gate | down] chunk
    constexpr int R = kStageBytes / kChunk;             // rows per stage (4 at d = 4096)
    constexpr int kPieces = kStageBytes / 1024;         // 1 KiB pieces per stage
    constexpr int kPpw = kPieces / kFusedUnionWaves;    // pieces a wave requests per stage (4)
    constexpr int kPpr = kChunk / 1024;                 // pieces per row
    static_assert(kPieces % kFusedUnionWaves == 0 && R >= 1, "stage split");
    extern __shared__ __align__(16) unsigned char lds[];
    unsigned char* ring = lds;                                              // [2][kStageBytes]
    int* lrow = reinterpret_cast<int*>(lds + 2 * kStageBytes);              // [cap]
    uint32_t* lbits = reinterpret_cast<uint32_t*>(lrow + a.cap);            // [cap]
    __shared__ int s_task[16];
    __shared__ float s_w[16];
    __shared__ int s_count;

    if ((int)blockIdx.y >= a.n_groups[0]) return;
    const TokenGroup* grp = a.groups + blockIdx.y;
    const int n_tok = grp->n;
    const DevExpert e = a.table[grp->expert];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int blk = blockIdx.x;
    union_tasks(a, grp, n_tok, s_task, s_w);
    const int count = union_list(a, grp, n_tok, blk, lrow, lbits, s_task, &s_count);
    const bool tok_wave = wave < n_tok;  // this wave owns a token (the others only help to request the rows)
    const int task = s_task[tok_wave ? wave : 0];
    const float w = s_w[tok_wave ? wave : 0];
    const float* vt = a.v + (size_t)task * a.f;

    // this token's activations: piece c of the lane = x[(c * 64 + lane) * 8 ..], the layout of a gate column in a chunk
    uint4 xr[NV];
    {
        const uint4* xp = reinterpret_cast<const uint4*>(a.x + (size_t)(task / a.slots) * d);
#pragma unroll
        for (int c = 0; c < NV; ++c) xr[c] = gload16(xp + c * kWave + lane);
    }
    float acc[8 * NV];
#pragma unroll
    for (int i = 0; i < 8 * NV; ++i) acc[i] = 0.0f;
    wait_vm_le<0>();  // x has arrived: inside the loop no wait may be charged to it (it would wait for the ring's loads)

    const int nstages = (count + R - 1) / R;
    const unsigned char* gd8 = reinterpret_cast<const unsigned char*>(e.gd);
    const uint32_t lrow_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) int*)lrow;
    const uint32_t lbits_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint32_t*)lbits;
    auto row_at = [&](int k) { return (int)lds_read_word(lrow_addr + 4 * (uint32_t)min(k, count - 1)); };
    // request stage s: piece p = wave * kPpw + j of the stage is 1 KiB number (p % kPpr) of row (p / kPpr); rows past
    // the end of the list repeat the last row (cache hits that nobody reads), so the request count never varies
    auto request = [&](int s) {
        unsigned char* dst = ring + (s & 1) * kStageBytes;
#pragma unroll
        for (int j = 0; j < kPpw; ++j) {
            const int p = wave * kPpw + j;
            const unsigned char* src = gd8 + (size_t)row_at(s * R + p / kPpr) * kChunk + (p % kPpr) * 1024 + lane * 16;
            dma1k_to_lds(src, dst + p * 1024);
        }
    };
    const uint32_t ring_addr = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)ring + lane * 16;
    if (nstages > 0) request(0);
    for (int s = 0; s < nstages; ++s) {
        // v of the stage's rows for this wave's token: lane r fetches row r's, handed out by readlane after the wait
        uint32_t vraw;
        gload4_unwaited(vt + row_at(s * R + (lane < R ? lane : 0)), vraw);
        if (s + 1 < nstages) {
            request(s + 1);
            wait_vm_le<kPpw>();  // everything but the kPpw requests just made: stage s and v have arrived
        } else {
            wait_vm_le<0>();
        }
        settle(vraw);
        __builtin_amdgcn_s_barrier();  // ... for every wave
        if (tok_wave) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int k = s * R + r;
                if (k >= count) break;                                                     // wave-uniform
                const uint32_t bits = __builtin_amdgcn_readfirstlane(lds_read_word(lbits_addr + 4 * (uint32_t)k));
                if (!((bits >> wave) & 1u)) continue;      // wave-uniform: the token did not select this row
                const uint32_t base = ring_addr + (s & 1) * kStageBytes + r * kChunk;
                float g = 0.0f;
#pragma unroll
                for (int c0 = 0; c0 < NV; c0 += 2) {
                    u32x4 q[2];
                    if (c0 + 1 < NV) lds_read2x16(base + c0 * 1024, q[0], q[1]);
                    else lds_read1x16(base + c0 * 1024, q[0]);
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        if (c0 + c >= NV) break;
                        g = dot2(xr[c0 + c].x, q[c].x, g);
                        g = dot2(xr[c0 + c].y, q[c].y, g);
                        g = dot2(xr[c0 + c].z, q[c].z, g);
                        g = dot2(xr[c0 + c].w, q[c].w, g);
                    }
                }
                g = wave_allreduce_sum(g);
                const float vv = __builtin_bit_cast(float, __builtin_amdgcn_readlane((int)vraw, r));
                const float h = silu(g) * vv * w;
#pragma unroll
                for (int c0 = 0; c0 < NV; c0 += 2) {
                    u32x4 q[2];
                    if (c0 + 1 < NV) lds_read2x16(base + 2 * d + c0 * 1024, q[0], q[1]);
                    else lds_read1x16(base + 2 * d + c0 * 1024, q[0]);
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        if (c0 + c >= NV) break;
                        const uint32_t wds[4] = {q[c].x, q[c].y, q[c].z, q[c].w};
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const h16x2 pr = as_h2(wds[i]);
                            acc[(c0 + c) * 8 + 2 * i + 0] = fmaf(h, (float)pr.x, acc[(c0 + c) * 8 + 2 * i + 0]);
                            acc[(c0 + c) * 8 + 2 * i + 1] = fmaf(h, (float)pr.y, acc[(c0 + c) * 8 + 2 * i + 1]);
                        }
                    }
                }
            }
        }
        __builtin_amdgcn_s_barrier();  // every wave is done with stage s: its half of the ring may be requested again
    }
    // lane owns columns [(c * 64 + lane) * 8, + 8)
    if (tok_wave) {
        float* out = a.partial + ((size_t)task * a.nblk + blk) * d;
#pragma unroll
        for (int c = 0; c < NV; ++c) {
            float4* o4 = reinterpret_cast<float4*>(out + (size_t)(c * kWave + lane) * 8);
            o4[0] = make_float4(acc[c * 8 + 0], acc[c * 8 + 1], acc[c * 8 + 2], acc[c * 8 + 3]);
            o4[1] = make_float4(acc[c * 8 + 4], acc[c * 8 + 5], acc[c * 8 + 6], acc[c * 8 + 7]);
        }
    }
}

// ---------------------------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------------------------
// Which kernels run steps 4-5 of a decode batch (floe_tuning): 0 = chosen per call (below), 1 = matrix cores
// (wide_batch.hip), 2 = rows staged through an LDS ring (union_fused_kernel), 3 = the one-token
// kernels launched in expert order (rows that several tokens selected are shared through the L2).  Process-wide:
// workspace sizes depend on it, so it must not change between a size query and the call that uses the workspace.
static std::atomic<int> g_union_mode{0};
int union_mode() { return g_union_mode.load(std::memory_order_relaxed); }
void set_union_mode(int m) { g_union_mode.store(m >= 0 && m <= 3 ? m : 0, std::memory_order_relaxed); }
// The wide kernels read a row once for a whole group, but bring three more launches with their prologues and the partial results
// of all pieces (half a megabyte per token of a group, whatever the layer); the one-token kernels in expert order read the rows of
// a task each.  What decides is therefore the rows that the tasks would read, in GB with all channels: q tasks per expert times
// the bytes G of the experts' rows, and what the up projections on both sides cost.  Measured, about 3000 calls of layers and 1200 of
// one expert, forced each way, at sparsities of 70, 85 and 95 %: the sparser, the fewer rows there are to share and the later the wide
// way pays.  A line is where it is no slower at 95 %.  one-token / wide, by q G, at 70, 85 and 95 %:
//   layers: 1.9 + 4 G, but at least 4.4 at the widths of the grouped up projection and where there is no wide one
//     8 experts  d 4096 f 4000 INT2 (G 0.52): q G 2.6 1.4 1.04 0.9, 5.2 1.6 1.14 0.95, 6.3 1.8 1.10 1.0;  d 2048 f 4000 INT4 g64: 4.2 0.93 and 5.2 1.05 at 85 %
//     d 4096 INT4 g128, 4 to 16 experts: 2.3 .. 2.8 1.28 - 0.90, 4.6 .. 5.4 1.47 - 0.93;  d 2048 INT3 g32: 2.8 .. 3.4 1.38 1.1 0.96, 4.6 .. 5.4 1.49 1.17 1.03
//     without a grouped kernel (1.9 + 4 G alone): d 3072 f 4000 INT2 (8 experts, G 0.39) 3.1 1.27, 3.9 1.51 at 85 %
//   d 4096 INT3, whose grouped kernel is bound by its unpacking: 2.0
//     f 1200 .. 10000, 4 to 16 experts: 1.3 .. 1.8 1.28 1.15 1.05, 2.3 .. 2.8 1.5 1.25 1.09, 4.6 .. 5.4 1.75 1.45 1.25
//   d 1024 INT4 g32, whose grouped kernel takes two to three times as long as the others: 1.0
//     f 1200 .. 10000, 4 to 66 experts: 0.9 .. 1.3 1.30 1.1 1.09, 2.3 .. 2.8 1.83 1.65 1.50
//   one expert, whose tokens otherwise go through the packed up projection one by one: 2.25 on up to 64 tokens (INT4 from 1.8
//   on, INT2 from 2.0), more take more partial results: 3.0 in any case
//     INT2 d 1024 f 14336: 1.6 (28 tokens) 1.52 1.07 0.91, 2.3 (40) 2.39 1.56 1.10;  d 4096 f 4000: 1.6 (24) 1.51 1.18 0.97, 2.1 (32) 1.59 1.21 1.02
//     INT4 d 2048 f 8000: 1.3 (20) 1.41 1.09 0.94, 1.8 (28) 1.56 1.25 1.09;  d 4096 f 1408 g32: 1.5 (64) 1.30 1.06 0.89, 2.2 (96) 1.42 1.13 0.95, 3.0 (128) 1.71 1.38 1.12
//     INT2 d 2048 f 1408: 1.8 (160) 1.08 0.86 0.71, 3.0 (256) 1.76 1.37 1.19
//   one expert without a wide up projection: 3.6, for the smaller widths 5 (generic) and 10 (packed up projection); at 85 %
//     d 4096 f 4000 INT4 g128: 2.1 (32 tokens) 0.91, 4.2 (64) 1.05;  d 4096 f 1408 INT8: 3.7 (160) 0.98, 4.6 (200) 1.24
//     d 1536 f 4000 INT4 g128: 2.4 (96) 0.79, 4.9 (200) 1.05;  d 2048 f 8000 INT4 g128: 4.2 (64) 0.96, 8.4 (128) 1.10
// Where the wide way's v is less accurate than the other's, the line lies by that and not by the time: the matrix cores drop low bits of
// products with subnormals, error of v against 64 bits (norm) INT2 2e-7 .. 3.6e-7, INT4 2.8e-7 .. 6.5e-7, INT3, whose fields lie lowest,
// 0.9e-5 .. 2.9e-5.  The packed up projection has 1.4e-6 .. 2.8e-6, the generic one 7e-8 .. 8e-8; the grouped one is the same arithmetic.
//   widths whose other way is the generic one: 1.9 + 4 G stays (85 %: d 1536 f 4000 INT4, 8 experts, 2.0 1.21, 3.1 1.53); with more than 64
//   tokens on one expert of a width beyond 4096, which has no split up projection, not below 4.0 (d 5120 f 1408 INT2: 2.8 0.81, 4.6 1.05)
//   INT3 layers with fewer than 3.5 tasks per expert, whose other way is the packed one (mfma_batch_pays): 1.9 + 4 G stays
//   one expert INT3 at the packed widths: 2.85, for the smaller widths 3.4, with groups of 32 5 (85 %: d 4096 f 4000 g64 2.1 1.39, 3.1 1.99)
int union_kernels_for(int n_all, int n_tasks, int d, int f, int bits, int group) {
    const int m = union_mode();
    if (m != 0) return m;
    const double gb = 4e-9 * d * (double)f, qg = n_tasks * gb;  // gb: of one expert
    const bool wide_up = up_wide_shape(d, f, bits, group), packed = packed_fast_shape(d, bits, group);
    double least = 1.9 + 4.0 * gb * n_all;
    if (n_all == 1) {
        if (wide_up && packed && bits != 3)
            return (n_tasks < 64 ? n_tasks : 64) * gb >= 2.25 || qg >= 3.0 ? 1 : 3;
        if (wide_up && d > 4096 && n_tasks > 64 && 64 * gb < 2.0) least = 4.0;
        else if (wide_up && packed) least = d > 2048 ? 2.85 : (group == 32 ? 5.0 : 3.4);
        else if (!wide_up) least = d > 2048 ? 3.6 : (packed ? 10.0 : 5.0);
    } else if (wide_up && d == 4096 && bits == 3 && 2 * n_tasks >= 7 * n_all) {
        least = 2.0;
    } else if (wide_up && d == 1024 && bits == 4 && group == 32) {
        least = 1.0;
    } else if ((!wide_up || packed) && least < 4.4) {
        least = 4.4;
    }
    return qg >= least ? 1 : 3;
}

UnionPlan union_plan(int d, int f, int n_tasks, int n_all, int chunk) {
    UnionPlan p{};
    const int nwords = mask_words_per_task(f);
    p.max_groups = mfma_max_groups(n_all, n_tasks);
    // A workgroup holds its ring in LDS, one per compute unit: a launch of a little less than one
    // workgroup per compute unit for the groups to be expected runs in one round (a few more and it takes two).
    const double est = expected_token_groups(n_all, n_tasks, 1, chunk);
    int nb = (int)(0.95 * num_cus() / (est > 1.0 ? est : 1.0));
    nb = nb < 1 ? 1 : (nb > nwords ? nwords : nb);
    const int by_len = (nwords + 7) / 8;  // at least 256 channels
    nb = nb > by_len ? by_len : nb;
    p.nblk = nb < 1 ? 1 : nb;
    const int per = (nwords + p.nblk - 1) / p.nblk;
    p.cap = ((per * 32 + 15) / 16) * 16;
    return p;
}

static size_t union_lds_bytes(const UnionPlan& p) { return (size_t)2 * kStageBytes + (size_t)p.cap * 8; }

bool union_shape_ok(int d, int f, const UnionPlan& p) {
    // (a token's 4 d bytes of accumulators sit in one wave's registers: d <= 4096)
    return mask_words_per_task(f) <= 2048 && union_lds_bytes(p) <= 150 * 1024 && d <= 4096;
}

template <int NV>
static hipError_t launch_fused_nv(const UnionArgs& a, const UnionPlan& p, hipStream_t stream) {
    constexpr int kMaxDevices = 64;
    static std::atomic<int> attr_bytes[kMaxDevices];  // largest dynamic LDS size enabled so far, per device
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    const int lds = (int)union_lds_bytes(p);
    if (attr_bytes[dev].load(std::memory_order_acquire) < lds) {
        hipError_t rc = hipFuncSetAttribute(reinterpret_cast<const void*>(&union_fused_kernel<NV>),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (rc != hipSuccess) return rc;
        attr_bytes[dev].store(lds, std::memory_order_release);
    }
    union_fused_kernel<NV><<<dim3(p.nblk, p.max_groups), dim3(kFusedUnionWaves * 64), lds, stream>>>(a);
    return hipGetLastError();
}

hipError_t launch_gate_down_union(const UnionArgs& a, const UnionPlan& p, int d, hipStream_t stream) {
    switch (d / 512) {
#define FLOE_NV_CASE(N) case N: return launch_fused_nv<N>(a, p, stream);
        FLOE_NV_CASE(1) FLOE_NV_CASE(2) FLOE_NV_CASE(3) FLOE_NV_CASE(4) FLOE_NV_CASE(5) FLOE_NV_CASE(6)
        FLOE_NV_CASE(7) FLOE_NV_CASE(8)
#undef FLOE_NV_CASE
        default: return hipErrorInvalidValue;
    }
}

}  // namespace floe
