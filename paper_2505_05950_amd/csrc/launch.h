// Internal launcher prototypes (host side).  Launchers validate nothing: shapes are checked once in
// api.hip against the limits each kernel states, before anything is enqueued.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "floe_dev.h"
#include "route.h"
#include "wide_plan.h"
#include "xprep.h"

namespace floe {

// Compute units of the current device (read once per device from its properties; 256 on an MI355X, which is also
// what the host-side size queries assume when no device is usable).
int num_cus();

// true when the packed-fp16 kernel applies to this shape (otherwise the generic kernel runs)
inline bool packed_fast_shape(int d, int bits, int group) {
    return (bits == 2 || bits == 3 || bits == 4) && group >= 32 && (d == 1024 || d == 2048 || d == 4096);
}
__host__ __device__ inline int mask_words_per_task(int f) { return (f + 31) / 32; }

// S0
hipError_t launch_quantize(const h16* w, uint32_t* codes, h16* scale, h16* zero, int d, int f, int bits, int group,
                           hipStream_t stream);

// S2 (+ the comparison of S3): v[task][j] for task in [0, n_tasks); token of a task = task / map.slots.
// task_tau / mask_words: when both are given, bit (j % 32) of mask_words[task][j / 32] = (|v_j| > tau[task]).
// route: when given (INT2, group >= 64, packed shapes, n_experts <= 16 only) the kernel routes in place and
// fills the task table itself; map.task_table and task_tau are then ignored.
hipError_t launch_up_gemv(const TaskMap& map, const h16* x, const RouteArgs* route, float* v, const float* task_tau,
                          uint32_t* mask_words, int d, int f, int bits, int group, int n_tasks, hipStream_t stream);
inline bool route_in_place_ok(int d, int bits, int group, int n_experts, int top_k, int n_shared) {
    return bits == 2 && group >= 64 && packed_fast_shape(d, bits, group) && top_k >= 1 && n_experts <= 16 &&
           top_k + n_shared <= 16;
}

// How the fused kernel gets its routing: 2 = all of S1 inside it (<= 16 experts), 1 = softmax and top-k inside it on
// logits that router_logits computed in front (<= 64 experts: repeated by every workgroup the dot products would cost
// more than that launch), 0 = a router kernel in front writes the task table.
inline int fused_route_mode(int n_experts, int top_k, int n_shared) {
    if (top_k < 1 || top_k + n_shared > 16) return 0;
    return n_experts <= 16 ? 2 : (n_experts <= 64 ? 1 : 0);
}

// (S1 +) S2-S5 of a small decode batch in one kernel (packed shapes, any bit width): every workgroup computes v for
// its own block of channels, selects among them and runs gate/down on what it selected (fused_ffn.h).
// With `route` the workgroup also routes in place (fused_route_mode); otherwise map / task_tau /
// task_scale describe the tasks.  partial[task][blocks][d], wg_count[task][blocks] (selected channels per
// workgroup), v_out (optional) [task][f].
// Besides the widths of the packed GEMV also 1536, 2560 and 3072, where a quarter to three eighths of a channel's lanes have no
// unit: the separate kernels there read codes with the generic GEMV, whose precision these instances keep (fused_ffn.h).  The widths
// left, 512 and 3584, have no instances (36 kernels each) and run the separate kernels; unmeasured.
// Calls at 80 %, separate kernels / this, us: INT4 g128 d 2560 f 6911 (6 experts, top-2) 1 token 26.2 / 16.9, 3 43.8 / 29.8, 8 75.1 / 53.7;
// INT2 g64 d 1536 f 5000 (8) 1 token 21.3 / 12.8, 8 46.9 / 29.4; INT3 g64 d 3072 f 8000 (8) 4 tokens 64.8 / 43.1; INT4 g32 d 1536
// f 1408 (64 + 2, top-6) 16 tokens 82.8 / 57.6.
inline bool fused_shape(int d, int bits, int group) {
    return (bits == 2 || bits == 3 || bits == 4) && group >= 32 && (packed_fast_shape(d, bits, group) || d == 1536 || d == 2560 || d == 3072);
}
// lanes that share a channel, a unit of 64 codes each; a width between two powers of two leaves some of them without one
constexpr int fused_lanes(int d) { return d <= 1024 ? 16 : (d <= 2048 ? 32 : 64); }
constexpr int fused_producers = 4;                          // producer waves per workgroup (+ 2 consumers each)
constexpr int fused_wgs_per_cu = 1;                         // workgroups per compute unit the block length aims at
// Channel passes per producer wave: a launch argument between these two.  The kernel exists in two sizes, for blocks of
// kFusedMinPasses passes (all of them in flight at once) and for anything up to kFusedMaxPasses (which sizes its queues).
constexpr int kFusedMinPasses = 7, kFusedMaxPasses = 448;
// passes in flight per producer wave: INT2 stages its codes in LDS, as deep as the ring fits the two result slabs it
// borrows (8 d bytes, 1 KiB per pass); INT3 and INT4 hold 4 passes in registers
constexpr int fused_depth(int d, int bits) { return bits == 2 ? (d / 128 < 14 ? d / 128 : 14) : 4; }
constexpr int kFusedMaxRouted = 64;       // routed experts a workgroup can pick among in place (one per lane)
constexpr int kFusedMaxTasks = 256;       // (token, slot) tasks up to which the fused kernel is considered
// Up to how many tasks a layer call takes the fused kernel.  Measured against the batch kernels (one-token, grouped or wide, whichever
// the call would run), it wins while experts see few tokens each.  us, fused / batch at 60, 80, 90, 95 %: 8 experts d 4096 f 14336 INT2 16 tasks
// 257 / 291  166 / 205  114 / 151  90 / 118, 32 367 / 461  249 / 311  184 / 219  158 / 159, 48 658 / 388  443 / 342  331 / 279  300 / 218; INT4 32 tasks 370 / 453
// 250 / 298  188 / 208  166 / 155; 64 + 2 experts d 2048 f 1408 INT3 128 tasks 106 / 132  69 / 97  51 / 79  47 / 67; 16 experts d 2048 f 5632 INT4 64 tasks
// 156 / 188  118 / 137  100 / 100  86 / 76, 96 261 / 263  206 / 182  185 / 130  164 / 96.  (At d 1024 and 1536 it would win beyond: 8 experts d 1024 f 3584
// INT2 48 tasks 52 / 73  37 / 54  29 / 44  27 / 37.)
// Rule: up to 16 tasks always, beyond that up to four tasks per expert.  fused_tasks_tuned() > 0 replaces the rule.
int fused_tasks_tuned();
void set_fused_tasks_tuned(int n);
inline int fused_task_limit(int n_all) {
    const int t = fused_tasks_tuned();
    const int rule = 4 * n_all > 16 ? 4 * n_all : 16;
    const int lim = t > 0 ? t : rule;
    return lim < kFusedMaxTasks ? lim : kFusedMaxTasks;
}
constexpr int kExpertOrderTasks = 16;     // batches of more tasks run their per-task kernels in expert order
constexpr int kFusedMaxWorkgroups = 2048;
// Widths whose kernels always have their consumers one entry ahead (kAhead in fused_ffn.h); d 4096 has kernels of both kinds.
constexpr bool fused_always_ahead(int d) { return d < 4096; }
struct FusedArgs {
    TaskMap map;
    const h16* x;
    const RouteArgs* route;
    const float* task_tau;
    const float* task_scale;
    float* v_out;
    float* partial;
    int32_t* wg_count;
    int d, f, group, n_tasks, passes;
};
int fused_passes(int d, int f, int bits, int n_tasks, int max_tasks = kExpertOrderTasks);  // 0: not fused
int fused_blocks(int d, int f, int passes);
bool fused_between_pays(int d, int f, int bits, int group, int n_all, int n_tasks, int slots, int passes);  // (widths between the powers of two)
hipError_t launch_fused(const FusedArgs& a, int bits, hipStream_t stream);

// S2 for decode batches on the matrix cores: tokens routed to the same expert share one pass over its codes.
struct TokenGroup {
    int32_t expert;    // index into the layer's expert table
    int32_t n;         // tasks in this chunk (<= chunk size)
    int32_t task[16];  // ascending task ids (token * slots + slot)
};
inline bool mfma_grouped_shape(int d, int bits, int group) {
    return ((bits == 2 && group == 64) || ((bits == 3 || bits == 4) && (group == 32 || group == 64))) &&
           (d == 1024 || d == 2048 || d == 4096);
}
// tasks per group (token rows of the MFMA tile that are used): 8 while experts see few tokens each, else 16
inline int mfma_chunk(int n_all, int n_tasks) { return n_tasks <= 8 * n_all ? 8 : 16; }
inline int mfma_max_groups(int n_all, int n_tasks) {
    return (n_all < n_tasks ? n_all : n_tasks) + n_tasks / mfma_chunk(n_all, n_tasks) + 1;
}
// Grouping pays once experts see about two tokens each; below that the per-token kernels read the same bytes.  The
// INT3 form is bound by its unpacking and by one round trip per eight units on short channels, not by the bytes: it
// needs three to four tokens per expert before it beats the per-token kernel.  grouped_gemv_mode: 0 = this rule,
// 1 = whenever the shape allows, 2 = never (floe_tuning).
int grouped_gemv_mode();
void set_grouped_gemv_mode(int m);
inline bool mfma_batch_pays(int n_all, int n_tasks, int bits) {
    const int mode = grouped_gemv_mode();
    if (mode == 1) return true;
    if (mode == 2) return false;
    return bits == 3 ? 2 * n_tasks >= 7 * n_all : n_tasks >= 2 * n_all;
}
struct WideGroup;
// wide (optional, with order and table): the same tasks cut into as few groups of at most wide_chunk as possible, of equal size per expert
hipError_t launch_group_tokens(const int32_t* task_expert, int n_tasks, int n_all, int chunk, TokenGroup* groups,
                               int32_t* n_groups, hipStream_t stream, int32_t* order = nullptr, int wide_chunk = 0,
                               WideGroup* wide = nullptr, int32_t* n_wide = nullptr, const DevExpert* table = nullptr);
hipError_t launch_up_gemv_grouped(const DevExpert* table, const TokenGroup* groups, const int32_t* n_groups,
                                  int max_groups, int chunk, const h16* x, int slots, float* v, const float* task_tau,
                                  uint32_t* mask_words, int d, int f, int bits, int group, hipStream_t stream);

// S3 as a kernel of its own: per task threshold tau[task]
hipError_t launch_select(const float* v, int f, int n_tasks, const float* tau, int32_t* idx, int32_t* count,
                         hipStream_t stream, bool pad = false);  // pad: -1 behind the last entry of a list
hipError_t launch_pad_list(int32_t* idx, int f, int n_tasks, hipStream_t stream);  // -1 everywhere

// S3 (compaction) + S4 + S5.  Index lists come either from mask_words (then idx/count are WRITTEN, both
// may be nullptr) or, with mask_words == nullptr, from idx/count (read).  partial[task][blk][d].
int gd_blocks(int n_tasks, int f);
// staged: nullptr, or the staging buffer [n_tasks][gd_rows][2][d] whose row k of task q holds channel idx[q][k];
// with rows (staged lists only) the k-th channel of task q sits in row rows[q * f + k] of the whole buffer (-1: absent)
hipError_t launch_gate_down(const TaskMap& map, const h16* staged, int gd_rows, const h16* x, const float* v,
                            const uint32_t* mask_words, int32_t* idx, int32_t* count, const float* task_scale,
                            float* partial, int d, int f, int n_tasks, int nblk, hipStream_t stream,
                            const int32_t* rows = nullptr, const int32_t* order = nullptr);

// S4 + S5 for decode batches, one read of every row that any token of an expert group selected, staged through an LDS ring
// (gate_down_union.hip, union_mode 2).  The groups are those of launch_group_tokens; mask_words / v come from the GEMV kernels.
struct UnionPlan {
    int nblk;                  // channel blocks per group
    int cap;                   // rows a block can hold (a multiple of 16)
    int max_groups;
};
constexpr int kStageWorkgroupsDefault = 32;  // 128 waves x 4 KiB in flight: the link is full, a GEMV beside it keeps most of its speed
int stage_workgroups();
void set_stage_workgroups(int n);  // 0 = default
int union_mode();
int union_kernels_for(int n_all, int n_tasks, int d, int f, int bits, int group);  // 1 matrix cores (wide groups), 2 LDS ring, 3 one-token kernels in expert order
void set_union_mode(int m);
struct UnionArgs {
    const DevExpert* table;
    const TokenGroup* groups;
    const int32_t* n_groups;
    const h16* x;
    const float* v;               // [n_tasks][f]
    const uint32_t* mask_words;   // [n_tasks][words]
    const float* task_scale;      // [n_tasks] or nullptr
    int32_t* count;               // [n_tasks][nblk] selected channels per (task, block), or nullptr
    float* partial;               // [n_tasks][nblk][d]
    int32_t slots, f, cap, nblk;
};
UnionPlan union_plan(int d, int f, int n_tasks, int n_all, int chunk);
bool union_shape_ok(int d, int f, const UnionPlan& p);
hipError_t launch_gate_down_union(const UnionArgs& a, const UnionPlan& p, int d, hipStream_t stream);

// S4 + S5 on the matrix cores for batches in which experts see many tokens (wide_batch.hip): groups of up to 16 * nt tokens.
struct WideGroup {
    int32_t share;             // of its channels, selected, in 2^-20 (from the up projection's first piece, or wide_prepare_kernel)
    int32_t n, first;          // tasks order[first .. first + n)
    int32_t tile;              // number of its first token tile: (first + 15 * group) / 16, so that no two groups share one
    DevExpert e;               // the expert's arrays, so that nobody has to look them up behind this load
};
static_assert(sizeof(WideGroup) == 48, "loaded as three vectors");
// Shares are that many words apart.  (The up projections take them by a pointer of their own: records that a kernel writes to are no longer
// loaded as scalars, 0.6 us of a call with 24 tokens on one expert.)
constexpr int kWideGroupWords = sizeof(WideGroup) / 4;
// all of a record but its share, for kernels that add to the shares meanwhile
__device__ __forceinline__ WideGroup wide_group_less_share(const WideGroup* __restrict__ groups, int g) {
    return WideGroup{0, groups[g].n, groups[g].first, groups[g].tile, groups[g].e};
}

// the groups of a single expert that all of n_tasks tasks belong to: as few of at most `chunk` as possible, of equal size
__host__ __device__ inline int wide_single_groups(int n_tasks, int chunk) { return (n_tasks + chunk - 1) / chunk; }
__host__ __device__ inline int wide_single_len(int n_tasks, int chunk) {
    const int ng = wide_single_groups(n_tasks, chunk);
    return (n_tasks + ng - 1) / ng;
}
__host__ __device__ inline WideGroup wide_single_group(const DevExpert& e, int n_tasks, int chunk, int g) {
    const int len = wide_single_len(n_tasks, chunk), first = g * len < n_tasks ? g * len : n_tasks;
    const int n = n_tasks - first < len ? n_tasks - first : len;
    return WideGroup{0, n, first, (first + 15 * g) >> 4, e};
}

constexpr int kWideMaxMaskWords = 2048;  // f <= 65536
struct WidePlan {
    int nt, chunk, max_groups, est_groups;
    int h_tiles;            // token tiles that the groups can have together
    int pairs;              // pairs of 16-row tiles an expert can have
    int wg_gate, wg_down;   // workgroups (the down kernel: per 512 output columns)
    size_t row_slots;       // pairs of row ids (wide_layout.h)
    size_t h_vecs;          // vectors of h
    int segments;           // entries of the segment table
    size_t partial_rows;    // rows of d floats
};
// What the gate kernel and those behind it find ready: the activations in the order of its operand, [token tile][k-step of 32
// columns][lane], and cleared counters.
struct WidePrep {
    uint4* xop;
    int32_t* count;
    uint32_t* hmax;
    int2* task_rows;
    int4* segments;
    int32_t n_segments;
    const float* task_tau;    // [n_tasks] and by position of the order
    const float* task_scale;  // or nullptr: ones
    float* tau;
    float* scale;
};
struct WideArgs {
    WideGroup* groups;
    const int32_t* n_groups;
    const int32_t* order;     // [n_tasks] tasks sorted by expert
    const h16* x;
    const float* v;           // [n_tasks][f] (see by_task)
    const float* tau;         // [n_tasks] by position of the order, as all that follows but count and task_rows
    const float* scale;       // [n_tasks]
    int32_t* count;           // [n_tasks] selected channels
    int32_t* rows;            // [row_slots][32] union rows of the segments (wide_layout.h)
    int4* segments;           // pairs, pair slot in the group, group, first of its group
    uint4* xop;               // [h_tiles][d / 32][64] activations in operand order (in the place of `partial`, which nobody has written yet)
    uint4* hbuf;              // [h_vecs] h (four floats: rows of a 16-row tile) in lane order
    uint32_t* hmax;           // [n_tasks] bits of the largest finite |h| of task order[i]
    int2* task_rows;          // [n_tasks] first partial row, number of partial rows (chunk rows apart)
    float* partial;           // [partial_rows][d]
    int32_t slots, f, max_groups, pieces;  // pieces: workgroups of the gate kernel
    int32_t by_task;          // v and the mask words are kept by task (up projections that do not know the groups), else by position
};
// S2 for the same groups (up_wide.hip)
inline bool up_wide_shape(int d, int f, int bits, int group) {
    return ((bits == 2 && group == 64) || ((bits == 3 || bits == 4) && (group == 32 || group == 64))) && d % 512 == 0 && f <= 65536;
}
// For shapes that the grouped kernel above takes as well, which of the two, where up_split.hip does not apply: it prepares the
// activations of at most 16 tokens in every workgroup, this one prepares them once and shares a pass over the codes among up to 144.
// Layer calls measured, grouped / this, us: INT4 g32 d 2048 f 5632 (8 experts) at 128 tasks per expert 324 / 275, d 1024 f 3000 (6) at
// 167: 385 / 166; INT4 g32 d 4096 f 2000 (4) at 250: 224 / 196; INT3 g32 d 2048 f 1000 (8) at 125: 134 / 134.  INT2, a wave taking 32
// channels of an expert, by the layer's blocks of 32 channels: 256 blocks (8 experts d 4096 f 1000) 137 / 161, 352 (16, d 2048 f 700)
// 102 / 115, 704 (4, d 2048 f 5632) 101 / 97, 896 (8, d 1024 f 3584) 140 / 134, 1144 (26, d 2048 f 1408) 187 / 178.
inline bool up_wide_pays(int d, int f, int bits, int group, int n_all, int n_tasks) {
    if (!up_wide_shape(d, f, bits, group)) return false;
    if (!mfma_grouped_shape(d, bits, group)) return true;
    if (grouped_gemv_mode() == 2) return false;  // the caller wants one pass per task
    return bits != 2 || (n_tasks >= 32 * n_all && n_all * ((f + 31) / 32) >= 600);
}
struct UpWideArgs {
    WideGroup* groups;
    const int32_t* n_groups;
    const int32_t* order;
    const h16* x;
    float* v;               // by position of the order, like the mask words
    uint32_t* mask_words;
    void* x_frag;   // h_tiles * 16 * d halves: the activations as operands
    void* x_sums;   // x_operand_sum_bytes()
    int32_t n_tasks, d, f, slots, nt, max_groups, est_groups;
    const DevExpert* single;  // one expert that every task belongs to: the launcher fills groups, n_groups and order in as well
    int32_t chunk;            // tasks per group at most
    const int32_t* task_expert;  // (not single, may be null) the same from the tasks' experts, of n_all in `table`; up to kOperandGroups tasks
    const DevExpert* table;
    int32_t n_all;
    WidePrep prep;
};
constexpr int kOperandGroups = 2048;
// the activations as matrix operands (up_split.hip)
struct XOperand {
    uint4* frag;   // [token tile][unit][two instructions][lane]
    float* gsum;   // [token tile][unit][groups per unit][16]
    float* back;   // [token tile][16]
};
size_t x_operand_sum_bytes(int tiles, int d, int group);  // tiles: token tiles that the groups can have together
hipError_t launch_x_operand(const UpWideArgs& a, int bits, int group, XOperand& x, hipStream_t stream);
hipError_t launch_up_wide(const UpWideArgs& a, int bits, int group, hipStream_t stream);

// S2 for groups of up to two token tiles, the columns split over the waves of a workgroup (up_split.hip)
inline bool up_split_shape(int d, int f, int bits, int group) { return up_wide_shape(d, f, bits, group) && d <= 4096; }
// Which of the up projections a batch of wide groups takes.  Layer calls, grouped or wide kernel / this, us: INT2 g64 d 4096 f 14336
// (8 experts, top-2) at 40 tokens 314 / 308, 96: 430 / 415; 4 experts 32 tokens 224 / 217; INT3 g64 d 2048 f 7000 at 64: 177 / 152;
// INT3 g32 d 4096 f 4096 (16 experts) at 128: 420 / 284; d 2048 f 1408 (66 experts, top-6) at 64: 220 / 195, 128: 260 / 245;
// INT4 g64 d 4096 f 7000 (6) at 48: 222 / 202; INT4 g32 d 2048 f 5632 at 64: 138 / 137; widths without a grouped kernel the same.
// With one token tile INT2 leaves the grouped kernel little to share a pass with and less to unpack: 24 tokens 243 / 251.  (Measured since this one
// brings the grouping with it, two launches fewer, at 80 %: 24 tokens 349 / 343, 16 experts d 4096 f 4000 64 tokens 253 / 240, d 2048 f 14336 404 / 375;
// three and four tiles, 66 experts d 2048 f 1408 200 tokens 288 / 258.  The line for INT2 is where it was.)
// More than two token tiles come in parts of two, which up_wide.hip does at once: INT2 at 130 tokens 485 / 470, d 2048 f 4096 (4 experts)
// at 90: 89 / 86; the wider codes leave it fewer token tiles: INT4 g32 d 2048 f 5632 at 200 tokens, that or grouped kernel / this, 184 / 162,
// INT3 g64 d 2048 f 7000 at 200: 196 / 182, INT3 g32 d 4096 f 3000 (4) at 90: 152 / 109.
// Still more tiles in parts as well where up_wide.hip has few blocks of 32 channels to deal to eight waves of each compute unit.  INT3 and
// INT4 by its blocks (layers and one expert, 85 to 250 tokens on an expert): below 512 1.01 to 1.49 times as long as in parts, 512 to 800
// 1.02 to 1.16, 800 to 1200 0.94 to 1.12, beyond 0.83 to 1.15.  INT4 g32 d 4096 f 500 (4 experts) at 260: 159 / 119, f 1408: 176 / 148;
// one expert INT3 g64 f 4000 at 130: 146 / 120.  INT2, where no grouped kernel is the alternative: below 128 1.03 to 1.53 (one expert d 4096
// f 2048 at 130: 148 / 99), 128 to 512 1.00 to 1.36, then even.
inline int up_wide_blocks(int f, int bits, int n_tasks, int est_groups) {
    const int most = bits == 2 ? 144 : 80, per = (n_tasks + est_groups - 1) / est_groups;  // tokens of a part at most, of a group
    return est_groups * ((per + most - 1) / most) * ((f + 31) / 32);
}
inline bool up_split_pays(int d, int f, int bits, int group, int n_all, int n_tasks, const WidePlan& p) {
    if (!up_split_shape(d, f, bits, group)) return false;
    const bool grouped = mfma_grouped_shape(d, bits, group) && n_all > 1;
    if (mfma_grouped_shape(d, bits, group) && grouped_gemv_mode() == 2) return false;  // the caller wants one pass per task
    const int blocks = up_wide_blocks(f, bits, n_tasks, p.est_groups);
    if (bits != 2) return p.nt <= 4 || blocks < 800;
    return grouped ? p.nt == 2 : p.nt <= 2 || blocks < 512;
}
hipError_t launch_up_split(const UpWideArgs& a, int bits, int group, hipStream_t stream);

WidePlan wide_plan(int d, int f, int T, int n_experts, int top_k, int n_shared, int max_down);
WidePlan wide_room(int d, int f, int T, int n_experts, int top_k, int n_shared);
// clears and copies what WidePrep names and fills in the groups' shares, where no up projection of wide groups has done so
hipError_t launch_wide_prepare(const WidePrep& prep, const WideArgs& a, const uint32_t* mask_words, int n_tasks, int d, hipStream_t stream);
hipError_t launch_gate_down_wide(const WideArgs& a, const WidePlan& p, const uint32_t* mask_words, int d, hipStream_t stream);
hipError_t launch_wide_single(const DevExpert& e, int n_tasks, int chunk, WideGroup* groups, int32_t* n_groups, int32_t* order,
                              hipStream_t stream);
hipError_t launch_combine_wide(const WideArgs& a, const WidePlan& p, int d, int T, float* y_acc, h16* y_half, hipStream_t stream);

// The other sparsification candidates of Sec. 3.2.1 (variants.hip): act = a_gate (which = 1) or a_down (which = 2) and
// h = a_gate * a_up for every channel; then the down rows of the kept channels only.
hipError_t launch_gate_dense(const h16* gd, const h16* x, const float* v, int which, int d, int f, int T, float* act,
                             float* hval, hipStream_t stream);
hipError_t launch_down_rows(const h16* gd, const float* hval, const int32_t* idx, const int32_t* count,
                            const float* out_scale, int d, int f, int T, int nblk, float* partial, hipStream_t stream);

// S6 (and the "+=" of the one-expert entry points): reduce partial over blocks and slots.
//   y_acc != nullptr: y_acc[t][i] += sum;   y_half != nullptr: y_half[t][i] = fp16(sum)
hipError_t launch_combine(const float* partial, int d, int T, int slots, int nblk, float* y_acc, h16* y_half,
                          hipStream_t stream);

// S6 of a one-expert call together with S3's index lists (from v and tau)
hipError_t launch_combine_select(const float* partial, int d, int T, int nblk, float* y_acc, const float* v, int f, const float* tau,
                                 int32_t* idx, int32_t* count, bool pad, hipStream_t stream);

// S1: router + per-task table (resolved expert pointers, weight, tau)
struct RouterArgs {
    const h16* router_cm;
    const h16* x;
    const float* tau;
    int32_t tau_stride_t;
    int32_t n_experts, top_k, n_shared, renormalize, d;
    const DevExpert* table;   // all experts of the layer
    DevExpert* task_table;    // [n_tasks] out
    int32_t* task_expert;     // [n_tasks] out
    float* task_weight;       // [n_tasks] out
    float* task_tau;          // [n_tasks] out
    float* logits;            // [T][n_experts] scratch of the two-launch form; nullptr = one launch always
};
// the router matrix of a token is worth spreading over several workgroups from this size on (two launches then)
inline bool router_split_pays(int n_experts, int d, int T) {
    return (size_t)n_experts * d * 2 >= (size_t)128 * 1024 && n_experts >= 32 && T <= 4096;
}
hipError_t launch_router(const RouterArgs& a, int T, hipStream_t stream);
hipError_t launch_router_logits(const RouterArgs& a, int T, hipStream_t stream);  // x . W_r only, into a.logits

// stats: (expert, count, weight) per task
struct SlotStat {
    int32_t expert;
    int32_t count;
    float weight;
    int32_t staged;
};
// count_parts != 0: the count of task q is the sum of count[q * count_parts .. + count_parts)
// staged (optional): rows of task q that were copied host -> HBM for this call; capacity > 0 clamps it (a list
// longer than the staging slab is truncated)
hipError_t launch_stats(const int32_t* task_expert, const int32_t* count, int count_parts, const float* task_weight,
                        SlotStat* stats, int n_tasks, hipStream_t stream, const int32_t* staged = nullptr, int capacity = 0);

// S7
hipError_t launch_stage(const h16* host_gd_dev, int d, int f, const int32_t* idx, const int32_t* count,
                        int capacity_rows, h16* dst, int32_t* overflow, hipStream_t stream);
// all tasks of a layer at once: source matrix of task q = task_table[q].gd (device view of pinned host memory),
// list idx[q][0..count[q]), destination dst[q][capacity_rows][2][d], overflow[q]
// dst_rows != nullptr: chunk k of task q goes to row dst_rows[q * f + k] of the whole buffer (capacity_rows and
// overflow are then not used: the rows were checked when they were assigned)
hipError_t launch_stage_tasks(const DevExpert* task_table, int d, int f, const int32_t* idx, const int32_t* count,
                              int capacity_rows, h16* dst, int32_t* overflow, int n_tasks, hipStream_t stream,
                              const int32_t* dst_rows = nullptr);

// Prefetch bookkeeping (reuse of the hidden state before layer i for layer i + 1, Sec. 3.3):
// after a predicted list has been staged: row_of[q][j] = k for j = idx[q][k], k < min(count[q], capacity), else -1;
// pred_expert / pred_count receive the predicted expert and the number of rows staged.
hipError_t launch_rowmap(const int32_t* idx, const int32_t* count, const int32_t* task_expert, int f, int capacity_rows,
                         int32_t* row_of, int32_t* pred_expert, int32_t* pred_count, int n_tasks, hipStream_t stream);
// per actual task q: find the predicted task of the same token with the same expert; rows[q][k] = staging row of
// channel idx[q][k] (the predicted one, or a fresh row behind the predicted ones / in the spare slab n_tasks + q);
// misses are listed in miss_idx[q][0..miss_count[q]) with their rows in miss_rows; stat[q] = {matched, predicted, hits, misses}
struct PrefetchStat {
    int32_t expert_predicted, predicted, hits, misses;
};
hipError_t launch_match_rows(const int32_t* idx, const int32_t* count, const int32_t* task_expert, int f, int slots,
                             int capacity_rows, const int32_t* row_of, const int32_t* pred_expert,
                             const int32_t* pred_count, int32_t* rows, int32_t* miss_idx, int32_t* miss_rows,
                             int32_t* miss_count, int32_t* overflow, PrefetchStat* stat, int n_tasks,
                             hipStream_t stream, const int32_t* expert_row_of = nullptr, int miss_first_row = 0);
// Resident-channel cache: with expert_row_of ([n_experts][f], pool row of a resident channel or -1) match_rows looks the
// channels up there instead (rows are rows of the whole pool; the misses of task q go to rows miss_first_row +
// q * capacity_rows + m).  launch_cache_load makes channels resident.
hipError_t launch_cache_load(const DevExpert* table, int expert, int d, int f, const int32_t* idx, const int32_t* count,
                             int first_row, int max_rows, h16* pool, int32_t* row_of, hipStream_t stream);

}  // namespace floe
