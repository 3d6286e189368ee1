// C ABI of the library (declared in include/floe.h): argument checks, workspace carving, launches.
// Nothing here computes on the host, and there is no host fallback: without a usable HIP device the
// launches fail and the error is returned.
#include "../../include/floe.h"

#include <hip/hip_runtime.h>

#include <vector>

#include "launch.h"

using namespace floe;

static_assert(sizeof(floe_slot_stat) == sizeof(SlotStat), "stat record layout");
static_assert(sizeof(DevExpert) == 32, "expert table entry");

namespace {

thread_local int g_last_hip_error = 0;

int hip_fail(hipError_t e) {
    g_last_hip_error = (int)e;
    return FLOE_EHIP;
}

#define FLOE_HIP(call)                             \
    do {                                           \
        hipError_t e__ = (call);                   \
        if (e__ != hipSuccess) return hip_fail(e__); \
    } while (0)

// Optional measurement hook: when armed for kernel `id`, the next launches of that kernel are bracketed
// by the two events on the launch stream (see floe_profile_kernel in floe.h).
struct ProfileHook {
    int id = 0;
    hipEvent_t start = nullptr, stop = nullptr;
};
thread_local ProfileHook g_hook;

struct Bracket {
    bool on;
    hipStream_t st;
    Bracket(int id, hipStream_t s) : on(g_hook.id == id && g_hook.start && g_hook.stop), st(s) {
        if (on) (void)hipEventRecord(g_hook.start, st);
    }
    ~Bracket() {
        if (on) (void)hipEventRecord(g_hook.stop, st);
    }
};

#define FLOE_LAUNCH(id, stream, call) \
    do {                              \
        Bracket br__((id), (stream)); \
        FLOE_HIP(call);               \
    } while (0)

constexpr size_t kAlign = 256;
size_t align_up(size_t n) { return (n + kAlign - 1) / kAlign * kAlign; }
bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

int check_shape(const floe_shape* s) {
    if (!s) return FLOE_EINVAL;
    if (s->d <= 0 || s->f <= 0 || s->group <= 0) return FLOE_EINVAL;
    if (s->bits != 1 && s->bits != 2 && s->bits != 3 && s->bits != 4 && s->bits != 8) return FLOE_EUNSUPPORTED;
    if (s->group != 32 && s->group != 64 && s->group != 128 && s->group != 256) return FLOE_EUNSUPPORTED;
    if (s->d % s->group != 0) return FLOE_ESHAPE;
    if ((s->group * s->bits) % 32 != 0) return FLOE_ESHAPE;
    if (s->d % 512 != 0) return FLOE_ESHAPE;
    if (s->d > 8192) return FLOE_EUNSUPPORTED;
    if (s->f > (1 << 20)) return FLOE_EUNSUPPORTED;
    return FLOE_OK;
}

int check_T(int T) {
    if (T < 0) return FLOE_EINVAL;
    if (T > 4096) return FLOE_EUNSUPPORTED;
    return FLOE_OK;
}

TaskMap single_map(const floe_expert* e) {
    TaskMap m;
    m.single.codes = e->up_codes;
    m.single.scale = reinterpret_cast<const h16*>(e->up_scale);
    m.single.zero = reinterpret_cast<const h16*>(e->up_zero);
    m.single.gd = reinterpret_cast<const h16*>(e->gd);
    m.task_table = nullptr;
    m.slots = 1;
    return m;
}

// workspace of the one-expert entry points: [v: T*f floats][mask words][counts][idx when not fused][partial: T*nblk*d floats]
struct ExpertWs {
    size_t v_off, mask_off, count_off, idx_off, partial_off, total;
    size_t order_off, ptau_off, wgroups_off, xsum_off, rows_off, segs_off, hbuf_off, hmax_off, trows_off;  // wide path
    int nblk, fused_passes, nblk_fused;
    bool wide;  // many tokens: one read of every row that any of a group of tokens selected (wide_batch.hip)
    WidePlan wp;
};
bool mask_path_ok(int f);
// which form of the wide path a plan may take: the one that a call runs, none, or room for any that a batch of up to T
// tokens can take
enum class Wide { kChosen, kNone, kRoom };
// h of the wide groups; before it is formed the activations that the up projection reads lie in the same place
size_t wide_h_bytes(const WidePlan& p, int d) {
    const size_t h = p.h_vecs * sizeof(uint4), x = (size_t)p.h_tiles * 16 * d * 2;
    return h > x ? h : x;
}
// partial results; before them the activations that the gate kernel reads
size_t wide_partial_bytes(const WidePlan& p, int d) {
    const size_t y = p.partial_rows * d * sizeof(float), x = (size_t)p.h_tiles * 16 * d * 2;
    return y > x ? y : x;
}
// Between the powers of two the fused kernel is what a call prefers, not what it needs: with less workspace (fuse =
// false), or kernels that share rows chosen by hand, it runs the separate ones.
bool fuse_optional(const floe_shape& s) { return !packed_fast_shape(s.d, s.bits, s.group); }
bool fuse_shape(const floe_shape& s, bool fuse) {
    return fused_shape(s.d, s.bits, s.group) && (!fuse_optional(s) || (fuse && union_mode() != 1 && union_mode() != 2));
}
// passes of the fused kernel, 0 where a batch does not run it
int fuse_passes(const floe_shape& s, int n_all, int n_tasks, int slots, int max_tasks, bool tuned, bool fuse) {
    const int passes = fuse_shape(s, fuse) ? fused_passes(s.d, s.f, s.bits, n_tasks, max_tasks) : 0;
    if (!passes || tuned || !fuse_optional(s)) return passes;
    return fused_between_pays(s.d, s.f, s.bits, s.group, n_all, n_tasks, slots, passes) ? passes : 0;
}
ExpertWs expert_ws(const floe_shape* s, int T, Wide form = Wide::kChosen, bool fuse = true) {
    ExpertWs w{};
    w.nblk = gd_blocks(T, s->f);
    w.fused_passes = fuse_passes(*s, 1, T, 1, kExpertOrderTasks, false, fuse);
    w.nblk_fused = w.fused_passes ? fused_blocks(s->d, s->f, w.fused_passes) : 0;
    const int nblk_alloc = w.nblk > w.nblk_fused ? w.nblk : w.nblk_fused;
    size_t o = 0;
    w.v_off = o;       o += align_up((size_t)T * s->f * sizeof(float));
    w.mask_off = o;    o += align_up((size_t)T * mask_words_per_task(s->f) * sizeof(uint32_t));
    w.count_off = o;   o += align_up((size_t)T * (w.nblk_fused > 1 ? w.nblk_fused : 1) * sizeof(int32_t));
    w.wide = form != Wide::kNone && !w.fused_passes && T >= 2 && mask_path_ok(s->f) && union_kernels_for(1, T, s->d, s->f, s->bits, s->group) == 1;
    if (w.wide) {
        w.wp = form == Wide::kRoom ? wide_room(s->d, s->f, T, 1, 1, 0) : wide_plan(s->d, s->f, T, 1, 1, 0, 0);
        w.order_off = o;   o += align_up((size_t)T * 4);
        w.ptau_off = o;    o += align_up((size_t)T * 8);  // thresholds and weights by position
        w.wgroups_off = o; o += align_up((size_t)w.wp.max_groups * sizeof(WideGroup) + 4);
        w.xsum_off = o;    o += align_up(x_operand_sum_bytes(w.wp.h_tiles, s->d, s->group));
        w.rows_off = o;    o += align_up(w.wp.row_slots * 32 * 4);
        w.segs_off = o;    o += align_up((size_t)w.wp.segments * sizeof(int4));
        w.hbuf_off = o;    o += align_up(wide_h_bytes(w.wp, s->d));
        w.hmax_off = o;    o += align_up((size_t)T * 4);
        w.trows_off = o;   o += align_up((size_t)T * sizeof(int2));
    }
    w.idx_off = o;     o += w.fused_passes || w.wide ? 0 : align_up((size_t)T * s->f * sizeof(int32_t));  // list for callers that pass none
    w.partial_off = o; o += align_up(w.wide ? wide_partial_bytes(w.wp, s->d) : (size_t)T * nblk_alloc * s->d * sizeof(float));
    w.total = o;
    return w;
}
// What a caller is asked to bring.  The plans of the wide path jump up and down with T (ten token tiles per group at 160 tokens,
// five at 161); a caller that sizes its workspace once, for its largest batch, has room for the smaller ones, and for the
// one-token kernels that batches below the wide ones run.
size_t one_token_rows(int n_tasks, int f) {  // partial results of the one-token kernels, the most of any batch up to n_tasks
    size_t rows = (size_t)n_tasks * gd_blocks(n_tasks, f);
    for (int n = n_tasks < 64 ? n_tasks : 64; n > 0; --n) {  // (from 64 on eight blocks each, before that up to 16 of them)
        const size_t r = (size_t)n * gd_blocks(n, f);
        rows = r > rows ? r : rows;
    }
    return rows;
}
size_t expert_bytes(const floe_shape* s, int T, bool fuse = true) {
    const ExpertWs w = expert_ws(s, T, Wide::kRoom, fuse);
    if (w.fused_passes && fuse_optional(*s)) {  // (floe_gate_down_sparse runs the separate kernels' plan)
        const size_t separate = expert_bytes(s, T, false);
        return w.total > separate ? w.total : separate;
    }
    if (!w.wide) return w.total;
    const ExpertWs n = expert_ws(s, T, Wide::kNone, fuse);
    const size_t one_token = n.partial_off + one_token_rows(T, s->f) * s->d * sizeof(float);
    return w.total > one_token ? w.total : one_token;
}

// lists longer than this are compacted by the select kernel instead of inside the gate/down kernel
bool mask_path_ok(int f) { return mask_words_per_task(f) <= 2048; }

// workspace of the layer: per-task table, counts, mask words, v, idx, partial
struct LayerWs {
    size_t table_off, expert_off, weight_off, tau_off, logit_off, count_off, mask_off, groups_off, ngroups_off, order_off, v_off, idx_off,
        rows_off, missidx_off, missrows_off, misscount_off, ptau_off, wgroups_off, xsum_off, urow_off, segs_off, hbuf_off, hmax_off, trows_off, partial_off, total;
    int n_tasks, nblk, nblk_fused, fused_passes;
    bool batch_mfma;  // tokens of an expert share one pass over its codes (matrix-core up GEMV)
    bool use_wide;    // batches: one read of every row an expert group selected, on the matrix cores (wide_batch.hip)
    bool up_wide;     // ... and so does the up projection (up_wide.hip)
    bool up_split;    // ... with the columns split over the waves (up_split.hip)
    bool use_union;   // the same through an LDS ring (gate_down_union.hip; by tuning only)
    int chunk;        // tasks per token group
    UnionPlan up;
    WidePlan wp;
};
// max_down: at most so many pieces in the down kernel of the wide path (0: its own choice)
LayerWs layer_plan(const floe_layer* L, int T, Wide form = Wide::kChosen, int max_down = 0, bool fuse = true) {
    LayerWs w{};
    const int slots = L->top_k + L->n_shared;
    w.n_tasks = T * slots;
    w.nblk = gd_blocks(w.n_tasks, L->s.f);
    const int n_all = L->n_experts + L->n_shared;
    w.fused_passes = fuse_passes(L->s, n_all, w.n_tasks, slots, fused_task_limit(n_all), fused_tasks_tuned() > 0, fuse && !L->gd_on_host);
    w.nblk_fused = w.fused_passes ? fused_blocks(L->s.d, L->s.f, w.fused_passes) : 0;
    w.chunk = mfma_chunk(n_all, w.n_tasks);
    // the grouped up GEMV: when forced, or where the fused kernel does not apply and grouping pays
    w.batch_mfma = T >= 2 && mfma_grouped_shape(L->s.d, L->s.bits, L->s.group) &&
                   (grouped_gemv_mode() == 1 || (!w.fused_passes && mfma_batch_pays(n_all, w.n_tasks, L->s.bits)));
    const bool share_rows = !L->gd_on_host && T >= 2 && (!w.fused_passes || w.batch_mfma) && mask_path_ok(L->s.f);
    const int kernels = union_kernels_for(n_all, w.n_tasks, L->s.d, L->s.f, L->s.bits, L->s.group);
    w.use_wide = share_rows && kernels == 1 && form != Wide::kNone;
    const bool room = w.use_wide && form == Wide::kRoom;
    if (share_rows && kernels == 2) {
        w.up = union_plan(L->s.d, L->s.f, w.n_tasks, n_all, w.chunk);
        w.use_union = union_shape_ok(L->s.d, L->s.f, w.up);
    }
    if (room) w.wp = wide_room(L->s.d, L->s.f, T, L->n_experts, L->top_k, L->n_shared);
    else if (w.use_wide) w.wp = wide_plan(L->s.d, L->s.f, T, L->n_experts, L->top_k, L->n_shared, max_down);
    int nblk_alloc = w.nblk > w.nblk_fused ? w.nblk : w.nblk_fused;
    if (w.use_union && w.up.nblk > nblk_alloc) nblk_alloc = w.up.nblk;
    int count_parts = w.nblk_fused > 1 ? w.nblk_fused : 1;
    if (w.use_union && w.up.nblk > count_parts) count_parts = w.up.nblk;
    if (w.use_wide) count_parts = 1;
    size_t o = 0;
    w.table_off = o;  o += align_up((size_t)w.n_tasks * sizeof(DevExpert));
    w.expert_off = o; o += align_up((size_t)w.n_tasks * 4);
    w.weight_off = o; o += align_up((size_t)w.n_tasks * 4);
    w.tau_off = o;    o += align_up((size_t)w.n_tasks * 4);
    // router logits in memory: between the two launches of a split router, or in front of a fused kernel that picks in place
    const bool logits_kept = router_split_pays(L->n_experts, L->s.d, T) ||
                             (w.fused_passes && fused_route_mode(L->n_experts, L->top_k, L->n_shared) == 1);
    w.logit_off = o;  o += logits_kept || room ? align_up((size_t)T * L->n_experts * 4) : 0;
    w.count_off = o;  o += align_up((size_t)w.n_tasks * count_parts * 4);
    w.mask_off = o;   o += align_up((size_t)w.n_tasks * mask_words_per_task(L->s.f) * 4);
    const int mfma_groups = mfma_max_groups(n_all, w.n_tasks) + (room ? w.n_tasks / 8 : 0);  // (groups of 8, or of 16)
    w.groups_off = o; o += align_up((size_t)mfma_groups * sizeof(TokenGroup));
    w.ngroups_off = o; o += align_up(4);
    w.order_off = o;   o += align_up((size_t)w.n_tasks * 4);
    w.v_off = o;      o += align_up((size_t)w.n_tasks * L->s.f * 4);
    w.idx_off = o;    o += w.use_wide ? 0 : align_up((size_t)w.n_tasks * L->s.f * 4);
    // host-resident gate/down: row map and miss lists of the prefetched decode
    const size_t per_list = L->gd_on_host ? align_up((size_t)w.n_tasks * L->s.f * 4) : 0;
    w.rows_off = o;      o += per_list;
    w.missidx_off = o;   o += per_list;
    w.missrows_off = o;  o += per_list;
    w.misscount_off = o; o += L->gd_on_host ? align_up((size_t)w.n_tasks * 4) : 0;
    const size_t wgroups = w.use_wide ? (size_t)w.wp.max_groups : 0;
    w.ptau_off = o;    o += w.use_wide ? align_up((size_t)w.n_tasks * 8) : 0;  // thresholds and weights by position
    w.wgroups_off = o; o += w.use_wide ? align_up(wgroups * sizeof(WideGroup) + 4) : 0;  // (+ their number)
    w.up_split = w.use_wide && up_split_pays(L->s.d, L->s.f, L->s.bits, L->s.group, n_all, w.n_tasks, w.wp);
    w.up_wide = w.use_wide && !w.up_split && up_wide_pays(L->s.d, L->s.f, L->s.bits, L->s.group, n_all, w.n_tasks);
    const bool room_for_x = room && up_wide_shape(L->s.d, L->s.f, L->s.bits, L->s.group) && grouped_gemv_mode() != 2;
    w.xsum_off = o;    o += w.up_wide || w.up_split || room_for_x ? align_up(x_operand_sum_bytes(w.wp.h_tiles, L->s.d, L->s.group)) : 0;
    w.urow_off = o;    o += w.use_wide ? align_up(w.wp.row_slots * 32 * 4) : 0;
    w.segs_off = o;    o += w.use_wide ? align_up((size_t)w.wp.segments * sizeof(int4)) : 0;
    w.hbuf_off = o;    o += w.use_wide ? align_up(wide_h_bytes(w.wp, L->s.d)) : 0;
    w.hmax_off = o;    o += w.use_wide ? align_up((size_t)w.n_tasks * 4) : 0;
    w.trows_off = o;   o += w.use_wide ? align_up((size_t)w.n_tasks * sizeof(int2)) : 0;
    w.partial_off = o;
    o += w.use_wide ? align_up(wide_partial_bytes(w.wp, L->s.d)) : align_up((size_t)w.n_tasks * nblk_alloc * L->s.d * 4);
    w.total = o;
    return w;
}
// What a caller is asked to bring (see expert_bytes)
size_t layer_bytes(const floe_layer* L, int T, bool fuse = true) {
    const LayerWs w = layer_plan(L, T, Wide::kRoom, 0, fuse);
    if (w.fused_passes && fuse_optional(L->s)) {
        const size_t separate = layer_bytes(L, T, false);
        return w.total > separate ? w.total : separate;
    }
    if (!w.use_wide) return w.total;
    const LayerWs n = layer_plan(L, T, Wide::kNone, 0, fuse);
    const size_t one_token = n.partial_off + one_token_rows(w.n_tasks, L->s.f) * L->s.d * 4;
    const size_t most = one_token > n.total ? one_token : n.total;
    return w.total > most ? w.total : most;
}
// The plan of a call with a workspace of `limit` bytes; total > limit: none fits.  With layer_bytes() that is the chosen one.  The
// wide kernels need more workspace per task; a batch that fits less (the static scratch array, say) with the one-token kernels
// keeps fitting: there the wide ones are taken only if they fit as well, with fewer pieces in the down kernel (each costs partial
// results, and nothing else in the plan depends on their number) as long as these occupy a third of the chip.
LayerWs layer_fit(const floe_layer* L, int T, size_t limit, bool fuse = true) {
    LayerWs w = layer_plan(L, T, Wide::kChosen, 0, fuse);
    if (w.fused_passes && w.total > limit && fuse_optional(L->s)) return layer_fit(L, T, limit, false);
    if (!w.use_wide || w.total <= limit || union_mode() == 1) return w;
    const LayerWs n = layer_plan(L, T, Wide::kNone, 0, fuse);
    if (n.total > limit) return w;
    const size_t row = (size_t)L->s.d * 4, rest = w.partial_off + (size_t)w.n_tasks * row;
    const size_t rows = rest < limit ? (limit - rest) / row : 0;  // for the pieces after the first
    const int pieces = (int)(rows / w.wp.chunk + 1) & ~7;
    if (rest > limit || pieces < 8 || 3 * pieces * (L->s.d / 512) < num_cus()) return n;
    const LayerWs fewer = layer_plan(L, T, Wide::kChosen, pieces, fuse);
    return fewer.total <= limit ? fewer : n;  // (the activations in operand order may need more than so few partial results)
}

int check_layer(const floe_layer* L) {
    if (!L) return FLOE_EINVAL;
    int rc = check_shape(&L->s);
    if (rc) return rc;
    if (L->n_experts < 0 || L->top_k < 0 || L->n_shared < 0) return FLOE_EINVAL;
    if (L->top_k > L->n_experts) return FLOE_EINVAL;
    if (L->top_k + L->n_shared <= 0) return FLOE_EINVAL;
    if (L->n_experts > 1024 || L->top_k + L->n_shared > 64) return FLOE_EUNSUPPORTED;
    if (L->top_k > 0 && !L->router_cm) return FLOE_EINVAL;
    if (!L->tau) return FLOE_EINVAL;
    if (L->tau_stride_t != 0 && L->tau_stride_t != L->n_experts + L->n_shared) return FLOE_EINVAL;
    return FLOE_OK;
}

// arguments of the stand-alone router: it fills the per-task arrays at the head of the workspace
RouterArgs router_args(const floe_layer* L, const LayerWs& w, char* base, const h16* xh) {
    RouterArgs ra;
    ra.router_cm = reinterpret_cast<const h16*>(L->router_cm);
    ra.x = xh;
    ra.tau = L->tau;
    ra.tau_stride_t = L->tau_stride_t;
    ra.n_experts = L->n_experts; ra.top_k = L->top_k; ra.n_shared = L->n_shared; ra.renormalize = L->renormalize;
    ra.d = L->s.d;
    ra.table = static_cast<const DevExpert*>(L->dev_table);
    ra.task_table = reinterpret_cast<DevExpert*>(base + w.table_off);
    ra.task_expert = reinterpret_cast<int32_t*>(base + w.expert_off);
    ra.task_weight = reinterpret_cast<float*>(base + w.weight_off);
    ra.task_tau = reinterpret_cast<float*>(base + w.tau_off);
    ra.logits = w.logit_off != w.count_off ? reinterpret_cast<float*>(base + w.logit_off) : nullptr;
    return ra;
}

// S1-S3 of a layer as separate results in the workspace (offloaded paths need the index lists in memory):
// task table / expert / weight / tau, v, idx, count.
int layer_lists(const floe_layer* L, const LayerWs& w, char* base, const h16* xh, int T, hipStream_t st) {
    DevExpert* task_table = reinterpret_cast<DevExpert*>(base + w.table_off);
    int32_t* task_expert = reinterpret_cast<int32_t*>(base + w.expert_off);
    float* task_weight = reinterpret_cast<float*>(base + w.weight_off);
    float* task_tau = reinterpret_cast<float*>(base + w.tau_off);
    int32_t* count = reinterpret_cast<int32_t*>(base + w.count_off);
    float* v = reinterpret_cast<float*>(base + w.v_off);
    int32_t* idx = reinterpret_cast<int32_t*>(base + w.idx_off);
    TaskMap map{};
    map.task_table = task_table;
    map.slots = L->top_k + L->n_shared;
    if (route_in_place_ok(L->s.d, L->s.bits, L->s.group, L->n_experts, L->top_k, L->n_shared)) {
        RouteArgs ro{};
        ro.router_cm = reinterpret_cast<const h16*>(L->router_cm);
        ro.tau = L->tau;
        ro.tau_stride_t = L->tau_stride_t;
        ro.n_experts = L->n_experts; ro.top_k = L->top_k; ro.n_shared = L->n_shared; ro.renormalize = L->renormalize;
        ro.table = static_cast<const DevExpert*>(L->dev_table);
        ro.task_table = task_table;
        ro.task_expert = task_expert; ro.task_weight = task_weight; ro.task_tau = task_tau;
        FLOE_LAUNCH(FLOE_KERNEL_UP_GEMV, st,
                    launch_up_gemv(map, xh, &ro, v, nullptr, nullptr, L->s.d, L->s.f, L->s.bits, L->s.group,
                                   w.n_tasks, st));
    } else {
        const RouterArgs ra = router_args(L, w, base, xh);
        FLOE_LAUNCH(FLOE_KERNEL_ROUTER, st, launch_router(ra, T, st));
        FLOE_LAUNCH(FLOE_KERNEL_UP_GEMV, st,
                    launch_up_gemv(map, xh, nullptr, v, nullptr, nullptr, L->s.d, L->s.f, L->s.bits, L->s.group,
                                   w.n_tasks, st));
    }
    FLOE_LAUNCH(FLOE_KERNEL_SELECT, st, launch_select(v, L->s.f, w.n_tasks, task_tau, idx, count, st));
    return FLOE_OK;
}

}  // namespace

extern "C" {

const char* floe_status_string(int status) {
    switch (status) {
        case FLOE_OK: return "ok";
        case FLOE_EINVAL: return "invalid argument (null pointer, negative size or misaligned buffer)";
        case FLOE_ESHAPE: return "shape violates a divisibility rule (d % group, group*bits % 32, d % 512)";
        case FLOE_EUNSUPPORTED: return "unsupported configuration (bits, group, d, f, T or expert count out of range)";
        case FLOE_EWORKSPACE: return "workspace too small";
        case FLOE_EHIP: return "HIP runtime error (see floe_last_hip_error)";
        default: return "unknown status";
    }
}

int floe_last_hip_error(void) { return g_last_hip_error; }
int floe_abi_version(void) { return 4; }

int floe_profile_kernel(int kernel_id, void* start_event, void* stop_event) {
    if (kernel_id < 0 || kernel_id > FLOE_KERNEL_FUSED_FFN) return FLOE_EINVAL;
    if (kernel_id != 0 && (!start_event || !stop_event)) return FLOE_EINVAL;
    g_hook.id = kernel_id;
    g_hook.start = (hipEvent_t)start_event;
    g_hook.stop = (hipEvent_t)stop_event;
    return FLOE_OK;
}

int floe_tuning(int key, int value) {
    switch (key) {
        case FLOE_TUNE_UNION_KERNELS:
            if (value < 0 || value > 3) return FLOE_EINVAL;
            set_union_mode(value);
            return FLOE_OK;
        case FLOE_TUNE_GROUPED_GEMV:
            if (value < 0 || value > 2) return FLOE_EINVAL;
            set_grouped_gemv_mode(value);
            return FLOE_OK;
        case FLOE_TUNE_FUSED_TASKS:
            if (value < 0 || value > kFusedMaxTasks) return FLOE_EINVAL;
            set_fused_tasks_tuned(value);
            return FLOE_OK;
        case FLOE_TUNE_STAGE_WORKGROUPS:
            if (value < 0 || value > 4096) return FLOE_EINVAL;
            set_stage_workgroups(value);
            return FLOE_OK;
        default: return FLOE_EINVAL;
    }
}

int floe_quantize_expert(const floe_shape* s, const floe_half* w_up_cm, uint32_t* codes, floe_half* scale,
                         floe_half* zero, void* stream) {
    int rc = check_shape(s);
    if (rc) return rc;
    if (!w_up_cm || !codes || !scale || !zero) return FLOE_EINVAL;
    if (!aligned(w_up_cm, 16) || !aligned(codes, 4) || !aligned(scale, 2) || !aligned(zero, 2)) return FLOE_EINVAL;
    FLOE_LAUNCH(FLOE_KERNEL_QUANTIZE, (hipStream_t)stream, launch_quantize(reinterpret_cast<const h16*>(w_up_cm), codes, reinterpret_cast<h16*>(scale),
                             reinterpret_cast<h16*>(zero), s->d, s->f, s->bits, s->group, (hipStream_t)stream));
    return FLOE_OK;
}

int floe_up_gemv(const floe_shape* s, const uint32_t* codes, const floe_half* scale, const floe_half* zero,
                 const floe_half* x, int T, float* v, void* stream) {
    int rc = check_shape(s);
    if (rc) return rc;
    if ((rc = check_T(T))) return rc;
    if (T == 0) return FLOE_OK;  // empty batch: pointers of empty arrays may be NULL
    if (!codes || !scale || !zero || !x || !v) return FLOE_EINVAL;
    if (!aligned(codes, 16) || !aligned(x, 16) || !aligned(v, 4)) return FLOE_EINVAL;
    floe_expert e{};
    e.up_codes = codes; e.up_scale = scale; e.up_zero = zero;
    FLOE_LAUNCH(FLOE_KERNEL_UP_GEMV, (hipStream_t)stream,
                launch_up_gemv(single_map(&e), reinterpret_cast<const h16*>(x), nullptr, v, nullptr, nullptr, s->d, s->f,
                               s->bits, s->group, T, (hipStream_t)stream));
    return FLOE_OK;
}

int floe_select_channels(const float* v, int f, int T, const float* tau, int32_t* idx, int32_t* count, void* stream) {
    if (f <= 0) return FLOE_EINVAL;
    if (f > (1 << 20)) return FLOE_EUNSUPPORTED;
    int rc = check_T(T);
    if (rc) return rc;
    if (T == 0) return FLOE_OK;
    if (!v || !tau || !idx || !count) return FLOE_EINVAL;
    FLOE_LAUNCH(FLOE_KERNEL_SELECT, (hipStream_t)stream, launch_select(v, f, T, tau, idx, count, (hipStream_t)stream));
    return FLOE_OK;
}

size_t floe_expert_workspace_bytes(const floe_shape* s, int T) {
    if (check_shape(s) != FLOE_OK || T < 0) return 0;
    return expert_bytes(s, T);
}

int floe_gate_down_sparse(const floe_expert* e, const floe_half* x, int T, const float* v, const int32_t* idx,
                          const int32_t* count, const float* out_scale, float* y_acc, void* workspace,
                          size_t workspace_bytes, void* stream) {
    if (!e) return FLOE_EINVAL;
    int rc = check_shape(&e->s);
    if (rc) return rc;
    if ((rc = check_T(T))) return rc;
    if (T == 0) return FLOE_OK;
    if (!e->gd || !x || !v || !idx || !count || !y_acc || !workspace) return FLOE_EINVAL;
    if (!aligned(e->gd, 16) || !aligned(x, 16) || !aligned(y_acc, 16) || !aligned(workspace, kAlign)) return FLOE_EINVAL;
    if (e->gd_is_staged && (T > 1 || e->gd_rows < 0)) return FLOE_EINVAL;
    if (!e->gd_is_staged && e->gd_rows != e->s.f) return FLOE_EINVAL;
    const ExpertWs w = expert_ws(&e->s, T, Wide::kNone, false);  // (the lists exist: nothing of the wide path runs here)
    if (workspace_bytes < w.total) return FLOE_EWORKSPACE;
    float* partial = reinterpret_cast<float*>(static_cast<char*>(workspace) + w.partial_off);
    hipStream_t st = (hipStream_t)stream;
    FLOE_LAUNCH(FLOE_KERNEL_GATE_DOWN, st, launch_gate_down(single_map(e), e->gd_is_staged ? reinterpret_cast<const h16*>(e->gd) : nullptr, e->gd_rows,
                              reinterpret_cast<const h16*>(x), v, nullptr,
                              const_cast<int32_t*>(idx), const_cast<int32_t*>(count), out_scale, partial, e->s.d, e->s.f, T, w.nblk, st));
    FLOE_LAUNCH(FLOE_KERNEL_COMBINE, st, launch_combine(partial, e->s.d, T, 1, w.nblk, y_acc, nullptr, st));
    return FLOE_OK;
}

// pad: the entries of idx behind a list become -1 (floe_expert_ffn_sparse_padded)
static int expert_ffn_sparse(const floe_expert* e, const floe_half* x, int T, const float* tau, const float* out_scale,
                             float* y_acc, int32_t* idx, int32_t* count, bool pad, void* workspace, size_t workspace_bytes,
                             void* stream) {
    if (!e) return FLOE_EINVAL;
    int rc = check_shape(&e->s);
    if (rc) return rc;
    if ((rc = check_T(T))) return rc;
    if (T == 0) return FLOE_OK;
    if (!e->up_codes || !e->up_scale || !e->up_zero || !e->gd || !x || !tau || !y_acc || !workspace) return FLOE_EINVAL;
    if ((idx == nullptr) != (count == nullptr)) return FLOE_EINVAL;  // the list and its length come together
    if (!aligned(e->up_codes, 16) || !aligned(e->gd, 16) || !aligned(x, 16) || !aligned(y_acc, 16) ||
        !aligned(workspace, kAlign))
        return FLOE_EINVAL;
    if (e->gd_is_staged || e->gd_rows != e->s.f) return FLOE_EINVAL;
    ExpertWs w = expert_ws(&e->s, T);
    if (w.fused_passes && workspace_bytes < w.total && fuse_optional(e->s)) w = expert_ws(&e->s, T, Wide::kChosen, false);
    if (w.wide && workspace_bytes < w.total && union_mode() != 1) w = expert_ws(&e->s, T, Wide::kNone, false);
    if (workspace_bytes < w.total) return FLOE_EWORKSPACE;
    float* v = reinterpret_cast<float*>(static_cast<char*>(workspace) + w.v_off);
    float* partial = reinterpret_cast<float*>(static_cast<char*>(workspace) + w.partial_off);
    hipStream_t st = (hipStream_t)stream;
    const TaskMap map = single_map(e);
    const h16* xh = reinterpret_cast<const h16*>(x);
    uint32_t* mask = reinterpret_cast<uint32_t*>(static_cast<char*>(workspace) + w.mask_off);
    int nblk = w.nblk;
    if (w.fused_passes) {
        // small batch: GEMV, selection and gate/down in one kernel; the list, when asked for, is cut from v afterwards
        FusedArgs a{};
        a.map = map; a.x = xh; a.route = nullptr; a.task_tau = tau; a.task_scale = out_scale;
        a.v_out = idx ? v : nullptr;
        a.partial = partial;
        a.wg_count = reinterpret_cast<int32_t*>(static_cast<char*>(workspace) + w.count_off);
        a.d = e->s.d; a.f = e->s.f; a.group = e->s.group; a.n_tasks = T; a.passes = w.fused_passes;
        FLOE_LAUNCH(FLOE_KERNEL_FUSED_FFN, st, launch_fused(a, e->s.bits, st));
        nblk = w.nblk_fused;
        if (idx) {
            Bracket list(FLOE_KERNEL_SELECT, st);  // one launch that is both: whichever of the two is armed sees it
            FLOE_LAUNCH(FLOE_KERNEL_COMBINE, st, launch_combine_select(partial, e->s.d, T, nblk, y_acc, v, e->s.f, tau, idx, count, pad, st));
            return FLOE_OK;
        }
    } else if (w.wide) {
        char* base = static_cast<char*>(workspace);
        WideGroup* groups = reinterpret_cast<WideGroup*>(base + w.wgroups_off);
        int32_t* n_groups = reinterpret_cast<int32_t*>(groups + w.wp.max_groups);
        int32_t* order = reinterpret_cast<int32_t*>(base + w.order_off);
        const WidePrep prep{reinterpret_cast<uint4*>(partial), reinterpret_cast<int32_t*>(base + w.count_off),
                            reinterpret_cast<uint32_t*>(base + w.hmax_off), reinterpret_cast<int2*>(base + w.trows_off),
                            reinterpret_cast<int4*>(base + w.segs_off), w.wp.segments, tau, out_scale,
                            reinterpret_cast<float*>(base + w.ptau_off), reinterpret_cast<float*>(base + w.ptau_off) + T};
        WideArgs wa{};
        wa.groups = groups; wa.n_groups = n_groups; wa.order = order; wa.x = xh; wa.v = v;
        wa.tau = prep.tau; wa.scale = prep.scale;
        wa.count = prep.count;
        wa.rows = reinterpret_cast<int32_t*>(base + w.rows_off);
        wa.segments = prep.segments;
        wa.hbuf = reinterpret_cast<uint4*>(base + w.hbuf_off);
        wa.hmax = prep.hmax;
        wa.task_rows = prep.task_rows;
        wa.partial = partial;
        wa.xop = prep.xop;
        wa.slots = 1; wa.f = e->s.f; wa.max_groups = w.wp.max_groups; wa.pieces = w.wp.wg_gate;
        // (scales and zeros need no more than their own alignment here; the wide kernel loads them 16 bytes at a time)
        if (up_wide_shape(e->s.d, e->s.f, e->s.bits, e->s.group) && aligned(e->up_scale, 16) && aligned(e->up_zero, 16)) {
            UpWideArgs u{};
            const bool split = up_split_pays(e->s.d, e->s.f, e->s.bits, e->s.group, 1, T, w.wp);
            u.groups = groups; u.n_groups = n_groups; u.order = order; u.x = xh; u.v = v;
            u.mask_words = mask; u.x_frag = base + w.hbuf_off; u.x_sums = base + w.xsum_off;
            u.n_tasks = T; u.d = e->s.d; u.f = e->s.f; u.slots = 1; u.nt = w.wp.nt;
            u.max_groups = w.wp.max_groups; u.est_groups = w.wp.est_groups;
            u.single = &map.single; u.chunk = w.wp.chunk; u.prep = prep;
            FLOE_LAUNCH(FLOE_KERNEL_UP_GEMV, st, split ? launch_up_split(u, e->s.bits, e->s.group, st) : launch_up_wide(u, e->s.bits, e->s.group, st));
        } else {
            FLOE_HIP(launch_wide_single(map.single, T, w.wp.chunk, groups, n_groups, order, st));
            FLOE_LAUNCH(FLOE_KERNEL_UP_GEMV, st,
                        launch_up_gemv(map, xh, nullptr, v, tau, mask, e->s.d, e->s.f, e->s.bits, e->s.group, T, st));
            FLOE_HIP(launch_wide_prepare(prep, wa, mask, T, e->s.d, st));
        }
        FLOE_LAUNCH(FLOE_KERNEL_GATE_DOWN, st, launch_gate_down_wide(wa, w.wp, mask, e->s.d, st));
        if (idx) FLOE_LAUNCH(FLOE_KERNEL_SELECT, st, launch_select(v, e->s.f, T, tau, idx, count, st, pad));
        FLOE_LAUNCH(FLOE_KERNEL_COMBINE, st, launch_combine_wide(wa, w.wp, e->s.d, T, y_acc, nullptr, st));
        return FLOE_OK;
    } else {
        // a caller that wants no list still gets one built, in the workspace
        if (idx && pad) FLOE_HIP(launch_pad_list(idx, e->s.f, T, st));
        int32_t* idx_ws = idx ? idx : reinterpret_cast<int32_t*>(static_cast<char*>(workspace) + w.idx_off);
        int32_t* count_ws = count ? count : reinterpret_cast<int32_t*>(static_cast<char*>(workspace) + w.count_off);
        if (mask_path_ok(e->s.f)) {
            // the GEMV leaves one mask bit per channel; the gate/down kernel compacts them and writes idx / count
            FLOE_LAUNCH(FLOE_KERNEL_UP_GEMV, st,
                        launch_up_gemv(map, xh, nullptr, v, tau, mask, e->s.d, e->s.f, e->s.bits, e->s.group, T, st));
            FLOE_LAUNCH(FLOE_KERNEL_GATE_DOWN, st,
                        launch_gate_down(map, nullptr, e->s.f, xh, v, mask, idx_ws, count_ws, out_scale, partial, e->s.d,
                                         e->s.f, T, w.nblk, st));
        } else {
            FLOE_LAUNCH(FLOE_KERNEL_UP_GEMV, st,
                        launch_up_gemv(map, xh, nullptr, v, nullptr, nullptr, e->s.d, e->s.f, e->s.bits, e->s.group, T, st));
            FLOE_LAUNCH(FLOE_KERNEL_SELECT, st, launch_select(v, e->s.f, T, tau, idx_ws, count_ws, st));
            FLOE_LAUNCH(FLOE_KERNEL_GATE_DOWN, st,
                        launch_gate_down(map, nullptr, e->s.f, xh, v, nullptr, idx_ws, count_ws, out_scale, partial, e->s.d,
                                         e->s.f, T, w.nblk, st));
        }
    }
    FLOE_LAUNCH(FLOE_KERNEL_COMBINE, st, launch_combine(partial, e->s.d, T, 1, nblk, y_acc, nullptr, st));
    return FLOE_OK;
}

int floe_expert_ffn_sparse(const floe_expert* e, const floe_half* x, int T, const float* tau, const float* out_scale,
                           float* y_acc, int32_t* idx, int32_t* count, void* workspace, size_t workspace_bytes,
                           void* stream) {
    return expert_ffn_sparse(e, x, T, tau, out_scale, y_acc, idx, count, false, workspace, workspace_bytes, stream);
}

int floe_expert_ffn_sparse_padded(const floe_expert* e, const floe_half* x, int T, const float* tau, const float* out_scale,
                                  float* y_acc, int32_t* idx, int32_t* count, void* workspace, size_t workspace_bytes,
                                  void* stream) {
    return expert_ffn_sparse(e, x, T, tau, out_scale, y_acc, idx, count, true, workspace, workspace_bytes, stream);
}

// workspace of the sparsification variants: [v][act][h: T*f floats each][partial: T*nblk*d floats]
namespace {
struct VariantWs {
    size_t v_off, act_off, h_off, partial_off, total;
    int nblk;
};
VariantWs variant_ws(const floe_shape* s, int T) {
    VariantWs w;
    w.nblk = gd_blocks(T, s->f);
    size_t o = 0;
    w.v_off = o;       o += align_up((size_t)T * s->f * 4);
    w.act_off = o;     o += align_up((size_t)T * s->f * 4);
    w.h_off = o;       o += align_up((size_t)T * s->f * 4);
    w.partial_off = o; o += align_up((size_t)T * w.nblk * s->d * 4);
    w.total = o;
    return w;
}
}  // namespace

size_t floe_expert_sparsified_workspace_bytes(const floe_shape* s, int T) {
    if (check_shape(s) != FLOE_OK || T < 0) return 0;
    const size_t a = expert_bytes(s, T), b = variant_ws(s, T).total;
    return a > b ? a : b;
}

int floe_expert_ffn_sparsified(const floe_expert* e, int which, const floe_half* x, int T, const float* tau,
                               const float* out_scale, float* y_acc, int32_t* idx, int32_t* count, void* workspace,
                               size_t workspace_bytes, void* stream) {
    if (which == FLOE_SPARSIFY_UP)
        return floe_expert_ffn_sparse(e, x, T, tau, out_scale, y_acc, idx, count, workspace, workspace_bytes, stream);
    if (which != FLOE_SPARSIFY_GATE && which != FLOE_SPARSIFY_DOWN) return FLOE_EINVAL;
    if (!e) return FLOE_EINVAL;
    int rc = check_shape(&e->s);
    if (rc) return rc;
    if ((rc = check_T(T))) return rc;
    if (T == 0) return FLOE_OK;
    if (!e->up_codes || !e->up_scale || !e->up_zero || !e->gd || !x || !tau || !y_acc || !idx || !count || !workspace)
        return FLOE_EINVAL;
    if (!aligned(e->up_codes, 16) || !aligned(e->gd, 16) || !aligned(x, 16) || !aligned(y_acc, 16) ||
        !aligned(workspace, kAlign))
        return FLOE_EINVAL;
    if (e->gd_is_staged || e->gd_rows != e->s.f) return FLOE_EINVAL;
    const VariantWs w = variant_ws(&e->s, T);
    if (workspace_bytes < w.total) return FLOE_EWORKSPACE;
    char* base = static_cast<char*>(workspace);
    float* v = reinterpret_cast<float*>(base + w.v_off);
    float* act = reinterpret_cast<float*>(base + w.act_off);
    float* hval = reinterpret_cast<float*>(base + w.h_off);
    float* partial = reinterpret_cast<float*>(base + w.partial_off);
    hipStream_t st = (hipStream_t)stream;
    const h16* xh = reinterpret_cast<const h16*>(x);
    const h16* gd = reinterpret_cast<const h16*>(e->gd);
    // a_up for every channel (the quantized up projection), a_gate for every channel, the chosen activation against t,
    // then only the down rows of the channels that are kept
    FLOE_LAUNCH(FLOE_KERNEL_UP_GEMV, st,
                launch_up_gemv(single_map(e), xh, nullptr, v, nullptr, nullptr, e->s.d, e->s.f, e->s.bits, e->s.group, T, st));
    FLOE_HIP(launch_gate_dense(gd, xh, v, which, e->s.d, e->s.f, T, act, hval, st));
    FLOE_LAUNCH(FLOE_KERNEL_SELECT, st, launch_select(act, e->s.f, T, tau, idx, count, st));
    FLOE_LAUNCH(FLOE_KERNEL_GATE_DOWN, st,
                launch_down_rows(gd, hval, idx, count, out_scale, e->s.d, e->s.f, T, w.nblk, partial, st));
    FLOE_LAUNCH(FLOE_KERNEL_COMBINE, st, launch_combine(partial, e->s.d, T, 1, w.nblk, y_acc, nullptr, st));
    return FLOE_OK;
}

size_t floe_layer_table_bytes(const floe_layer* L) {
    if (!L || L->n_experts < 0 || L->n_shared < 0) return 0;
    return align_up((size_t)(L->n_experts + L->n_shared) * sizeof(DevExpert));
}

int floe_layer_build_table(const floe_layer* L, void* dev_table, size_t bytes, void* stream) {
    int rc = check_layer(L);
    if (rc) return rc;
    if (!L->experts || !dev_table || !aligned(dev_table, kAlign)) return FLOE_EINVAL;
    if (bytes < floe_layer_table_bytes(L)) return FLOE_EWORKSPACE;
    const int n = L->n_experts + L->n_shared;
    std::vector<DevExpert> host(n);
    for (int i = 0; i < n; ++i) {
        const floe_expert& e = L->experts[i];
        if (e.s.d != L->s.d || e.s.f != L->s.f || e.s.bits != L->s.bits || e.s.group != L->s.group) return FLOE_ESHAPE;
        if (!e.up_codes || !e.up_scale || !e.up_zero || !e.gd) return FLOE_EINVAL;
        // the batch kernels fetch scales and zeros with 16-byte loads: checked here, once, for every expert, so that
        // no decode call has to look at the host array again
        if (!aligned(e.up_codes, 16) || !aligned(e.gd, 16) || !aligned(e.up_scale, 16) || !aligned(e.up_zero, 16))
            return FLOE_EINVAL;
        if (e.gd_is_staged || e.gd_rows != e.s.f) return FLOE_EINVAL;
        host[i].codes = e.up_codes;
        host[i].scale = reinterpret_cast<const h16*>(e.up_scale);
        host[i].zero = reinterpret_cast<const h16*>(e.up_zero);
        host[i].gd = reinterpret_cast<const h16*>(e.gd);
        if (L->gd_on_host) {  // the kernels read pinned host memory through its device-side address
            void* dev_view = nullptr;
            FLOE_HIP(hipHostGetDevicePointer(&dev_view, const_cast<floe_half*>(e.gd), 0));
            host[i].gd = static_cast<const h16*>(dev_view);
        }
    }
    hipStream_t st = (hipStream_t)stream;
    FLOE_HIP(hipMemcpyAsync(dev_table, host.data(), (size_t)n * sizeof(DevExpert), hipMemcpyHostToDevice, st));
    FLOE_HIP(hipStreamSynchronize(st));
    return FLOE_OK;
}

size_t floe_layer_workspace_bytes(const floe_layer* L, int T) {
    if (check_layer(L) != FLOE_OK || T < 0) return 0;
    return layer_bytes(L, T);
}

int floe_moe_layer_decode(const floe_layer* L, const floe_half* x, int T, floe_half* y, floe_slot_stat* stats,
                          void* workspace, size_t workspace_bytes, void* stream) {
    int rc = check_layer(L);
    if (rc) return rc;
    if ((rc = check_T(T))) return rc;
    if (T == 0) return FLOE_OK;
    if (!L->dev_table || !x || !y || !workspace) return FLOE_EINVAL;
    if (L->gd_on_host) return FLOE_EINVAL;  // host-resident gate/down: use floe_moe_layer_decode_offloaded
    if (!aligned(x, 16) || !aligned(y, 8) || !aligned(workspace, kAlign)) return FLOE_EINVAL;
    const LayerWs w = layer_fit(L, T, workspace_bytes);
    if (workspace_bytes < w.total) return FLOE_EWORKSPACE;
    char* base = static_cast<char*>(workspace);
    DevExpert* task_table = reinterpret_cast<DevExpert*>(base + w.table_off);
    int32_t* task_expert = reinterpret_cast<int32_t*>(base + w.expert_off);
    float* task_weight = reinterpret_cast<float*>(base + w.weight_off);
    float* task_tau = reinterpret_cast<float*>(base + w.tau_off);
    int32_t* count = reinterpret_cast<int32_t*>(base + w.count_off);
    uint32_t* mask = reinterpret_cast<uint32_t*>(base + w.mask_off);
    float* v = reinterpret_cast<float*>(base + w.v_off);
    int32_t* idx = reinterpret_cast<int32_t*>(base + w.idx_off);
    float* partial = reinterpret_cast<float*>(base + w.partial_off);
    hipStream_t st = (hipStream_t)stream;
    const h16* xh = reinterpret_cast<const h16*>(x);
    const int slots = L->top_k + L->n_shared;

    TaskMap map{};
    map.task_table = task_table;
    map.slots = slots;
    const bool mask_ok = mask_path_ok(L->s.f);
    const bool batch_mfma = w.batch_mfma;
    int nblk = w.nblk, count_parts = 0;
    if (w.fused_passes && !batch_mfma) {
        // small batch: [(router +) up GEMV + selection + gate/down on the workgroup's own channels] -> [combine];
        // with <= 16 experts the router runs inside the same kernel; with <= 64 its dot products run in a kernel in front
        // and softmax / top-k inside; otherwise the whole router runs in front
        const int route_mode = fused_route_mode(L->n_experts, L->top_k, L->n_shared);
        const bool in_place = route_mode != 0;
        RouteArgs ro{};
        ro.router_cm = reinterpret_cast<const h16*>(L->router_cm);
        ro.tau = L->tau;
        ro.tau_stride_t = L->tau_stride_t;
        ro.n_experts = L->n_experts; ro.top_k = L->top_k; ro.n_shared = L->n_shared; ro.renormalize = L->renormalize;
        ro.table = static_cast<const DevExpert*>(L->dev_table);
        ro.task_table = task_table;
        ro.task_expert = task_expert; ro.task_weight = task_weight; ro.task_tau = task_tau;
        if (route_mode == 0) {
            const RouterArgs ra = router_args(L, w, base, xh);
            FLOE_LAUNCH(FLOE_KERNEL_ROUTER, st, launch_router(ra, T, st));
        } else if (route_mode == 1) {
            const RouterArgs ra = router_args(L, w, base, xh);
            if (!ra.logits) return FLOE_EWORKSPACE;
            FLOE_LAUNCH(FLOE_KERNEL_ROUTER, st, launch_router_logits(ra, T, st));
            ro.logits = ra.logits;
        }
        FusedArgs a{};
        a.map = map; a.x = xh; a.route = in_place ? &ro : nullptr; a.task_tau = task_tau; a.task_scale = task_weight;
        a.v_out = nullptr; a.partial = partial; a.wg_count = count;
        a.d = L->s.d; a.f = L->s.f; a.group = L->s.group; a.n_tasks = w.n_tasks; a.passes = w.fused_passes;
        FLOE_LAUNCH(FLOE_KERNEL_FUSED_FFN, st, launch_fused(a, L->s.bits, st));
        nblk = w.nblk_fused;
        count_parts = w.nblk_fused;
    } else if (w.use_wide || w.use_union) {
        // decode batch: [router] -> [token groups per expert] -> [up GEMV + mask bits] -> [gate/down on the union of the
        // group's rows]; every selected row is read once per expert group
        const RouterArgs ra = router_args(L, w, base, xh);
        FLOE_LAUNCH(FLOE_KERNEL_ROUTER, st, launch_router(ra, T, st));
        TokenGroup* groups = reinterpret_cast<TokenGroup*>(base + w.groups_off);
        int32_t* n_groups = reinterpret_cast<int32_t*>(base + w.ngroups_off);
        const int n_all = L->n_experts + L->n_shared;
        WideGroup* wide = reinterpret_cast<WideGroup*>(base + w.wgroups_off);
        int32_t* n_wide = reinterpret_cast<int32_t*>(wide + w.wp.max_groups);
        int32_t* order = reinterpret_cast<int32_t*>(base + w.order_off);
        const bool group_here = (w.up_wide || w.up_split) && w.n_tasks <= kOperandGroups;  // by the kernel that prepares the activations
        WideArgs wa{};
        WidePrep prep{};
        if (w.use_wide) {
            prep = WidePrep{reinterpret_cast<uint4*>(partial), count, reinterpret_cast<uint32_t*>(base + w.hmax_off),
                            reinterpret_cast<int2*>(base + w.trows_off), reinterpret_cast<int4*>(base + w.segs_off), w.wp.segments, task_tau, task_weight,
                            reinterpret_cast<float*>(base + w.ptau_off), reinterpret_cast<float*>(base + w.ptau_off) + w.n_tasks};
            wa.groups = wide; wa.n_groups = n_wide; wa.order = order; wa.x = xh; wa.v = v;
            wa.tau = prep.tau; wa.scale = prep.scale; wa.count = count;
            wa.by_task = !w.up_wide && !w.up_split;
            wa.rows = reinterpret_cast<int32_t*>(base + w.urow_off);
            wa.segments = prep.segments;
            wa.hbuf = reinterpret_cast<uint4*>(base + w.hbuf_off);
            wa.hmax = prep.hmax;
            wa.task_rows = prep.task_rows;
            wa.partial = partial;
            wa.xop = prep.xop;
            wa.slots = slots; wa.f = L->s.f; wa.max_groups = w.wp.max_groups; wa.pieces = w.wp.wg_gate;
        }
        if (group_here) {
        } else if (w.use_wide)
            FLOE_HIP(launch_group_tokens(task_expert, w.n_tasks, n_all, w.chunk, groups, n_groups, st, order, w.wp.chunk, wide, n_wide,
                                         static_cast<const DevExpert*>(L->dev_table)));
        else
            FLOE_HIP(launch_group_tokens(task_expert, w.n_tasks, n_all, w.chunk, groups, n_groups, st));
        if (w.up_wide || w.up_split) {
            UpWideArgs u{};
            u.groups = wide; u.n_groups = n_wide; u.order = order; u.x = xh; u.v = v;
            u.mask_words = mask; u.x_frag = base + w.hbuf_off; u.x_sums = base + w.xsum_off;
            u.n_tasks = w.n_tasks; u.d = L->s.d; u.f = L->s.f; u.slots = slots; u.nt = w.wp.nt;
            u.max_groups = w.wp.max_groups; u.est_groups = w.wp.est_groups; u.chunk = w.wp.chunk; u.prep = prep;
            u.task_expert = group_here ? task_expert : nullptr; u.table = static_cast<const DevExpert*>(L->dev_table); u.n_all = n_all;
            FLOE_LAUNCH(FLOE_KERNEL_UP_GEMV, st,
                        w.up_split ? launch_up_split(u, L->s.bits, L->s.group, st) : launch_up_wide(u, L->s.bits, L->s.group, st));
        } else if (batch_mfma)
            FLOE_LAUNCH(FLOE_KERNEL_UP_GEMV, st,
                        launch_up_gemv_grouped(static_cast<const DevExpert*>(L->dev_table), groups, n_groups,
                                               mfma_max_groups(n_all, w.n_tasks), w.chunk, xh, slots, v, task_tau, mask, L->s.d, L->s.f,
                                               L->s.bits, L->s.group, st));
        else
            FLOE_LAUNCH(FLOE_KERNEL_UP_GEMV, st,
                        launch_up_gemv(map, xh, nullptr, v, task_tau, mask, L->s.d, L->s.f, L->s.bits, L->s.group,
                                       w.n_tasks, st));
        if (w.use_wide) {
            if (!w.up_wide && !w.up_split) FLOE_HIP(launch_wide_prepare(prep, wa, mask, w.n_tasks, L->s.d, st));
            FLOE_LAUNCH(FLOE_KERNEL_GATE_DOWN, st, launch_gate_down_wide(wa, w.wp, mask, L->s.d, st));
            FLOE_LAUNCH(FLOE_KERNEL_COMBINE, st, launch_combine_wide(wa, w.wp, L->s.d, T, nullptr, reinterpret_cast<h16*>(y), st));
            if (stats)
                FLOE_HIP(launch_stats(task_expert, count, 0, task_weight, reinterpret_cast<SlotStat*>(stats), w.n_tasks, st));
            return FLOE_OK;
        }
        UnionArgs ua{};
        ua.table = static_cast<const DevExpert*>(L->dev_table);
        ua.groups = groups; ua.n_groups = n_groups; ua.x = xh; ua.v = v; ua.mask_words = mask;
        ua.task_scale = task_weight; ua.count = count; ua.partial = partial;
        ua.slots = slots; ua.f = L->s.f; ua.cap = w.up.cap; ua.nblk = w.up.nblk;
        FLOE_LAUNCH(FLOE_KERNEL_GATE_DOWN, st, launch_gate_down_union(ua, w.up, L->s.d, st));
        nblk = w.up.nblk;
        count_parts = w.up.nblk;
    } else if (mask_ok && !batch_mfma &&
               route_in_place_ok(L->s.d, L->s.bits, L->s.group, L->n_experts, L->top_k, L->n_shared)) {
        // larger batches of shapes without a matrix-core path: [router + up GEMV + mask] -> [compaction + gate/down]
        RouteArgs ro{};
        ro.router_cm = reinterpret_cast<const h16*>(L->router_cm);
        ro.tau = L->tau;
        ro.tau_stride_t = L->tau_stride_t;
        ro.n_experts = L->n_experts; ro.top_k = L->top_k; ro.n_shared = L->n_shared; ro.renormalize = L->renormalize;
        ro.table = static_cast<const DevExpert*>(L->dev_table);
        ro.task_table = task_table;
        ro.task_expert = task_expert; ro.task_weight = task_weight; ro.task_tau = task_tau;
        FLOE_LAUNCH(FLOE_KERNEL_UP_GEMV, st,
                    launch_up_gemv(map, xh, &ro, v, nullptr, mask, L->s.d, L->s.f, L->s.bits, L->s.group,
                                   w.n_tasks, st));
        FLOE_LAUNCH(FLOE_KERNEL_GATE_DOWN, st,
                    launch_gate_down(map, nullptr, L->s.f, xh, v, mask, nullptr, count, task_weight, partial, L->s.d, L->s.f,
                                     w.n_tasks, w.nblk, st));
    } else {
        const RouterArgs ra = router_args(L, w, base, xh);
        FLOE_LAUNCH(FLOE_KERNEL_ROUTER, st, launch_router(ra, T, st));
        // batches: the gate/down workgroups are launched in expert order (tasks that share an expert run side by side
        // and share its rows in the L2)
        TokenGroup* groups = reinterpret_cast<TokenGroup*>(base + w.groups_off);
        int32_t* n_groups = reinterpret_cast<int32_t*>(base + w.ngroups_off);
        // (only where the grouping kernel runs anyway: on its own it costs what the sharing saves)
        int32_t* order = (mask_ok && batch_mfma && w.n_tasks > kExpertOrderTasks) ? reinterpret_cast<int32_t*>(base + w.order_off) : nullptr;
        const int n_all = L->n_experts + L->n_shared;
        const int chunk = mfma_chunk(n_all, w.n_tasks);
        if (order || (mask_ok && batch_mfma))
            FLOE_HIP(launch_group_tokens(task_expert, w.n_tasks, n_all, chunk, groups, n_groups, st, order));
        if (mask_ok && batch_mfma) {
            // decode batch: tokens routed to the same expert share one pass over its codes (matrix cores)
            FLOE_LAUNCH(FLOE_KERNEL_UP_GEMV, st,
                        launch_up_gemv_grouped(static_cast<const DevExpert*>(L->dev_table), groups, n_groups,
                                               mfma_max_groups(n_all, w.n_tasks), chunk, xh, slots, v, task_tau,
                                               mask, L->s.d, L->s.f, L->s.bits, L->s.group, st));
            FLOE_LAUNCH(FLOE_KERNEL_GATE_DOWN, st,
                        launch_gate_down(map, nullptr, L->s.f, xh, v, mask, nullptr, count, task_weight, partial, L->s.d,
                                         L->s.f, w.n_tasks, w.nblk, st, nullptr, order));
        } else if (mask_ok) {
            FLOE_LAUNCH(FLOE_KERNEL_UP_GEMV, st,
                        launch_up_gemv(map, xh, nullptr, v, task_tau, mask, L->s.d, L->s.f, L->s.bits, L->s.group,
                                       w.n_tasks, st));
            FLOE_LAUNCH(FLOE_KERNEL_GATE_DOWN, st,
                        launch_gate_down(map, nullptr, L->s.f, xh, v, mask, nullptr, count, task_weight, partial, L->s.d,
                                         L->s.f, w.n_tasks, w.nblk, st, nullptr, order));
        } else {
            FLOE_LAUNCH(FLOE_KERNEL_UP_GEMV, st,
                        launch_up_gemv(map, xh, nullptr, v, nullptr, nullptr, L->s.d, L->s.f, L->s.bits,
                                       L->s.group, w.n_tasks, st));
            FLOE_LAUNCH(FLOE_KERNEL_SELECT, st, launch_select(v, L->s.f, w.n_tasks, task_tau, idx, count, st));
            FLOE_LAUNCH(FLOE_KERNEL_GATE_DOWN, st,
                        launch_gate_down(map, nullptr, L->s.f, xh, v, nullptr, idx, count, task_weight, partial, L->s.d,
                                         L->s.f, w.n_tasks, w.nblk, st));
        }
    }
    FLOE_LAUNCH(FLOE_KERNEL_COMBINE, st, launch_combine(partial, L->s.d, T, slots, nblk, nullptr, reinterpret_cast<h16*>(y), st));
    if (stats)
        FLOE_HIP(launch_stats(task_expert, count, count_parts, task_weight, reinterpret_cast<SlotStat*>(stats), w.n_tasks, st));
    return FLOE_OK;
}

int floe_moe_layer_decode_offloaded(const floe_layer* L, const floe_offload* o, const floe_half* x, int T, floe_half* y,
                                    floe_slot_stat* stats, void* workspace, size_t workspace_bytes, void* stream) {
    int rc = check_layer(L);
    if (rc) return rc;
    if ((rc = check_T(T))) return rc;
    if (T == 0) return FLOE_OK;
    if (!o || !o->staging || !o->ev_lists_ready || !o->ev_staged || o->capacity_rows <= 0) return FLOE_EINVAL;
    if (!L->dev_table || !L->gd_on_host || !x || !y || !workspace) return FLOE_EINVAL;
    if (!aligned(x, 16) || !aligned(y, 8) || !aligned(workspace, kAlign) || !aligned(o->staging, 16)) return FLOE_EINVAL;
    const LayerWs w = layer_plan(L, T);
    if (workspace_bytes < w.total) return FLOE_EWORKSPACE;
    char* base = static_cast<char*>(workspace);
    DevExpert* task_table = reinterpret_cast<DevExpert*>(base + w.table_off);
    int32_t* task_expert = reinterpret_cast<int32_t*>(base + w.expert_off);
    float* task_weight = reinterpret_cast<float*>(base + w.weight_off);
    int32_t* count = reinterpret_cast<int32_t*>(base + w.count_off);
    float* v = reinterpret_cast<float*>(base + w.v_off);
    int32_t* idx = reinterpret_cast<int32_t*>(base + w.idx_off);
    float* partial = reinterpret_cast<float*>(base + w.partial_off);
    hipStream_t st = (hipStream_t)stream, side = (hipStream_t)o->side_stream;
    const h16* xh = reinterpret_cast<const h16*>(x);
    const int slots = L->top_k + L->n_shared;

    TaskMap map{};
    map.task_table = task_table;
    map.slots = slots;
    if ((rc = layer_lists(L, w, base, xh, T, st))) return rc;
    FLOE_HIP(hipEventRecord((hipEvent_t)o->ev_lists_ready, st));
    FLOE_HIP(hipStreamWaitEvent(side, (hipEvent_t)o->ev_lists_ready, 0));
    FLOE_LAUNCH(FLOE_KERNEL_STAGE, side,
                launch_stage_tasks(task_table, L->s.d, L->s.f, idx, count, o->capacity_rows,
                                   reinterpret_cast<h16*>(o->staging), o->overflow, w.n_tasks, side));
    FLOE_HIP(hipEventRecord((hipEvent_t)o->ev_staged, side));
    FLOE_HIP(hipStreamWaitEvent(st, (hipEvent_t)o->ev_staged, 0));
    FLOE_LAUNCH(FLOE_KERNEL_GATE_DOWN, st,
                launch_gate_down(map, reinterpret_cast<const h16*>(o->staging), o->capacity_rows, xh, v, nullptr, idx,
                                 count, task_weight, partial, L->s.d, L->s.f, w.n_tasks, w.nblk, st));
    FLOE_LAUNCH(FLOE_KERNEL_COMBINE, st,
                launch_combine(partial, L->s.d, T, slots, w.nblk, nullptr, reinterpret_cast<h16*>(y), st));
    if (stats)
        FLOE_HIP(launch_stats(task_expert, count, 0, task_weight, reinterpret_cast<SlotStat*>(stats), w.n_tasks, st, count,
                              o->capacity_rows));
    return FLOE_OK;
}

int floe_moe_layer_prefetch(const floe_layer* L, const floe_prefetch* p, const floe_half* x_cur, int T, void* workspace,
                            size_t workspace_bytes, void* stream) {
    int rc = check_layer(L);
    if (rc) return rc;
    if ((rc = check_T(T))) return rc;
    if (T == 0) return FLOE_OK;
    if (!p || !p->staging || !p->pred_expert || !p->pred_count || !p->row_of || !p->ev_inputs_ready || !p->ev_prefetched ||
        p->capacity_rows <= 0)
        return FLOE_EINVAL;
    if (!L->dev_table || !L->gd_on_host || !x_cur || !workspace) return FLOE_EINVAL;
    if (!aligned(x_cur, 16) || !aligned(workspace, kAlign) || !aligned(p->staging, 16)) return FLOE_EINVAL;
    const LayerWs w = layer_plan(L, T);
    if (workspace_bytes < w.total) return FLOE_EWORKSPACE;
    char* base = static_cast<char*>(workspace);
    hipStream_t st = (hipStream_t)stream, side = (hipStream_t)p->prefetch_stream;
    // everything below runs on the prefetch stream, after whatever produced x_cur on `stream`
    FLOE_HIP(hipEventRecord((hipEvent_t)p->ev_inputs_ready, st));
    FLOE_HIP(hipStreamWaitEvent(side, (hipEvent_t)p->ev_inputs_ready, 0));
    if ((rc = layer_lists(L, w, base, reinterpret_cast<const h16*>(x_cur), T, side))) return rc;
    const DevExpert* task_table = reinterpret_cast<const DevExpert*>(base + w.table_off);
    const int32_t* task_expert = reinterpret_cast<const int32_t*>(base + w.expert_off);
    const int32_t* count = reinterpret_cast<const int32_t*>(base + w.count_off);
    const int32_t* idx = reinterpret_cast<const int32_t*>(base + w.idx_off);
    FLOE_LAUNCH(FLOE_KERNEL_STAGE, side,
                launch_stage_tasks(task_table, L->s.d, L->s.f, idx, count, p->capacity_rows,
                                   reinterpret_cast<h16*>(p->staging), nullptr, w.n_tasks, side));
    FLOE_HIP(launch_rowmap(idx, count, task_expert, L->s.f, p->capacity_rows, p->row_of, p->pred_expert, p->pred_count,
                           w.n_tasks, side));
    FLOE_HIP(hipEventRecord((hipEvent_t)p->ev_prefetched, side));
    return FLOE_OK;
}

int floe_moe_layer_decode_prefetched(const floe_layer* L, const floe_prefetch* p, const floe_miss_path* m,
                                     const floe_half* x, int T, floe_half* y, floe_slot_stat* stats,
                                     floe_prefetch_stat* prefetch_stats, void* workspace, size_t workspace_bytes,
                                     void* stream) {
    static_assert(sizeof(floe_prefetch_stat) == sizeof(PrefetchStat), "prefetch stat record layout");
    int rc = check_layer(L);
    if (rc) return rc;
    if ((rc = check_T(T))) return rc;
    if (T == 0) return FLOE_OK;
    if (!p || !p->staging || !p->pred_expert || !p->pred_count || !p->row_of || !p->ev_prefetched || p->capacity_rows <= 0)
        return FLOE_EINVAL;
    if (!m || !m->ev_lists_ready || !m->ev_staged) return FLOE_EINVAL;
    if (!L->dev_table || !L->gd_on_host || !x || !y || !workspace) return FLOE_EINVAL;
    if (!aligned(x, 16) || !aligned(y, 8) || !aligned(workspace, kAlign) || !aligned(p->staging, 16)) return FLOE_EINVAL;
    const LayerWs w = layer_plan(L, T);
    if (workspace_bytes < w.total) return FLOE_EWORKSPACE;
    char* base = static_cast<char*>(workspace);
    DevExpert* task_table = reinterpret_cast<DevExpert*>(base + w.table_off);
    int32_t* task_expert = reinterpret_cast<int32_t*>(base + w.expert_off);
    float* task_weight = reinterpret_cast<float*>(base + w.weight_off);
    int32_t* count = reinterpret_cast<int32_t*>(base + w.count_off);
    float* v = reinterpret_cast<float*>(base + w.v_off);
    int32_t* idx = reinterpret_cast<int32_t*>(base + w.idx_off);
    int32_t* rows = reinterpret_cast<int32_t*>(base + w.rows_off);
    int32_t* miss_idx = reinterpret_cast<int32_t*>(base + w.missidx_off);
    int32_t* miss_rows = reinterpret_cast<int32_t*>(base + w.missrows_off);
    int32_t* miss_count = reinterpret_cast<int32_t*>(base + w.misscount_off);
    float* partial = reinterpret_cast<float*>(base + w.partial_off);
    hipStream_t st = (hipStream_t)stream, side = (hipStream_t)m->miss_stream;
    const h16* xh = reinterpret_cast<const h16*>(x);
    const int slots = L->top_k + L->n_shared;
    TaskMap map{};
    map.task_table = task_table;
    map.slots = slots;

    if ((rc = layer_lists(L, w, base, xh, T, st))) return rc;
    FLOE_HIP(hipStreamWaitEvent(st, (hipEvent_t)p->ev_prefetched, 0));
    FLOE_HIP(launch_match_rows(idx, count, task_expert, L->s.f, slots, p->capacity_rows, p->row_of, p->pred_expert,
                               p->pred_count, rows, miss_idx, miss_rows, miss_count, m->overflow,
                               reinterpret_cast<PrefetchStat*>(prefetch_stats), w.n_tasks, st));
    FLOE_HIP(hipEventRecord((hipEvent_t)m->ev_lists_ready, st));
    FLOE_HIP(hipStreamWaitEvent(side, (hipEvent_t)m->ev_lists_ready, 0));
    FLOE_LAUNCH(FLOE_KERNEL_STAGE, side,
                launch_stage_tasks(task_table, L->s.d, L->s.f, miss_idx, miss_count, p->capacity_rows,
                                   reinterpret_cast<h16*>(p->staging), nullptr, w.n_tasks, side, miss_rows));
    FLOE_HIP(hipEventRecord((hipEvent_t)m->ev_staged, side));
    FLOE_HIP(hipStreamWaitEvent(st, (hipEvent_t)m->ev_staged, 0));
    FLOE_LAUNCH(FLOE_KERNEL_GATE_DOWN, st,
                launch_gate_down(map, reinterpret_cast<const h16*>(p->staging), p->capacity_rows, xh, v, nullptr, idx, count,
                                 task_weight, partial, L->s.d, L->s.f, w.n_tasks, w.nblk, st, rows));
    FLOE_LAUNCH(FLOE_KERNEL_COMBINE, st,
                launch_combine(partial, L->s.d, T, slots, w.nblk, nullptr, reinterpret_cast<h16*>(y), st));
    if (stats)
        FLOE_HIP(launch_stats(task_expert, count, 0, task_weight, reinterpret_cast<SlotStat*>(stats), w.n_tasks, st, miss_count));
    return FLOE_OK;
}

int floe_channel_cache_load(const floe_layer* L, const floe_channel_cache* c, int expert, const int32_t* idx,
                            const int32_t* count, int first_row, int max_rows, void* stream) {
    int rc = check_layer(L);
    if (rc) return rc;
    if (!c || !c->pool || !c->row_of || !idx || !count || !L->dev_table || !L->gd_on_host) return FLOE_EINVAL;
    if (expert < 0 || expert >= L->n_experts + L->n_shared || first_row < 0 || max_rows < 0) return FLOE_EINVAL;
    if ((long long)first_row + max_rows > c->resident_rows) return FLOE_EINVAL;  // the resident part of the pool ends there
    if (!aligned(c->pool, 16)) return FLOE_EINVAL;
    FLOE_LAUNCH(FLOE_KERNEL_STAGE, (hipStream_t)stream,
                launch_cache_load(static_cast<const DevExpert*>(L->dev_table), expert, L->s.d, L->s.f, idx, count, first_row,
                                  max_rows, reinterpret_cast<h16*>(c->pool), c->row_of, (hipStream_t)stream));
    return FLOE_OK;
}

int floe_moe_layer_decode_cached(const floe_layer* L, const floe_channel_cache* c, const floe_miss_path* m,
                                 const floe_half* x, int T, floe_half* y, floe_slot_stat* stats,
                                 floe_prefetch_stat* cache_stats, void* workspace, size_t workspace_bytes, void* stream) {
    int rc = check_layer(L);
    if (rc) return rc;
    if ((rc = check_T(T))) return rc;
    if (T == 0) return FLOE_OK;
    if (!c || !c->pool || !c->row_of || c->capacity_rows <= 0 || c->resident_rows < 0) return FLOE_EINVAL;
    if (!m || !m->ev_lists_ready || !m->ev_staged) return FLOE_EINVAL;
    if (!L->dev_table || !L->gd_on_host || !x || !y || !workspace) return FLOE_EINVAL;
    if (!aligned(x, 16) || !aligned(y, 8) || !aligned(workspace, kAlign) || !aligned(c->pool, 16)) return FLOE_EINVAL;
    const LayerWs w = layer_plan(L, T);
    if (workspace_bytes < w.total) return FLOE_EWORKSPACE;
    char* base = static_cast<char*>(workspace);
    DevExpert* task_table = reinterpret_cast<DevExpert*>(base + w.table_off);
    int32_t* task_expert = reinterpret_cast<int32_t*>(base + w.expert_off);
    float* task_weight = reinterpret_cast<float*>(base + w.weight_off);
    int32_t* count = reinterpret_cast<int32_t*>(base + w.count_off);
    float* v = reinterpret_cast<float*>(base + w.v_off);
    int32_t* idx = reinterpret_cast<int32_t*>(base + w.idx_off);
    int32_t* rows = reinterpret_cast<int32_t*>(base + w.rows_off);
    int32_t* miss_idx = reinterpret_cast<int32_t*>(base + w.missidx_off);
    int32_t* miss_rows = reinterpret_cast<int32_t*>(base + w.missrows_off);
    int32_t* miss_count = reinterpret_cast<int32_t*>(base + w.misscount_off);
    float* partial = reinterpret_cast<float*>(base + w.partial_off);
    hipStream_t st = (hipStream_t)stream, side = (hipStream_t)m->miss_stream;
    const h16* xh = reinterpret_cast<const h16*>(x);
    const int slots = L->top_k + L->n_shared;
    TaskMap map{};
    map.task_table = task_table;
    map.slots = slots;

    // lists on `stream`; where each selected channel sits (resident row, or a fresh row of the task's slab) and which
    // ones are missing; the misses cross the bus on the miss stream; gate/down on the pool's rows
    if ((rc = layer_lists(L, w, base, xh, T, st))) return rc;
    FLOE_HIP(launch_match_rows(idx, count, task_expert, L->s.f, slots, c->capacity_rows, nullptr, nullptr, nullptr, rows,
                               miss_idx, miss_rows, miss_count, m->overflow, reinterpret_cast<PrefetchStat*>(cache_stats),
                               w.n_tasks, st, c->row_of, c->resident_rows));
    FLOE_HIP(hipEventRecord((hipEvent_t)m->ev_lists_ready, st));
    FLOE_HIP(hipStreamWaitEvent(side, (hipEvent_t)m->ev_lists_ready, 0));
    FLOE_LAUNCH(FLOE_KERNEL_STAGE, side,
                launch_stage_tasks(task_table, L->s.d, L->s.f, miss_idx, miss_count, c->capacity_rows,
                                   reinterpret_cast<h16*>(c->pool), nullptr, w.n_tasks, side, miss_rows));
    FLOE_HIP(hipEventRecord((hipEvent_t)m->ev_staged, side));
    FLOE_HIP(hipStreamWaitEvent(st, (hipEvent_t)m->ev_staged, 0));
    FLOE_LAUNCH(FLOE_KERNEL_GATE_DOWN, st,
                launch_gate_down(map, reinterpret_cast<const h16*>(c->pool), c->capacity_rows, xh, v, nullptr, idx, count,
                                 task_weight, partial, L->s.d, L->s.f, w.n_tasks, w.nblk, st, rows));
    FLOE_LAUNCH(FLOE_KERNEL_COMBINE, st,
                launch_combine(partial, L->s.d, T, slots, w.nblk, nullptr, reinterpret_cast<h16*>(y), st));
    if (stats)
        FLOE_HIP(launch_stats(task_expert, count, 0, task_weight, reinterpret_cast<SlotStat*>(stats), w.n_tasks, st, miss_count,
                              c->capacity_rows));
    return FLOE_OK;
}

int floe_stage_channels(const floe_half* host_gd, int d, int f, const int32_t* idx, const int32_t* count, int capacity_rows,
                        floe_half* hbm_dst, int32_t* overflow, void* side_stream, void* done) {
    if (!host_gd || !idx || !count || !hbm_dst) return FLOE_EINVAL;
    if (d <= 0 || f <= 0 || capacity_rows < 0) return FLOE_EINVAL;
    if (d % 4 != 0) return FLOE_ESHAPE;
    if (!aligned(host_gd, 16) || !aligned(hbm_dst, 16)) return FLOE_EINVAL;
    // the device view of the pinned matrix; callers stage from the same few matrices over and over
    static thread_local const floe_half* last_host = nullptr;
    static thread_local void* last_dev = nullptr;
    if (host_gd != last_host) {
        void* dev_view = nullptr;
        FLOE_HIP(hipHostGetDevicePointer(&dev_view, const_cast<floe_half*>(host_gd), 0));
        last_host = host_gd;
        last_dev = dev_view;
    }
    void* dev_view = last_dev;
    hipStream_t st = (hipStream_t)side_stream;
    FLOE_LAUNCH(FLOE_KERNEL_STAGE, st, launch_stage(static_cast<const h16*>(dev_view), d, f, idx, count, capacity_rows,
                          reinterpret_cast<h16*>(hbm_dst), overflow, st));
    if (done) FLOE_HIP(hipEventRecord((hipEvent_t)done, st));
    return FLOE_OK;
}

}  // extern "C"

namespace floe {

bool layer_fits(const floe_layer* L, int T, size_t bytes) { return check_layer(L) != FLOE_OK || layer_fit(L, T, bytes).total <= bytes; }

}  // namespace floe
