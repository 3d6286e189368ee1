// Host side of the fused small-batch kernel: block-size choice and dispatch on the bit width.
#include "launch.h"

#include <atomic>

namespace floe {

int num_cus() {
    constexpr int kMaxDevices = 64, kDefault = 256;
    static std::atomic<int> cached[kMaxDevices];  // 0 = not asked yet
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return kDefault;
    int n = cached[dev].load(std::memory_order_relaxed);
    if (n > 0) return n;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = kDefault;
    cached[dev].store(n, std::memory_order_relaxed);
    return n;
}

static std::atomic<int> g_fused_tasks{0};
int fused_tasks_tuned() { return g_fused_tasks.load(std::memory_order_relaxed); }
void set_fused_tasks_tuned(int n) { g_fused_tasks.store(n > 0 ? n : 0, std::memory_order_relaxed); }

hipError_t launch_fused_int2(const FusedArgs& a, hipStream_t stream);
hipError_t launch_fused_int3(const FusedArgs& a, hipStream_t stream);
hipError_t launch_fused_int4(const FusedArgs& a, hipStream_t stream);
hipError_t launch_fused_ahead_int2(const FusedArgs& a, hipStream_t stream);
hipError_t launch_fused_ahead_int3(const FusedArgs& a, hipStream_t stream);
hipError_t launch_fused_ahead_int4(const FusedArgs& a, hipStream_t stream);
hipError_t launch_fused_between_int2(const FusedArgs& a, hipStream_t stream);
hipError_t launch_fused_between_int3(const FusedArgs& a, hipStream_t stream);
hipError_t launch_fused_between_int4(const FusedArgs& a, hipStream_t stream);

int fused_blocks(int d, int f, int passes) {
    const int ch = fused_producers * passes * (64 / fused_lanes(d));
    return (f + ch - 1) / ch;
}

// Passes per producer wave such that the launch is about one workgroup per compute unit, all of them with the same
// number of channels: every round of workgroups pays the kernel's prologue, the start of its streams and its tail again,
// and a round that is not full leaves compute units idle.  0 = do not fuse.
int fused_passes(int d, int f, int bits, int n_tasks, int max_tasks) {
    if (n_tasks <= 0 || n_tasks > max_tasks || n_tasks > kFusedMaxTasks || f <= 0) return 0;
    const int unit = fused_producers * (64 / fused_lanes(d));  // channels of one pass of all producers
    const int cus = num_cus() * fused_wgs_per_cu;
    int want_blocks = cus / n_tasks;  // rounded down: a few workgroups more than compute units cost a whole second round
    if (want_blocks < 1) want_blocks = 1;
    const int per_block = (f + want_blocks - 1) / want_blocks;
    int passes = (per_block + unit - 1) / unit;
    if (passes <= kFusedMinPasses) {
        passes = kFusedMinPasses;
    } else if (bits == 2) {  // staged codes: whole rounds of the ring
        const int depth = fused_depth(d, bits);
        passes = (passes + depth - 1) / depth * depth;
    }
    if (passes > kFusedMaxPasses) passes = bits == 2 ? kFusedMaxPasses / fused_depth(d, bits) * fused_depth(d, bits) : kFusedMaxPasses;
    return (long long)fused_blocks(d, f, passes) * n_tasks <= kFusedMaxWorkgroups ? passes : 0;
}

// Whether a batch at a width between the powers of two is better off in the fused kernel than in the separate ones.  What counts is how
// many channel passes its producers do one after another (a pass 0.35 to 0.45 us, whatever the selection is): a launch that is one
// even round does n_tasks f / (1024 producers x channels per pass).  Calls fused / one-token / wide kernels, us, at sparsities 60, 80, 90, 95 %:
//   few passes: the fused kernel saves launches and overlaps the two streams
//     INT4 g64 d 2560 f 8000, 4 experts top-2, 3 tokens (47 passes)        45/59/77  32/44/70  28/37/64  27/31/62
//     INT2 g64 d 3072 f 8000, 8 experts, 10 tokens (156)                   0.58 0.59 0.65 0.79 times the one-token kernels
//     INT4 g128 d 2560 f 8000, 8 experts, 16 tokens (250)                  0.67 0.74 0.88 1.08
//   a launch of a second round, or one that leaves so many compute units idle that it takes a quarter longer: not that
//     INT4 g64 d 2560 f 2048, 48 + 2 experts top-6, 18 tokens (512 in two rounds, 288 if it were even)  1.49 1.77 2.33 2.83
//     INT3 g32 d 1536 f 2048, the same (256, even 144)                     0.98 1.04 1.28 1.40
//     just inside: INT4 g64 d 2560 f 2048, 12 tokens (256, even 192)       0.81 0.84 1.04 1.23
//   many passes, where tokens are enough for the wide kernels by their own line: those, but for INT3, whose v the matrix cores form
//   less accurately (1e-5 against 8e-8 here)
//     one expert INT2 g64 d 2560 f 14336, 16 tokens (224 passes)           98/162/67  91/116/67  88/94/65  87/79/63
//     one expert INT4 g64 d 3072 f 14336, 16 tokens (224)                  110/171/69 at 60 %, 91/89/60 at 95 %
//     layers, which reach that line with two or three experts only, break even later: INT4 g64 d 2560 f 8000, 8 experts, 16 tokens (250)
//     0.95 0.87 1.02 1.17 times the wide kernels, 12 (188) 0.94 0.80 0.91 1.01; INT2 f 12000, 16 experts, 16 tokens (375) 0.83 0.75 0.84 1.00
bool fused_between_pays(int d, int f, int bits, int group, int n_all, int n_tasks, int slots, int passes) {
    const int cus = num_cus() * fused_wgs_per_cu;
    if ((long long)fused_blocks(d, f, passes) * n_tasks > cus) return false;  // a second round
    const double even = (double)n_tasks * f / ((double)cus * fused_producers * (64 / fused_lanes(d)));
    if (passes > kFusedMinPasses && passes > 1.25 * even + 20.0) return false;
    const bool wide = union_mode() == 0 && bits != 3 && n_tasks >= 2 * slots && up_wide_shape(d, f, bits, group) && mask_words_per_task(f) <= kWideMaxMaskWords &&
                      union_kernels_for(n_all, n_tasks, d, f, bits, group) == 1;
    if (!wide) return true;
    return passes < (n_all == 1 ? (bits == 2 ? 170 : 105) : (bits == 2 ? 300 : 200));
}

// Whether d 4096 takes the kernels whose consumers are one entry ahead: with few passes per producer the queues are short, and the code stream
// that the producers of those kernels keep in flight stands in the way of the first chunks.  us, without / with, d 4096 f 14336 g64, 8 experts
// top-2, sparsities 60, 75, 90 %:
//   INT2   1 token (28 passes) 41.9 / 42.4  30.8 / 31.9  22.7 / 23.7     4 (112) 136 / 136  100 / 99  51.2 / 51.8    8 (224) 234 / 225  166 / 165  97.6 / 98.6
//         16 (448) 372 / 313  240 / 238  168 / 168
//   INT4   1 (28) 44.9 / 44.8  33.9 / 34.0  24.7 / 25.8    4 (112) 141 / 142  108 / 111  75 / 65    8 (224) 237 / 238  182 / 182  137 / 112
//         16 (448) 342 / 346  286 / 264  235 / 186
//   INT3   1 (28) 53.2 / 52.8  38.6 / 39.1  27.8 / 26.3    4 (112) 146 / 146  110 / 112  76 / 66    8 (224) 231 / 234  180 / 182  137 / 111
//         16 (448) 356 / 350  299 / 271  247 / 194   groups of 32: 8 240 / 244  186 / 187  140 / 111    16 365 / 363  303 / 277  254 / 194
// With many experts and more than 32 tasks it costs up to a tenth at 60 % and saves a fifth at 90 %: 32 tokens top-2 of 16, INT4 f 4894 (306) 271 / 294
// 219 / 219  174 / 137, INT3 f 4894 275 / 288  213 / 206  176 / 142, f 7000 (448) 370 / 401  297 / 287  245 / 196; of 24, INT4 f 4000 258 / 274
// 198 / 206  151 / 123.  Producers that do not wait for each other's rows let the tasks of an expert drift apart, and they find less of each
// other's rows in the L2 (INT4 f 4894 at 60 %: 7.8 / 6.0 million hits, 1.84 / 2.07 GB from HBM).
static bool fused_ahead_pays(int bits, int passes) { return passes >= (bits == 2 ? 300 : 160); }

hipError_t launch_fused(const FusedArgs& a, int bits, hipStream_t stream) {
    if ((a.d & (a.d - 1)) != 0) {
        switch (bits) {
            case 2: return launch_fused_between_int2(a, stream);
            case 3: return launch_fused_between_int3(a, stream);
            case 4: return launch_fused_between_int4(a, stream);
            default: return hipErrorInvalidValue;
        }
    }
    if (!fused_always_ahead(a.d) && fused_ahead_pays(bits, a.passes)) {
        switch (bits) {
            case 2: return launch_fused_ahead_int2(a, stream);
            case 3: return launch_fused_ahead_int3(a, stream);
            case 4: return launch_fused_ahead_int4(a, stream);
            default: return hipErrorInvalidValue;
        }
    }
    switch (bits) {
        case 2: return launch_fused_int2(a, stream);
        case 3: return launch_fused_int3(a, stream);
        case 4: return launch_fused_int4(a, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace floe
