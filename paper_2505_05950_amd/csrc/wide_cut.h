// How the work of wide token groups is cut into pieces, and where the gate kernel puts what a piece hands to the down kernel
// (wide_layout.h): whole numbers only, for the kernels and for a host program alike.
#pragma once

#include <math.h>
#include <stddef.h>
#include <stdint.h>

#ifdef __HIP__
#define FLOE_BOTH __host__ __device__ __forceinline__
#else
#define FLOE_BOTH inline
#endif

namespace floe {

// floor(a * b / c) and floor((a * b - 1) / c); in 32 bits where the product fits (a 64-bit quotient is 200 instructions of a kernel's first
// microseconds)
FLOE_BOTH int scaled(int a, int b, int less, int c) {
    if ((uint32_t)a < (1u << 21) && (uint32_t)b < (1u << 11)) return (int)(((uint32_t)a * (uint32_t)b - (uint32_t)less) / (uint32_t)c);
    return (int)(((long long)a * b - less) / c);
}
// piece w of W equal pieces starts at pair floor(total * w / W)
FLOE_BOTH int wide_cut(int total, int W, int w) { return scaled(total, w, 0, W); }
// pair p belongs to piece ((p + 1) * W - 1) / total
FLOE_BOTH int wide_owner(int total, int W, int p) { return scaled(p + 1, W, 1, total); }
// n / d as a whole number from 1 / d, for n up to a few hundred thousand and quotients up to a few hundred: taken half a unit above a
// whole number, so that rounding cannot matter
FLOE_BOTH int small_quotient(int n, float inverse) { return (int)(((float)n + 0.5f) * inverse); }

// ---- gate: the channels of a group are units of eight, each of the group's weight
FLOE_BOTH int wide_piece_units(int f) { return (f + 7) >> 3; }
// The share of a group's channels that its tokens selected, in 2^-20, as far as the part of them goes that a wave has seen.
constexpr float kWideShareOne = 1048576.0f;
FLOE_BOTH int wide_selected_share(int selected, int seen) { return (int)((float)selected * (kWideShareOne / (float)seen)); }
// What eight channels of a group of n tokens cost, 1 to 32: the share of rows that somebody selected, if each token takes a channel with the
// group's own probability.
FLOE_BOTH int wide_weight(int n, int share) {
    const float rest = fmaxf(1.0f - (float)share * (1.0f / kWideShareOne), 0.0f);  // of a token's channels
#ifdef __HIP_DEVICE_COMPILE__
    const float nobody = __builtin_amdgcn_exp2f((float)n * __builtin_amdgcn_logf(rest));
#else
    const float nobody = exp2f((float)n * log2f(rest));
#endif
    const int w = 32 - (int)(32.0f * nobody);
    return w < 1 ? 1 : w;
}
// Pieces end where groups end (wide_share) unless the largest then has 96 rows more than an equal cut's: a second segment costs a workgroup
// about as much, at any d.  Layer calls, whole pieces / equal ones, us, by the rows that whole ones have more: INT4 g64 d 2048 f 768 (128 experts
// top-8) 29 259 / 267, 77 248 / 253, 62 236 / 233, 490 394 / 358; INT3 d 2048 f 1408 (64 + 2) 68 218 / 222, 93 239 / 239; d 4096 f 1024 (100) 102
// 580 / 589, 120 466 / 461; d 1024 f 1024 (200) 55 165 / 169, 104 200 / 193, 336 264 / 250; d 5120 f 1536 (160 + 2) 129 726 / 722, 570 1323 / 1278.
FLOE_BOTH int wide_most_limit(int most) { return most + 96 * 32 / 8; }
FLOE_BOTH int wide_next_most(int most) { return most + (most >> 5) + 4; }
// Pieces of a group, of at most `most` each (per_most: its reciprocal), and never more than it has units: a piece without channels writes no
// segment, and the down kernel takes a group's first segment for the start of its slots.  (Few tokens' worth of groups in a launch sized
// for many, as where a router sends a whole batch to one expert, leaves `most` below a unit's weight.)
FLOE_BOTH int wide_share(int weight, int units, int most, float per_most) {
    const int k = small_quotient(weight * units + most - 1, per_most);
    return k < units ? k : units;
}
struct WideUnits {
    int begin, end;
};
// piece `at` of the k that a group is cut into (long pieces end at multiples of 32 channels: where every channel is selected, as in groups of
// a hundred tokens, no pair is padded)
FLOE_BOTH WideUnits wide_units_of_share(int units, int k, int at) {
    const int step = units >= 64 * k ? 4 : 1, steps = (units + step - 1) / step;
    const int end = steps * (at + 1) / k * step;
    return WideUnits{steps * at / k * step, end < units ? end : units};
}
// the same for a piece that spans [from, to) of a sequence in which the group lies from 0 on: a unit belongs to the piece that holds the start
// of its share
FLOE_BOTH WideUnits wide_units_of_span(int units, int weight, int from, int to) {
    const int begin = from + weight - 1, end = to + weight - 1;
    const int last = (end > 0 ? end : 0) / weight;
    return WideUnits{(begin > 0 ? begin : 0) / weight, last < units ? last : units};
}

// ---- slots.  first: the first piece that has a segment of the group
FLOE_BOTH int wide_slot(int first_unit, int piece, int first) { return (first_unit >> 2) + piece - first; }
FLOE_BOTH size_t wide_row_slot(int g, int first, int pmax) { return (size_t)g * pmax + first + 2 * g; }
// h of a group lies in [pair slot][token tile][half of the pair's rows][lane], the group's own tiles only, from this vector on
FLOE_BOTH size_t wide_h_first(int tile, int g, int first, int pmax, int nt) { return ((size_t)tile * pmax + (size_t)nt * (first + 2 * g)) * 128; }
// what that takes for `pieces` workgroups and up to max_groups groups of nt token tiles, h_tiles tiles together
FLOE_BOTH size_t wide_row_slots(int max_groups, int pmax, int pieces) { return (size_t)max_groups * (pmax + 2) + pieces; }
FLOE_BOTH size_t wide_h_vecs(int h_tiles, int pmax, int nt, int max_groups, int pieces) {
    return ((size_t)h_tiles * pmax + (size_t)nt * (pieces + 2 * max_groups)) * 128;
}

}  // namespace floe
