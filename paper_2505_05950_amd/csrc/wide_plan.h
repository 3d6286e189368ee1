// Host arithmetic of the plans for token groups: how many groups there will be, how many there can be, and how large they are made.
// Plain C++, so that a host program can walk it.
#pragma once

#include <math.h>

namespace floe {

// Expected number of groups of `chunk` tokens when each of T tokens goes to top_k of n_experts experts uniformly.  Per expert
// E[ceil(X / chunk)] = sum over k >= 0 of P(X > k * chunk), X binomial, by its normal approximation.  Terms further
// than 8.5 deviations from the mean are 1 and 0 to the last bit of a double: every layer call plans, so only the others are formed.
inline double expected_token_groups(int n_experts, int T, int top_k, int chunk) {
    if (n_experts <= 0 || top_k <= 0) return 0.0;
    const double pr = (double)top_k / n_experts, mu = T * pr, sd = sqrt(T * pr * (1.0 - pr)) + 1e-9;
    const double lo = (mu - 8.5 * sd - 0.5) / chunk, hi = mu + 8.5 * sd;
    int k = lo > 0.0 ? (int)lo : 0;
    double per = k;
    for (; k * chunk < T && k * chunk < hi; ++k) per += 0.5 * erfc(((double)k * chunk + 0.5 - mu) / (sd * 1.4142135623730951));
    return per * n_experts;
}

// Token tiles per group: the fewest expected reads of the experts' rows, weighed by what a read costs.  Calls with each number of
// tiles forced, us: 8 experts d 4096 f 14336 INT2 at 85 %, 56 tokens 410 (one tile) 390 394 404 405 416 (ten), 72 tokens 503 419 421 430 432
// 445, 512 tokens 2611 1663 1342 1126 799 740; 64 + 2 experts d 2048 f 1408 INT3 g32, 148 tokens 272 257 259 265 319 355.  Over 255 calls
// the choice costs 4 % on average against the best of the six.  It misses most where one number holds a group and a smaller one its
// halves: 8 experts, 320 tokens 718 (five, taken) 608 (ten); one expert of the same size, 160 tokens 169 (five) 198 (ten, taken), 200
// tokens 240 (five, taken) 203 (ten).
inline int wide_tiles_for(int T, int n_experts, int top_k, int n_shared, double& groups) {
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

// the most groups that n_tasks tasks of n_all experts can form, whatever the routing
inline int wide_max_groups(int n_all, int n_tasks, int nt) { return (n_all < n_tasks ? n_all : n_tasks) + n_tasks / (16 * nt); }
// Entries of the segment table, which the down kernel holds in LDS (ten bytes each): a piece of the gate kernel and a group each, at most.  A
// layer call has up to 1087 experts, 64 * 4096 tasks and 256 pieces.  Four token tiles per group: 1087 + 262144 / 64 + 256.  More tiles
// make fewer groups, and fewer tiles are not chosen for so many tasks: N tasks form N / (16 nt) groups at least and, ten tiles each, 1087 + N / 160
// at most, so that ten tiles have the better score from 171,000 tasks on against three (4903 entries), 92,000 against two and 39,000 against one.
// (Reached: 4435.)
constexpr int kWideMaxSegments = 5440;

}  // namespace floe
