// Walks the cut of wide token groups and its slots as the gate kernel does, then as the down kernel does, over routings from even to
// collapsed, and reports the first place where the two differ (see test_wide_cut.py).
#include <math.h>
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <vector>

#include "wide_cut.h"
#include "wide_plan.h"

using namespace floe;

struct Group {
    int n, tile;
};
struct Segment {
    int pairs = 0, slot = 0, g = 0, first = 0;
};
struct Written {  // who wrote a slot
    int g = -1, index = 0;
};

static unsigned g_seed = 1;
static unsigned rnd() { return g_seed = g_seed * 1664525u + 1013904223u; }

#define CHECK(c, ...)                                                                                                             \
    do {                                                                                                                          \
        if (!(c)) {                                                                                                               \
            printf("groups %d (n of the first %d) f %d workgroups %d keep %d: ", (int)groups.size(), groups[0].n, f, W, keep);     \
            printf(__VA_ARGS__);                                                                                                  \
            printf("\n");                                                                                                         \
            exit(1);                                                                                                              \
        }                                                                                                                         \
    } while (0)

// keep: of 100 channels the ones that a token selects
static void walk(const std::vector<Group>& groups, int max_groups, int h_tiles, int nt, int f, int W, int keep) {
    const int ng = (int)groups.size(), units = wide_piece_units(f), pmax = (f + 31) / 32;
    std::vector<std::vector<char>> chosen(ng, std::vector<char>(f));  // by somebody
    std::vector<int> weight(ng);
    for (int g = 0; g < ng; ++g) {
        const double somebody = 1.0 - pow(1.0 - 0.01 * keep, groups[g].n);
        for (auto& b : chosen[g]) b = (rnd() >> 8) * 0x1p-24 < somebody;
        weight[g] = wide_weight(groups[g].n, wide_selected_share((int)(0.01 * keep * groups[g].n * f), groups[g].n * f));
        CHECK(weight[g] >= 1 && weight[g] <= 32 && fabs(weight[g] - 32.0 * somebody) <= 1.01 + 32.0 / f, "weight %d of group %d", weight[g], g);
    }
    std::vector<Written> rows(wide_row_slots(max_groups, pmax, W)), h(wide_h_vecs(h_tiles, pmax, nt, max_groups, W) / 128);
    std::vector<Segment> table(W + max_groups);
    std::vector<std::vector<int>> list(ng);  // what the down kernel should meet: pairs of a group, in order
    std::vector<int> unit_seen(ng, 0);
    // ---- gate
    int total = 0;
    for (int g = 0; g < ng; ++g) total += weight[g] * units;
    bool whole = ng <= std::min(W, 256);
    int most = std::max((total + W - 1) / W, 1);
    const int limit = wide_most_limit(most);
    while (whole) {
        int sum = 0;
        for (int g = 0; g < ng; ++g) sum += wide_share(weight[g], units, most, 1.0f / (float)most);
        if (sum <= W) break;
        most = wide_next_most(most);
        whole = most <= limit;
    }
    std::vector<int> starts(ng + 1, 0);  // in pieces, or in weighted units
    auto share = [&](int g) { return starts[g + 1] - starts[g]; };
    for (int g = 0; g < ng; ++g)
        starts[g + 1] = starts[g] + (whole ? wide_share(weight[g], units, most, 1.0f / (float)most) : weight[g] * units);
    long rows_all = 0, rows_most = 0;
    for (int piece = 0; piece < W; ++piece) {
        long rows_here = 0;
        int pos = whole ? piece : wide_cut(total, W, piece);
        const int end = whole ? piece + 1 : wide_cut(total, W, piece + 1);
        while (pos < end) {
            const int g = (int)(std::upper_bound(starts.begin(), starts.end(), pos) - starts.begin()) - 1, base = starts[g];
            if (g == ng) break;
            WideUnits u;
            int first;
            if (whole) {
                u = wide_units_of_share(units, share(g), pos - base);
                first = base;
                pos = end;
            } else {
                u = wide_units_of_span(units, weight[g], pos - base, end - base);
                first = wide_owner(total, W, base);
                pos = base + share(g);
            }
            CHECK(!whole || u.begin < u.end, "piece %d of group %d is empty", piece - first, g);
            if (u.end <= u.begin) continue;
            CHECK(u.begin == unit_seen[g], "group %d: unit %d behind %d", g, u.begin, unit_seen[g]);
            unit_seen[g] = u.end;
            int count = 0;
            for (int c = 8 * u.begin; c < std::min(8 * u.end, f); ++c) count += chosen[g][c];
            rows_here += count;
            const int pairs = (count + 31) / 32, slot = wide_slot(u.begin, piece, first), tiles = (groups[g].n + 15) / 16;
            Segment& s = table[piece + g];
            CHECK(s.pairs == 0 && s.first == 0, "segment %d is written twice", piece + g);
            s = Segment{pairs, slot, g, u.begin == 0};
            for (int p = 0; p < pairs; ++p) {
                const int index = (int)list[g].size();
                list[g].push_back(index);
                const size_t r = wide_row_slot(g, first, pmax) + slot + p, v = wide_h_first(groups[g].tile, g, first, pmax, nt) / 128 + (size_t)(slot + p) * tiles;
                CHECK(r < rows.size() && rows[r].g < 0, "row slot %zu of group %d is taken or outside", r, g);
                rows[r] = Written{g, index};
                for (int t = 0; t < tiles; ++t) {
                    CHECK(v + t < h.size() && h[v + t].g < 0, "h of group %d, pair %d is taken or outside", g, index);
                    h[v + t] = Written{g, index * tiles + t};
                }
            }
        }
        rows_all += rows_here;
        rows_most = std::max(rows_most, rows_here);
    }
    // (96 rows more than an even cut, whole units or 32 channels, and what the weights' rounding makes of it)
    CHECK(ng > 300 || (double)(rows_most - 96 - 32) * W <= 1.25 * rows_all, "the largest piece has %ld rows of %ld", rows_most, rows_all);
    for (int g = 0; g < ng; ++g) CHECK(unit_seen[g] == units, "group %d ends at unit %d of %d", g, unit_seen[g], units);
    // ---- down
    std::vector<int> first_seg(ng, -1), met(ng, 0);
    int before = -1;
    for (int i = 0; i < W + ng; ++i)
        if (table[i].first) {
            CHECK(first_seg[table[i].g] < 0 && table[i].g == before + 1, "group %d begins out of turn", table[i].g);
            first_seg[before = table[i].g] = i;
        }
    CHECK(before == ng - 1, "group %d has no first segment", before + 1);
    for (int i = 0; i < W + ng; ++i) {
        const int g = table[i].g, tiles = (groups[g].n + 15) / 16;
        for (int p = 0; p < table[i].pairs; ++p) {
            const size_t r = wide_row_slot(g, first_seg[g] - g, pmax) + table[i].slot + p;
            const size_t v = wide_h_first(groups[g].tile, g, first_seg[g] - g, pmax, nt) / 128 + (size_t)(table[i].slot + p) * tiles;
            CHECK(r < rows.size() && rows[r].g == g && rows[r].index == met[g], "row ids of group %d, pair %d are read from another place", g, met[g]);
            for (int t = 0; t < tiles; ++t)
                CHECK(v + t < h.size() && h[v + t].g == g && h[v + t].index == met[g] * tiles + t, "h of group %d, pair %d is read from another place", g, met[g]);
            ++met[g];
        }
    }
    for (int g = 0; g < ng; ++g) CHECK(met[g] == (int)list[g].size(), "group %d: %d of %d pairs are met", g, met[g], (int)list[g].size());
}

// The segment table holds what any layer that the argument checks accept can ask for: up to 1024 routed experts, 64 slots, 4096 tokens.
static int plans() {
    int most = 0;
    double groups;
    for (const int experts : {1024, 1023, 960, 700, 300, 64, 0})
        for (int slots = 1; slots <= 64; slots += slots < 61 ? 4 : 1)
            for (int top_k = 0; top_k <= slots && top_k <= experts; ++top_k)
                for (int T = 1; T <= 4096; T += slots > 60 ? 3 : 45) {
                    const int shared = slots - top_k, nt = wide_tiles_for(T, experts, top_k, shared, groups);
                    const int entries = wide_max_groups(experts + shared, T * slots, nt) + 256;
                    if (entries > kWideMaxSegments) {
                        printf("%d experts top-%d, %d shared, %d tokens: %d segments\n", experts, top_k, shared, T, entries);
                        exit(1);
                    }
                    most = std::max(most, entries);
                }
    return most;
}

int main() {
    const int most = plans(), keeps[5] = {0, 5, 20, 40, 100};
    long walked = 0;
    // tasks per expert from one routing to another: even, all on one, all on a few, one crowded among single tokens, random
    for (const int nt : {1, 2, 3, 4, 5, 10})
        for (const int experts : {1, 2, 5, 8, 25, 66, 300, 1030})
            for (const int per : {1, 3, 12, 80})
                for (int routing = 0; routing < 6; ++routing) {
                    const int n_tasks = experts * per;
                    std::vector<int> tasks(experts, 0);
                    for (int t = 0; t < n_tasks; ++t) {
                        const int even = t % experts;
                        int e = even;
                        if (routing == 1) e = experts / 2;
                        if (routing == 2) e = t % std::min(experts, 3);
                        if (routing == 3) e = t < experts ? even : 0;
                        if (routing == 4) e = (int)(rnd() >> 8) % experts;
                        if (routing == 5) e = (int)sqrt((double)((rnd() >> 8) % (unsigned)(experts * experts)));
                        ++tasks[e];
                    }
                    const int max_groups = std::min(experts, n_tasks) + n_tasks / (16 * nt), h_tiles = (n_tasks + 15 * max_groups) / 16;
                    std::vector<Group> groups;
                    int first = 0;
                    for (int e = 0; e < experts; ++e) {
                        const int parts = (tasks[e] + 16 * nt - 1) / (16 * nt), len = parts ? (tasks[e] + parts - 1) / parts : 0;
                        for (int p = 0, left = tasks[e]; p < parts; ++p) {
                            const int n = std::min(len, left);
                            groups.push_back(Group{n, (first + 15 * (int)groups.size()) >> 4});
                            first += n;
                            left -= n;
                        }
                    }
                    for (const int f : {1, 9, 64, 161, 704, 900, 1408, 4096})
                        for (const int est : {(int)groups.size(), max_groups, (max_groups + 1) / 2}) {
                            const long pairs = (long)est * ((f + 31) / 32);
                            int W = (int)std::min(pairs, 256l);  // as the plan has it
                            if (W > 8) W &= ~7;
                            if ((long)groups.size() * f > 150000) continue;
                            walk(groups, max_groups, h_tiles, nt, f, W, keeps[(rnd() >> 8) % 5]);
                            ++walked;
                        }
                }
    printf("ok %ld cuts, up to %d segments\n", walked, most);
    return 0;
}
