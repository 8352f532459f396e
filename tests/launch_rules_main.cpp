// The launch rules of the library (csrc/launch_rules.h) on the CPU.
#include <cstdio>
#include <initializer_list>
#include "launch_rules.h"

// The projection of few rows reads U (d x k) NB floats a lane, 32 rows a tile: no unguarded load may pass its end.
static int check_unguarded_tiles() {
    for (int nb : {2, 4})
        for (int d : {1, 2, 3, 31, 32, 33, 34, 35, 63, 64, 256, 257, 258, 259, 260, 287, 288, 289, 290, 291, 2050})
            for (int k = 1; k <= 40 && k <= d; ++k) {
                const int n = splc::unguarded_tiles(d, k, nb, 32);
                if (n < 0 || n > d / 32 || (k % nb == 0 && n != d / 32) || n < d / 32 - 1) {
                    printf("d %d k %d nb %d: %d tiles\n", d, k, nb, n);
                    return 1;
                }
                for (int row = 0; row < 32 * n; ++row)
                    for (int col = 0; col < k + nb; col += nb) {
                        const long first = (long)row * k + (col < k ? col : 0);
                        if (first + nb > (long)d * k) {
                            printf("d %d k %d nb %d: row %d column %d reads element %ld of %ld\n", d, k, nb, row, col,
                                   first + nb - 1, (long)d * k);
                            return 1;
                        }
                    }
            }
    return 0;
}

// Replicas go side by side only where nothing one of them writes is another one's.
static int check_side_by_side() {
    using Ranges = std::vector<std::pair<uintptr_t, uintptr_t>>;
    const struct { Ranges r; bool apart; } cases[] = {
        {{}, true}, {{{100, 200}}, true}, {{{100, 200}, {200, 300}}, true}, {{{200, 300}, {100, 200}}, true},
        {{{100, 200}, {100, 200}}, false}, {{{150, 250}, {100, 200}}, false}, {{{100, 400}, {150, 200}, {300, 301}}, false},
        {{{100, 400}, {400, 500}, {499, 600}}, false}, {{{100, 100}, {100, 200}, {150, 150}}, true}, {{{0, 0}, {0, 0}}, true}};
    for (const auto& c : cases)
        if (splc::disjoint(c.r) != c.apart) { printf("disjoint: wrong answer\n"); return 1; }
    for (int64_t chunks : {1, 100, 512, 513, 100000})
        for (int replicas : {1, 2, 3, 1024})
            for (bool step : {false, true})
                if (splc::replicas_side_by_side(chunks, replicas, step, false)) {
                    printf("%ld chunks: shared buffers\n", (long)chunks);
                    return 1;
                }
    // the largest plan each number of replicas is taken side by side on (0: none)
    const struct { int replicas; bool step; int64_t most; } lines[] = {
        {1, false, 512}, {2, false, 512}, {1024, false, 512}, {1, true, 0}, {2, true, 512}, {3, true, 512}, {1024, true, 512}};
    for (const auto& l : lines)
        if ((l.most > 0 && !splc::replicas_side_by_side(l.most, l.replicas, l.step, true)) ||
            splc::replicas_side_by_side(l.most + 1, l.replicas, l.step, true)) {
            printf("line of %d replicas%s\n", l.replicas, l.step ? ", step" : "");
            return 1;
        }
    return 0;
}

// Fewer workgroups per compute unit only where memory bounds the launch.
static int check_few_streams() {
    const struct { int64_t chunks; int kappa; bool params, general, want; } cases[] = {
        {8192, 32, true, false, true}, {8191, 32, true, false, false}, {220000, 128, true, false, true},
        {220000, 129, true, false, false}, {220000, 1000, true, false, false}, {220000, 32, false, false, false},
        {220000, 32, true, true, false}};
    for (const auto& c : cases)
        if (splc::few_streams(c.chunks, c.kappa, c.params, c.general) != c.want) {
            printf("few_streams: %ld chunks, kappa %d\n", (long)c.chunks, c.kappa);
            return 1;
        }
    return 0;
}

// The aggregation's pace on both sides of each line (the second half: test_large_plans of test_gpu_aggregate_kernels.py).
static int check_aggregate_pace() {
    const struct { int64_t chunks; int replicas, kappa; bool quantised, flat, update; int groups; bool late; } cases[] = {
        {8191, 8, 64, true, true, true, 0, false}, {8191, 32, 128, false, false, false, 0, false}, {8191, 3, 16, false, true, true, 0, false},
        // the mean alone: only unquantised messages of the order of the chunk itself
        {8192, 32, 128, true, true, false, 0, false}, {8192, 7, 128, false, true, false, 0, false}, {8192, 8, 63, false, true, false, 0, false},
        {8192, 8, 64, false, true, false, 5, false}, {8192, 8, 127, false, true, false, 5, false}, {8192, 8, 128, false, true, false, 4, false},
        {8192, 8, 256, false, false, false, 4, false}, {8192, 9, 128, false, true, false, 5, false}, {220000, 17, 64, false, true, false, 5, false},
        {220000, 32, 256, false, false, false, 5, false}, {220000, 1024, 4096, false, true, false, 5, false},
        // with the update, quantised
        {8192, 8, 16, true, true, true, 5, true}, {8192, 9, 16, true, true, true, 5, false}, {8192, 9, 63, true, true, true, 5, false},
        {8192, 9, 64, true, true, true, 5, true}, {8192, 24, 128, true, true, true, 5, true}, {8192, 25, 128, true, true, true, 5, false},
        {8192, 1, 128, true, true, true, 5, true}, {8192, 1, 129, true, true, true, 0, false}, {8192, 8, 64, true, false, true, 5, false},
        {220000, 32, 64, true, false, true, 5, false},
        // with the update, unquantised
        {8192, 7, 64, false, true, true, 5, true}, {8192, 8, 63, false, true, true, 5, true}, {8192, 8, 64, false, true, true, 4, true},
        {8192, 1024, 128, false, true, true, 4, true}, {8192, 32, 129, false, true, true, 0, false}, {8192, 32, 64, false, false, true, 5, false},
        {8192, 3, 16, true, true, true, 5, true}, {8192, 9, 16, true, true, true, 5, false}, {8192, 9, 64, true, true, true, 5, true},
        {8192, 2, 200, true, true, true, 0, false}, {8192, 8, 64, false, true, true, 4, true}, {8192, 8, 128, false, true, true, 4, true},
        {8192, 5, 32, false, true, true, 5, true}, {8192, 9, 64, true, true, false, 0, false}, {8192, 8, 64, false, true, false, 5, false},
        {8192, 8, 128, false, true, false, 4, false}, {8192, 5, 32, false, true, false, 0, false}};
    for (const auto& c : cases) {
        const splc::AggregatePace p = splc::aggregate_pace(c.chunks, c.replicas, c.kappa, c.quantised, c.flat, c.update);
        if (p.groups_per_unit != c.groups || p.theta_late != c.late) {
            printf("aggregate_pace: %ld chunks, %d replicas, kappa %d, %d %d %d: %d %d\n", (long)c.chunks, c.replicas, c.kappa,
                   c.quantised, c.flat, c.update, p.groups_per_unit, p.theta_late);
            return 1;
        }
    }
    return 0;
}

// Division and stores of the mean on both sides of each line (second half: the plans of test_gpu_aggregate_kernels.py).
static int check_mean_stores() {
    using splc::MeanStores;
    const MeanStores turn = MeanStores::in_turn, together = MeanStores::together, divided = MeanStores::divided;
    const struct { int64_t chunks; int replicas, kappa; bool flat; MeanStores want; } cases[] = {
        {8192, 3, 64, true, together}, {8191, 3, 64, true, turn}, {8192, 3, 63, true, turn}, {8192, 4, 64, true, turn}, {220000, 1024, 128, false, turn},
        {220000, 1023, 1, true, together}, {8192, 7, 4096, false, together}, {8192, 191, 1, true, turn}, {8192, 193, 1, false, together},
        {8192, 1, 64, true, divided}, {8191, 1, 64, true, turn}, {8192, 1, 65, true, turn}, {8192, 1, 64, false, turn}, {220000, 2, 32, true, divided},
        {8192, 2, 33, true, turn}, {8192, 4, 16, true, turn}, {8192, 1, 4096, true, turn}, {8192, 2, 4096, false, turn}, {1, 1, 1, true, turn},
        {8192, 9, 64, true, together}, {8192, 2, 200, true, turn}, {8192, 2, 16, true, divided}, {8320, 3, 64, false, together},
        {8320, 9, 31, false, together}, {8320, 17, 200, false, together}, {8320, 7, 300, false, together}};
    for (const auto& c : cases)
        if (splc::mean_stores(c.chunks, c.replicas, c.kappa, c.flat) != c.want) {
            printf("mean_stores: %ld chunks, %d replicas, kappa %d, %d\n", (long)c.chunks, c.replicas, c.kappa, c.flat);
            return 1;
        }
    return 0;
}

// A lane takes as few entries as hold the message.
static int check_entries_per_lane() {
    const struct { uint32_t entries; int want; } cases[] = {{1, 1}, {64, 1}, {65, 2}, {128, 2}, {129, 4}, {256, 4}, {257, 0}, {4096, 0}};
    for (const auto& c : cases)
        if (splc::entries_per_lane(c.entries) != c.want) {
            printf("entries_per_lane(%u)\n", c.entries);
            return 1;
        }
    return 0;
}

// A slot is left out exactly where none of its rows exists.
static int check_slot_used() {
    for (int rows = 1; rows <= 64; ++rows)
        for (int s = 0; s < 4; ++s) {
            bool any = false;
            for (int r = 16 * s; r < 16 * s + 16; ++r) any |= r < rows;
            if (splc::slot_used(rows, s) != any) {
                printf("slot %d of %d rows\n", s, rows);
                return 1;
            }
        }
    return 0;
}

// Strips on both sides of each line.  Every plan of test_gpu_strips.py and of test_edge_chunks.py's test of both sides is on one.
static int check_strips_pay() {
    const struct { int64_t least; int kappa; bool params; } lines[] = {
        {2700, 1, true}, {2700, 64, true}, {2700, 128, true}, {2700, 192, true}, {-1, 193, true}, {-1, 4096, true},
        {6500, 1, false}, {6500, 32, false}, {6500, 64, false}, {6500, 65, false}, {6500, 128, false}, {6500, 160, false}, {6500, 192, false},
        {-1, 193, false}, {-1, 4096, false}};
    for (const auto& l : lines)
        if (splc::strips_pay(0, l.kappa, l.params) ||
            (l.least < 0 ? splc::strips_pay(int64_t(1) << 27, l.kappa, l.params)
                         : splc::strips_pay(l.least - 1, l.kappa, l.params) || !splc::strips_pay(l.least, l.kappa, l.params))) {
            printf("strips_pay: kappa %d, %d\n", l.kappa, l.params);
            return 1;
        }
    return 0;
}

int main() {
    if (check_unguarded_tiles() || check_side_by_side() || check_few_streams() || check_aggregate_pace() || check_mean_stores() || check_entries_per_lane() ||
        check_slot_used() || check_strips_pay())
        return 1;
    printf("ok\n");
    return 0;
}
