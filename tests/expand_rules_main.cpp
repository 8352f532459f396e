// How expand_kernel's workgroups share the output tiles and the aggregation's the chunks (csrc/launch_rules.h), on the CPU:
// every one exactly once.
#include <algorithm>
#include <cstdio>
#include <initializer_list>
#include <vector>

#include "launch_rules.h"

static int check(int row_blocks, int col_tiles, int units) {
    const int parts = splc::parts_of_row_block(row_blocks, col_tiles, units);
    const int tiles = row_blocks * col_tiles, groups = parts ? parts * row_blocks : std::min(tiles, units);
    std::vector<char> seen(tiles, 0);
    int most = 0;
    for (int place = 0; place < groups; ++place) {
        const splc::TileRun r = splc::tile_run(place, groups, row_blocks, col_tiles, parts);
        const int first = r.row_block * col_tiles + r.col_tile;
        if (r.tiles < 0 || (r.tiles > 0 && (r.row_block < 0 || r.col_tile < 0 || r.col_tile >= col_tiles))) return 1;
        if (parts && r.col_tile + r.tiles > col_tiles) return 2;         // a part stays in its row block
        most = std::max(most, r.tiles);
        for (int t = first; t < first + r.tiles; ++t) {
            if (t >= tiles || seen[t]) return 3;
            seen[t] = 1;
        }
    }
    if (std::count(seen.begin(), seen.end(), 1) != tiles) return 4;
    if (groups > units || most > (tiles + units - 1) / units + 2) return 5;
    return 0;
}

int main() {
    for (int units : {1, 8, 104, 256})
        for (int row_blocks : {1, 2, 3, 5, 16, 100, 127, 128, 129, 200, 250, 255, 256, 257, 300, 393, 513})
            for (int col_tiles = 1; col_tiles <= 64; ++col_tiles)
                if (const int rc = check(row_blocks, col_tiles, units)) {
                    printf("%d row blocks x %d tiles on %d units: %d\n", row_blocks, col_tiles, units, rc);
                    return 1;
                }
    // what the kernel cannot take is never sent to it
    for (int k : {1, 16, 32, 33, 80, 224, 225, 256, 257, 512})
        for (int width : {512, 520, 2048, 2050, 1 << 20})
            for (bool split : {false, true})
                for (bool update : {false, true})
                    for (int tables : {0, 1, 2})
                        if (splc::expand_applies(1 << 20, width, k, tables, update, split, [] { return 256; }) &&
                            (width % 32 || width >= 1 << 20 || k <= 32 || k > (split ? 224 : 256))) {
                            printf("width %d k %d\n", width, k);
                            return 1;
                        }
    // nor across lines, and whatever is sent has a kernel (a launch of other steps would do nothing)
    for (int width = 1; width <= 2100; width += width < 300 ? 1 : 7)
        for (int wide : {width, width + 30000, (1 << 20) - 32 + width % 64})
            for (int k = 1; k <= 300; ++k)
                for (bool split : {false, true})
                    for (int tables : {0, 1, 2})
                        for (int64_t rows : {0, 1, 1000, 16384, 100000, 1 << 30}) {
                            if (!splc::expand_applies_across_lines(rows, wide, k, tables, split)) continue;
                            const bool steps = splc::expand_takes_steps_across_lines((k + 31) / 32, tables, split);
                            const int64_t tiles = (rows + 127) / 128 * ((wide + 31) / 32);
                            if (rows < 1 || wide % 32 == 0 || wide < 33 || wide >= 1 << 20 || k <= (split ? 32 : 80) || k > (split ? 224 : 256) ||
                                (!split && tables == 0) || tiles >= int64_t(1) << 31 || !steps) {
                                printf("across lines: rows %ld width %d k %d, %d tables\n", (long)rows, wide, k, tables);
                                return 1;
                            }
                        }
    for (bool split : {false, true})
        for (int tables : {0, 1, 2})
            for (int steps = 1; steps <= 9; ++steps) {
                bool taken = false;
                for (int k = 32 * steps - 31; k <= 32 * steps; ++k)
                    for (int64_t rows : {1, 16384, 50304})
                        for (int width : {100, 257, 1090, 2050}) taken |= splc::expand_applies_across_lines(rows, width, k, tables, split);
                if (taken != splc::expand_takes_steps_across_lines(steps, tables, split)) {
                    printf("across lines, %d steps, %d tables\n", steps, tables);
                    return 1;
                }
            }
    const struct { int64_t rows; int width, k, tables; bool split, taken; } across[] = {
        {1, 33, 33, 1, true, true}, {1, 33, 33, 0, true, false}, {1, 130, 65, 0, true, true}, {1, 130, 64, 0, true, false},
        {1, 31, 31, 1, true, false}, {1, 2050, 224, 2, true, true}, {1, 2050, 225, 2, true, false}, {1, 2048, 100, 1, true, false},
        {15872, 1000, 40, 2, true, true}, {16384, 1000, 40, 2, true, false}, {16384, 1000, 65, 2, true, true}, {48000, 1000, 128, 2, true, false},
        {47872, 1000, 128, 2, true, true}, {48000, 1000, 129, 2, true, true}, {48000, 1000, 33, 1, true, true},
        {1792, 1100, 70, 0, true, true}, {1920, 1100, 70, 0, true, false}, {15104, 1100, 70, 0, true, true}, {14976, 1100, 70, 0, true, false},
        {896, 1060, 70, 0, true, true}, {1024, 1060, 70, 0, true, false}, {7808, 1060, 70, 0, true, true}, {7680, 1060, 70, 0, true, false},
        {1, 130, 81, 1, false, true}, {1, 130, 80, 1, false, false}, {100000, 130, 100, 0, false, false}, {1, 1001, 256, 1, false, true},
        {1, 1001, 257, 1, false, false}, {12288, 1000, 100, 1, false, true}, {12160, 1000, 100, 1, false, false}, {12288, 1000, 100, 2, false, false},
        {3200, 1307, 161, 2, false, true}, {3072, 1307, 161, 2, false, false}, {4096, 1001, 129, 1, false, true}, {3968, 1001, 129, 1, false, false},
        {12800, 1307, 200, 1, false, true}, {12672, 1307, 200, 1, false, false}, {12800, 1307, 100, 2, false, false},
        {12672, 1307, 100, 2, false, true}, {12800, 1307, 100, 1, false, true}, {1, 1001, 200, 2, false, true}};
    for (const auto& c : across)
        if (splc::expand_applies_across_lines(c.rows, c.width, c.k, c.tables, c.split) != c.taken) {
            printf("across lines, line: rows %ld width %d k %d, %d tables, %d\n", (long)c.rows, c.width, c.k, c.tables, c.split);
            return 1;
        }
    for (int64_t rows : {0, 1, 5440, 11008, 16384, 16448, 32768, 1 << 24})
        for (int k : {1, 64, 65, 128, 129, 192, 193, 256, 257, 600})
            for (int d : {16, 511, 512, 1023, 1024, 2050, 1 << 20, 1 << 23})
                for (bool split : {false, true})
                    for (int tables : {0, 1, 2})
                        for (int units : {1, 104, 256}) {
                            int asked = 0;
                            const bool applies = splc::contract_applies(rows, d, k, tables, split, [&] { return ++asked, units; });
                            const bool refused = d < (split ? 512 : 1024) || (int64_t)d * k * 4 >= int64_t(1) << 32 || k <= (split ? 64 : 128) ||
                                                 k > (split ? 192 : 256);
                            if ((applies && (rows == 0 || refused)) || (refused && asked) || asked > 1) {      // asking takes runtime calls
                                printf("rows %d d %d k %d, units asked for %d times\n", (int)rows, d, k, asked);
                                return 1;
                            }
                        }
    // where the GEMM kernel was measured to be faster, and neighbours of these shapes where it was not
    const auto card = [] { return 256; };
    const struct { int64_t rows; int d, k, tables; bool split, taken; } first[] = {
        {50304, 1728, 161, 0, false, false}, {36864, 1393, 190, 0, false, false}, {47104, 1984, 175, 0, false, true},
        {14336, 1059, 167, 0, false, false}, {16384, 1536, 167, 0, false, true}, {16384, 1280, 160, 0, false, true},
        {16384, 1279, 160, 0, false, false}, {37888, 1088, 170, 1, false, false}, {37532, 1059, 173, 1, false, true},
        {45056, 1216, 137, 1, false, true}, {84992, 1344, 170, 1, false, false}, {36864, 1088, 170, 2, false, true},
        {14336, 1297, 247, 2, false, false}, {16384, 1536, 247, 2, false, true}, {30720, 1088, 200, 2, false, false},
        {30720, 1280, 200, 2, false, true}, {45056, 1088, 200, 2, false, true},
        {54245, 512, 115, 0, true, false}, {54272, 799, 120, 0, true, false}, {54272, 1024, 120, 0, true, true},
        {36622, 576, 97, 0, true, false}, {36622, 640, 97, 0, true, true}, {38912, 576, 160, 0, true, false},
        {38912, 640, 160, 0, true, true}, {49743, 704, 180, 0, true, false}, {36072, 512, 132, 1, true, false},
        {37060, 519, 136, 1, true, true}, {46859, 576, 148, 1, true, true}, {5876, 545, 151, 2, true, false},
        {5876, 576, 151, 2, true, true}, {8597, 549, 135, 2, true, true}, {5120, 512, 78, 2, true, false},
        {6144, 660, 116, 2, true, false}, {6052, 832, 91, 2, true, true}};
    for (const auto& c : first)
        if (splc::contract_applies(c.rows, c.d, c.k, c.tables, c.split, card) != c.taken) {
            printf("first product %d x %d onto %d, %d tables\n", (int)c.rows, c.d, c.k, c.tables);
            return 1;
        }
    const struct { int64_t rows; int width, k, tables; bool update, split, taken; } second[] = {
        {43008, 960, 64, 2, false, true, false}, {30720, 896, 59, 2, false, true, true}, {22016, 448, 47, 2, false, true, true},
        {6144, 1088, 48, 2, false, true, false}, {6144, 1024, 48, 2, false, true, true}, {82853, 1536, 44, 2, false, true, false},
        {82853, 1536, 44, 1, false, true, true}, {82853, 1536, 73, 2, false, true, true}, {12288, 1024, 38, 2, false, true, false},
        {1024, 1024, 38, 2, false, true, true}, {8529, 896, 97, 0, false, true, false}, {8529, 896, 113, 0, false, true, true},
        {8192, 896, 97, 0, false, true, true}, {47046, 256, 130, 0, false, true, false}, {4096, 256, 130, 0, false, true, true},
        {5840, 192, 163, 0, true, true, false}, {3072, 192, 134, 0, true, true, true}, {64, 192, 34, 0, true, true, false},
        {4096, 256, 224, 0, true, true, true}, {59653, 1984, 41, 0, true, true, false}, {30000, 1984, 41, 0, true, true, true},
        {94208, 192, 133, 1, false, false, false}, {41984, 320, 188, 2, false, false, true}, {41984, 576, 101, 2, false, false, false},
        {41984, 704, 101, 2, false, false, true}, {41984, 576, 92, 2, false, false, true}, {14336, 1152, 97, 1, false, false, false},
        {16384, 1152, 97, 1, false, false, true}, {9126, 1792, 80, 2, false, false, false}, {9126, 1792, 81, 2, false, false, true},
        {14218, 1216, 162, 0, false, false, false}, {22918, 896, 192, 0, false, false, true}, {42739, 1024, 136, 0, false, false, false},
        {39888, 832, 33, 0, true, false, false}, {35968, 512, 40, 0, true, false, false}, {40858, 1216, 48, 0, true, false, false},
        {40858, 1216, 49, 0, true, false, true}, {43043, 1216, 46, 0, true, false, true}};
    for (const auto& c : second)
        if (splc::expand_applies(c.rows, c.width, c.k, c.tables, c.update, c.split, card) != c.taken) {
            printf("second product %d x %d from %d, %d tables\n", (int)c.rows, c.width, c.k, c.tables);
            return 1;
        }
    for (uint32_t entries : {1u, 127u, 128u, 129u, 255u, 256u, 9000u, 9087u, 9088u, 37105u}) {
        std::vector<char> seen(entries, 0);
        for (uint32_t place = 0; place < entries; ++place) {
            const uint32_t e = splc::entry_in_runs(place, entries);
            if (e >= entries || seen[e]++) {
                printf("%u of %u entries\n", place, entries);
                return 1;
            }
        }
    }
    // whatever is taken has a kernel, and every kernel has something that is taken
    for (bool split : {false, true})
        for (int tables : {0, 1, 2}) {
            for (bool update : {false, true})
                for (int steps = 1; steps <= 9; ++steps) {
                    bool taken = false;
                    for (int k = 32 * steps - 31; k <= 32 * steps; ++k)
                        for (int64_t rows : {1, 1000, 16384, 50304})
                            for (int width : {256, 512, 1088, 2048})
                                taken |= splc::expand_applies(rows, width, k, update ? 0 : tables, update, split, card);
                    if (taken != splc::expand_takes_steps(steps, update ? 0 : tables, update, split)) {
                        printf("second product of %d steps, %d tables\n", steps, tables);
                        return 1;
                    }
                }
            for (int times = 1; times <= 5; ++times) {
                bool taken = false;
                for (int k = 64 * times - 63; k <= 64 * times; ++k)
                    for (int64_t rows : {1, 5000, 16384, 32768, 50304})
                        for (int d : {512, 1023, 1088, 2048}) taken |= splc::contract_applies(rows, d, k, tables, split, card);
                if (taken != splc::contract_takes_columns(times, tables, split)) {
                    printf("first product of %d x 64 columns, %d tables\n", times, tables);
                    return 1;
                }
            }
        }
    // (the first ones are the plans of test_gpu_aggregate_runs.py)
    const struct { int64_t entries; int replicas, kappa; bool update, runs; } aggregations[] = {
        {9000, 32, 16, false, true}, {8999, 32, 16, true, false}, {9084, 24, 33, true, true}, {12160, 33, 64, true, true},
        {9084, 24, 33, false, true}, {12160, 33, 64, false, true}, {9000, 32, 16, true, true},
        {200000, 24, 24, false, false}, {200000, 24, 24, true, true}, {130000, 28, 32, false, false}, {130000, 32, 32, true, true},
        {130000, 40, 48, true, false}, {200000, 40, 24, true, false}, {100000, 40, 24, true, true}, {100000, 48, 48, true, false},
        {37105, 64, 32, true, true}, {37105, 23, 32, true, false}, {240000, 24, 16, false, true}, {100000, 24, 65, true, false}};
    for (const auto& c : aggregations)
        if (splc::chunks_in_runs(c.entries, c.replicas, c.kappa, true, c.update) != c.runs ||
            splc::chunks_in_runs(c.entries, c.replicas, c.kappa, false, c.update)) {
            printf("aggregation of %d chunks, %d replicas, kappa %d\n", (int)c.entries, c.replicas, c.kappa);
            return 1;
        }
    printf("ok\n");
    return 0;
}
