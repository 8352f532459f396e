// Rules of the launches and kernels that are plain integer arithmetic: compiled into the library's host and device
// code, and by themselves into a CPU test.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <utility>
#include <vector>

namespace splc {

// A product walks the rows of a row-major `rows` x `width` operand in tiles of `tile_rows`, every lane loading `floats`
// consecutive floats per row from a column that is a multiple of `floats` and below `width` (or from column 0).  A lane
// that straddles the last column reads up to floats - 1 floats of the rows that follow: of one row, or of several where
// the operand is narrower than a load (then (floats - 1) / width of them, rounded up, which floats - width covers).
// Returns how many leading tiles have those rows behind them, so that their loads need no guard.  (floats <= tile_rows:
// where rows < spare the quotient is 0.  A select for that case, or a division by the width, made the compiler address
// the loads of project_rows_kernel through scalar registers instead, up to 18 % slower: 2450 x 1472 onto 160, 19.0 ->
// 22.5 us.)
constexpr int unguarded_tiles(int rows, int width, int floats, int tile_rows) {
    const int spare = width % floats == 0 ? 0 : (width < floats - 1 ? floats - width : 1);
    return (rows - spare) / tile_rows;
}

// How expand_kernel's workgroups share the tiles: `parts` of them each take an equal part of one row block's column tiles,
// or (parts 0) each takes an equal run of all tiles, row block after row block, and new rows on the way.
struct TileRun { int row_block, col_tile, tiles; };
constexpr TileRun tile_run(int place, int groups, int row_blocks, int col_tiles, int parts) {
    if (parts > 0) {
        const int part = place % parts, each = col_tiles / parts, more = col_tiles % parts;
        return TileRun{place / parts, part * each + (part < more ? part : more), each + (part < more ? 1 : 0)};
    }
    const int tiles = row_blocks * col_tiles, each = tiles / groups, more = tiles % groups;
    const int first = place * each + (place < more ? place : more);
    return TileRun{first / col_tiles, first % col_tiles, each + (place < more ? 1 : 0)};
}
// Parts of a row block, unless equal runs are shorter by more than the two tiles that taking new rows costs (their loads,
// 3 to 4 us, and the two tiles in flight, which are finished first).
constexpr int parts_of_row_block(int row_blocks, int col_tiles, int units) {
    const int parts = units / row_blocks < col_tiles ? units / row_blocks : col_tiles;
    const int64_t run = ((int64_t)row_blocks * col_tiles + units - 1) / units;
    return parts > 0 && (col_tiles + parts - 1) / parts <= run + 2 ? parts : 0;
}

// Whether expand_kernel's workgroups, one per compute unit, are at work nine tenths of the time of the longest.
constexpr bool shared_evenly(int64_t rows, int width, int units) {
    const int64_t tiles = (rows + 127) / 128 * (width / 32);
    const int parts = parts_of_row_block((int)((rows + 127) / 128), width / 32, units);
    const int64_t most = parts > 0 ? (width / 32 + parts - 1) / parts : (tiles + units - 1) / units;
    return tiles * 10 >= most * units * 9;
}

// Second product of the subspace calls (out [rows, width] = coefficients [rows, k] U^T): expand_kernel, which keeps rows of
// coefficients in registers and walks along the columns, instead of the GEMM kernel's tile per workgroup.  It needs k above
// 32 (below, memory bounds both) and what fits its registers and LDS: k <= 256, split products 224; for the update also whole
// 128-byte lines in a row.  tiles: of 128 rows x 32 columns.
// half: the last step of 32 k is at most half used.  Time of the GEMM kernel over time of expand_kernel, MI355X, inputs that the
// call before did not leave in a cache (profiles/subspace_rules_measured.txt):
//   update (re-projection, both passes), split, width above 320: 0.94 ... 1.6 (median 1.12), but k to 48 from 19,000 tiles on
//     0.93 ... 1.03; width to 320, an even number of 64-column blocks: 1.0 ... 1.6 up to 1024 tiles; an odd number, from 10 tiles
//     and up to 3072 rows 0.91 ... 1.24, single rows of few tiles 0.91 ... 1.0, more rows 0.84 ... 1.17;
//   update, fp32, from 3072 tiles on 0.97 ... 1.23 (k 41 ... 47 0.98 ... 1.13, k 48 0.96 ... 1.03, k to 40 0.95 ... 1.08, median 1.0),
//     1248 ... 2760 tiles 0.90 ... 1.06, fewer 0.73 ... 1.0;
//   reconstruction, split, one table: 0.95 ... 2.4 (an odd number of 64-column blocks, whose GEMM tile is 64 columns wide, 0.95 ...
//     1.1 up to 700 tiles, 1.0 ... 1.44 from 1200 on);
//   reconstruction, split, no table: k from 65 on 1.1 ... 1.98 below 1024 tiles, from there 0.92 ... 1.45 (half and not shared
//     evenly 0.81 ... 1.1), width to 256 0.89 ... 1.2; k to 64 0.83 ... 1.3 with no clear line;
//   reconstruction, split, both tables: below 1024 tiles 1.2 ... 2.4; from there k from 73 on 0.92 ... 1.9; k 41 ... 72, where memory
//     bounds it, 0.94 ... 1.48 where workgroups stay in a row block, or take up to 4096 tiles, but 0.77 ... 1.18 where more tiles
//     are shared as equal runs and 0.86 ... 1.0 for four parts and more of an odd number of 64-column blocks; k to 40
//     0.86 ... 1.32 (median 1.04);
//   reconstruction, fp32, from 3072 tiles on, with tables: k from 81 on 0.97 ... 1.26, but half 0.94 ... 1.1 (width to 640, one table
//     and fewer than 4096 tiles, or not shared evenly: 0.88 ... 1.09), width to 256 0.88 ... 1.06, k 80 0.89 ... 1.06 (the GEMM kernel's
//     steps are of 16 k); without, from 4096 tiles (k above 224: 8192) and k 128 on 0.97 ... 1.13, half 0.90 ... 1.07 (median 0.98);
//     fewer tiles 0.77 ... 1.06.
constexpr bool expand_takes_k(int k, int tables, bool update, bool split) {
    if (k <= 32 || k > (split ? 224 : 256)) return false;
    if (split) return update || tables > 0 || k > 64;
    if (update) return k > 40 && k != 48;
    return tables > 0 ? k > 80 : k >= 128 && (k - 1) % 32 >= 16;
}
// Whether there are products of so many steps of 32 k: what the launch instantiates.
constexpr bool expand_takes_steps(int steps, int tables, bool update, bool split) {
    for (int k = 32 * steps - 31; k <= 32 * steps; ++k)
        if (expand_takes_k(k, tables, update, split)) return true;
    return false;
}
template <class Units>
constexpr bool expand_applies(int64_t rows, int width, int k, int tables, bool update, bool split, Units units) {
    if (width % 32 != 0 || width >= 1 << 20 || !expand_takes_k(k, tables, update, split)) return false;
    const int64_t tiles = (rows + 127) / 128 * (width / 32);
    if (tiles >= int64_t(1) << 31) return false;
    if (update && !split) return tiles >= 3072;
    if (update) {
        if (k <= 48 && tiles >= 19000) return false;
        return width > 320 || (tiles < 1024 && (width % 128 == 0 || (tiles >= 10 && rows <= 3072)));
    }
    const bool half = (k - 1) % 32 < 16;
    if (split) {
        if (width % 128 != 0 && tiles < 1200) return false;
        if (tables == 1 || tiles < 1024) return true;
        if (tables == 0) return width > 256 && (!half || shared_evenly(rows, width, units()));
        if (k <= 40) return false;
        const int parts = k > 72 ? 1 : parts_of_row_block((int)((rows + 127) / 128), width / 32, units());
        return parts > 0 ? parts < 4 || width % 128 == 0 : tiles < 4096;
    }
    if (width <= 256 || tiles < 3072) return false;
    if (tables == 0) return width > 320 && tiles >= (k > 224 ? 8192 : 4096);
    return !half || (width > 640 && tiles >= (tables == 2 ? 3072 : 4096) && shared_evenly(rows, width, units()));
}

// The same for the reconstruction where rows are no whole lines (the GEMM kernel's non-temporal accesses there lose the lines that
// its tiles share), on 256 compute units.  The lines are those of 3300 shapes of 257 to 2050 columns, measured on both sides; what
// they give to expand_kernel was measured from 33 to 16,000 columns (profiles/subspace_across_lines_measured.txt: narrow
// rows too gain 1.03 to 2.6 in the median of every class, the least in fp32 with both tables, to 256 columns, from 1024
// tiles on: 0.92 ... 1.3).  Time of the GEMM kernel over time of expand_kernel:
//   split, one table 1.04 ... 4.2 (median 1.6); both, below 4096 tiles 0.94 ... 3.9 (median 1.6), from there k from 65 on 0.95 ...
//     1.29, to 64 and, from 12,000 tiles on, to 128 0.87 ... 1.25; none, k from 65 on: an even number of 64-column blocks, below 512
//     tiles 0.97 ... 1.69, from 4096 on 0.95 ... 1.31, between 0.81 ... 1.35; an odd number, below 256 0.99 ... 1.27, from 2048 on
//     0.99 ... 1.48, between 0.82 ... 1.5;
//   fp32 with tables, width no multiple of 4: k 81 ... 128 0.91 ... 1.54 (both, odd, from 4096 tiles on 0.94 ... 1.09); k 129 ... 192,
//     from 1024 tiles on 0.93 ... 1.35, below 0.85 ... 1.39; k from 193 on, even 0.98 ... 1.79, odd, from 4096 tiles on 0.99 ... 1.16,
//     below 0.80 ... 1.19; a multiple of 4, one table, from 3072 tiles on 0.95 ... 1.3, else 0.83 ... 1.4; none 0.69 ... 1.15.
constexpr bool expand_takes_k_across_lines(int k, int tables, bool split) {
    if (split) return k > (tables > 0 ? 32 : 64) && k <= 224;
    return tables > 0 && k > 80 && k <= 256;
}
constexpr bool expand_takes_steps_across_lines(int steps, int tables, bool split) {
    for (int k = 32 * steps - 31; k <= 32 * steps; ++k)
        if (expand_takes_k_across_lines(k, tables, split)) return true;
    return false;
}
constexpr bool expand_applies_across_lines(int64_t rows, int width, int k, int tables, bool split) {
    if (width % 32 == 0 || width < 33 || width >= 1 << 20 || !expand_takes_k_across_lines(k, tables, split)) return false;
    const int64_t tiles = (rows + 127) / 128 * ((width + 31) / 32);
    if (rows < 1 || tiles >= int64_t(1) << 31) return false;
    const bool odd = (width + 63) / 64 % 2 != 0;
    if (split) {
        if (tables == 0) return odd ? tiles < 256 || tiles >= 2048 : tiles < 512 || tiles >= 4096;
        return tables == 1 || tiles < 4096 || (k > 64 && (tiles < 12000 || k > 128));
    }
    if (width % 4 == 0) return tables == 1 && tiles >= 3072;
    if (k <= 128) return !(tables == 2 && odd && tiles >= 4096);
    return k > 192 ? !odd || tiles >= 4096 : tiles >= 1024;
}

// First product of the subspace calls: contract_kernel (split products) and contract_fp32_kernel, one workgroup per compute
// unit and 64 rows with all columns, instead of the GEMM kernel.  Time of the GEMM kernel over theirs, MI355X, by blocks of
// 64 rows (256 units; a second round of workgroups begins with block 257; profiles/subspace_rules_measured.txt, and below
// the lines profiles/contract_fp32_rule_measured.txt):
//   split (rounds of workgroups, and percent of the units that have one on average over them; lines: rows of whole 128-byte
//   lines, which the GEMM kernel reads faster; inputs that the call before did not leave in a cache):
//     k 129 ... 192, one round from a third of the units on 0.97 ... 1.71, but with tables on other rows than lines, d below 768
//       and less than half of the units 0.94 ... 1.1; more rounds from 68 % on 0.97 ... 1.87, below 0.84 ... 1.12; there without
//       tables below d 640 0.87 ... 1.1 (four rounds and more, below d 768: 0.87 ... 1.07), and with one table on lines, d
//       below 640 and less than 88 % 0.91 ... 1.09;
//     k 65 ... 128, no table, from a quarter of the units on: one and two rounds 0.95 ... 1.78 (31456 x 512 onto 118: 0.89), three
//       1.0 ... 1.18 from d 640 on (below 0.94 ... 1.04), more 0.91 ... 1.2 from d 1024 on (below 0.84 ... 1.08);
//     k 65 ... 128, tables, 72 to 256 blocks: one 0.95 ... 1.52, both from half of the units on 1.07 ... 1.35, fewer 1.0 ... 1.22 on
//       lines from d 768 on and 0.90 ... 1.14 elsewhere; 257 blocks and more 0.91 ... 1.11;
//   fp32, measured and told apart in the same way:
//     k 129 ... 192 (the GEMM tile pads them to 256), both tables, from 67 % on 1.00 ... 1.81, below 0.70 ... 1.0; one table, one
//       and two rounds 0.95 ... 1.66, three and four on lines 0.87 ... 1.07 below 88 % and 0.99 ... 1.25 above, more rounds
//       0.90 ... 1.14, other rows 1.00 ... 1.53; no table, one and two rounds 0.97 ... 1.07 from d 1536 (on lines 1280) on and
//       0.93 ... 1.02 below, three and four 0.84 ... 0.94 below 88 % and 1.01 ... 1.17 above; no table, k to 159: 0.92 ... 1.05;
//     k 193 ... 256 with tables: one round from 60 % and d 1536 on 0.95 ... 1.04, of smaller d 0.93 ... 1.03 (median 0.98), two
//       rounds from d 1280 on 0.97 ... 1.14, below 0.94 ... 1.02, three 0.97 ... 1.31, four and more 0.97 ... 1.11, below d 1280
//       0.95 ... 1.07; fewer percent 0.57 ... 1.0; no table 0.95 ... 1.06 with no clear line;
//   fp32, k to 128: 0.85 ... 1.07; d 512 to 1023: 0.63 ... 1.19.
// Fewer blocks go to the projection of few rows or, some of them, to the GEMM kernel (0.5 ... 0.9).  d is bounded because the
// kernels address U and 64 rows of x by 32-bit byte offsets.  units_of_device(): compute units, asked of the runtime only where
// d and k do not refuse by themselves.
constexpr bool contract_takes_k(int k, int tables, bool split) {
    if (split) return k > 64 && k <= 192;
    return tables > 0 ? k > 128 && k <= 256 : k >= 160 && k <= 192;
}
// Whether there are products of so many times 64 columns: what the launch instantiates.
constexpr bool contract_takes_columns(int times, int tables, bool split) {
    for (int k = 64 * times - 63; k <= 64 * times; ++k)
        if (contract_takes_k(k, tables, split)) return true;
    return false;
}
template <class Units>
constexpr bool contract_applies(int64_t rows, int d, int k, int tables, bool split, Units units_of_device) {
    if (!contract_takes_k(k, tables, split) || d < (split ? 512 : 1024) || d >= 1 << 20) return false;
    const int64_t units = units_of_device();
    const int64_t blocks = (rows + 63) / 64, rounds = (blocks + units - 1) / units;
    const int64_t percent = rounds > 0 ? blocks * 100 / (rounds * units) : 0;       // of the units, in the rounds' average
    const bool lines = d % 32 == 0;              // rows of whole 128-byte lines
    if (!split) {
        if (k > 192) return percent >= (rounds == 1 ? 60 : 80) && d >= (rounds == 1 ? 1536 : rounds == 3 ? 1024 : 1280);
        if (percent < 67) return false;
        const bool full = rounds <= 2 || (rounds <= 4 && percent >= 88);
        if (tables == 0) return full && d >= (lines ? 1280 : 1536);
        return tables == 2 || full || !lines;
    }
    if (k > 128) {
        if (rounds == 1) return blocks * 3 >= units && (tables == 0 || lines || d >= 768 || percent >= 50);
        if (percent < 68) return false;
        if (tables == 0) return d >= (rounds == 2 ? 512 : rounds == 3 ? 640 : 768);
        return tables == 2 || rounds == 2 || !lines || d >= 640 || percent >= 88;
    }
    if (tables == 0) return blocks * 4 > units && d >= (rounds <= 2 ? 512 : rounds == 3 ? 640 : 1024);
    return rounds == 1 && blocks * 32 >= units * 9 && (tables == 1 || blocks * 2 > units || (lines && d >= 768));
}

// Batched calls (compress of several replicas, one-launch step): on plans of few chunks every replica of a chunk gets a
// workgroup of its own, and the one-launch step becomes two launches with the same results: the walk over the replicas
// is a chain, some 4 us each.  Measured, kappa 32, walk / side by side, in us:
//   compress alone: 1 chunk, 1 replica 5.7 / 5.4, 8: 29.4 / 5.5; 300 chunks, 1: 7.9 / 7.6, 4: 23.2 / 13.3; 512, 1: 8.8 /
//     8.7, 8: 46.7 / 37.1, 64: 328 / 296; 700, 8: 54.5 / 56.3, 64: 400 / 461;
//   the step: 1 chunk, 2: 10.2 / 8.9, 8: 31.0 / 10.8; 300, 2: 14.5 / 14.1, 4: 24.0 / 20.0; 512, 2: 16.3 / 15.6, 8: 48.7 /
//     41.6, 64: 332 / 305; 600, 3: 24.1 / 25.4; 700, 8: 56.7 / 61.6;
//   the step with 1 replica, where there is no walk to split: 1 chunk 6.4 / 7.7; 300: 9.0 / 11.0; 512: 10.1 / 12.5.
// Workgroups of different replicas run in any order, and the second launch reads the messages back.  Where the
// replicas' message buffers or error-feedback sets share memory (a caller may have no use for them), the walk, which
// takes the replicas in order and keeps their sum on chip, is what gives the documented result.
constexpr int64_t kFewChunks = 512;
constexpr bool replicas_side_by_side(int64_t chunks, int replicas, bool step, bool buffers_disjoint) {
    return chunks <= kFewChunks && !(step && replicas == 1) && buffers_disjoint;
}

// Compression of a tiled plan: strips of four tiles (1024 lanes, two per compute unit) and a second launch for the tiles
// outside them, or every tile by itself in one launch.  A strip asks for nine cache lines where its tiles ask for twelve,
// which is what large plans are bound by; it takes longer from end to end, and below some rounds of workgroups that, and
// the second launch, are what counts.  Where the general path of the selection is taken often (from some 200 entries on) all four
// tiles of a strip take it together.  Time of the tiles over time of the strips, MI355X, 2050 columns, arrays as the call before left
// them / four replicas in turn (from parameters) / nothing in a cache (profiles/strips_measured.txt):
//   from parameters, kappa 32 and 128: 1496 strips 0.76 / 0.93 / 0.94, 2240 0.95 ... 0.99 / 0.99 / 0.98 ... 0.99, 3240 1.01 ... 1.03 / 1.04 ... 1.05 / 1.03 ...
//     1.05, 4488 1.02 ... 1.04 / 1.02 ... 1.03 / 1.00 ... 1.03, 9984 1.03 ... 1.07 / 1.03 ... 1.05 / 1.03 ... 1.04;
//   from fp32: 2240 0.77 ... 0.78 / 0.91 ... 0.96, 3240 0.98 ... 0.99 / 1.03 ... 1.05, 4488 0.98 ... 0.99 / 0.95 ... 0.97, 9984 1.05 ... 1.09 / 1.04 ... 1.08;
//   from bf16: 2240 0.69 ... 0.75 / 0.92 ... 0.93, 3240 0.83 ... 0.87 / 0.97 ... 1.00, 4488 0.93 ... 0.96 / 0.95 ... 0.99, 9984 0.99 ... 1.04 / 1.02 ... 1.03;
//   kappa 256: 0.67 ... 0.78 at every size from every source.
constexpr bool strips_pay(int64_t strips, int kappa, bool params) { return kappa <= 192 && strips >= (params ? 2700 : 6500); }

// Large plans stream far more than the last-level cache holds, and there fewer workgroups per compute unit than would fit
// keep the memory busier (fewer streams in flight at once) -- as long as memory is what bounds: with other sources, which
// move less per chunk, and with messages or data that need the general path of the selection, the workgroups left out are
// missed.  Measured, all that fit / three per compute unit, in us:
//   compress from parameters: 9000 chunks, kappa 32 / 128: 96.7 / 97.5 -> 94.6 / 96.5; 37,105: 400 / 395 -> 381 / 380;
//     120,000: 1319 / 1319 -> 1228 / 1218; coarse values, 32: 394 -> 378; 1 % nonzeros, 32: 421 -> 521 (that data took 702
//     before the general path left zeros out); kappa 200: 408 -> 477, 256: 407 -> 661, 1000: 419 -> 608; 4096 chunks, 32:
//     43.3 -> 44.1 (a few rounds of workgroups only).  Four per unit change little, two lose 7 to 25 %;
//   compress from bf16: 9000 chunks, kappa 32 / 128: 62.9 / 63.5 -> 73.9 / 81.9; from fp32 differences 72 -> 77;
//   one-launch step: 37,105 chunks (150M parameters), kappa 32, 8 replicas: 2862 -> 2833, 2: 832 -> 799; 8192, 8: 625 ->
//     601, 2: 179 -> 179; 2000, 2: 48.4 -> 51.6;
//   outer update, two per unit: 228,000 chunks (0.9B model): 1866 -> 1803, 120,000: 959 -> 945; 24,000 to 37,105: the same.
constexpr int64_t kFewStreams = 8192, kFewStreamsUpdate = 24000;
constexpr bool few_streams(int64_t chunks, int kappa, bool from_params, bool general_path) {
    return chunks >= kFewStreams && kappa <= 128 && from_params && !general_path;
}

// Aggregation over a flat plan: the entry of the chunk table that a workgroup takes where every XCD (workgroups go to the
// eight of them round-robin by number) is to get runs of kChunkRun consecutive ones; those behind the last whole round of
// eight runs keep their place.  kChunkRun chunks' levels (8 bytes each) are one cache line, and so are two to four
// chunks' pairs at kappa 32 ... 16: taken one by one, every XCD fetches each of these lines for itself.
// Worth it where messages are a large part of the traffic and a small part of a line; otherwise the order of the table keeps
// memory busier.  Time in the table's order / in runs, MI355X, quantised, 9000 to 240,000 chunks
// (profiles/aggregate_runs_measured.txt):
//   aggregate_update, kappa 16 ... 48: 24 and 32 replicas 1.01 ... 1.29, 20: 0.98 ... 1.18, 16: 0.95 ... 1.09, 2 to 8: 0.93 ... 0.97; 40 to
//     64: 1.01 ... 1.14 while the messages are below 240 MB, from there 0.93 ... 1.04; kappa 64: 24 to 48 replicas 1.00 ... 1.15 from
//     12,000 chunks on, 0.99 at 9000, 64 replicas 0.96 ... 0.99; kappa 96 and 128: 0.97 ... 1.17; 4096 chunks, 32 replicas: 0.97 ...
//     1.16, 1500: 0.93 ... 0.97;
//   aggregate, kappa 16 ... 64: 24 to 64 replicas 1.00 ... 1.34 below 240 MB, 0.94 ... 1.05 from 260 MB on (the last-level cache
//     holds 256), 20: 0.94 ... 1.13, 4: 0.92 ... 1.05;
//   without quantisation (the values are whole lines), 32, kappa 32: 0.95 ... 1.12; 128: 0.94 ... 1.01.
constexpr uint32_t kChunkRun = 16;
constexpr uint32_t entry_in_runs(uint32_t place, uint32_t entries) {
    constexpr uint32_t kRound = 8 * kChunkRun;
    if (place >= entries / kRound * kRound) return place;
    const uint32_t slot = place / 8;
    return (slot / kChunkRun * 8 + place % 8) * kChunkRun + slot % kChunkRun;
}
constexpr bool chunks_in_runs(int64_t entries, int replicas, int kappa, bool quantised, bool update) {
    if (!quantised || replicas < 24 || entries < 9000) return false;
    if (kappa > 48 && (kappa > 64 || replicas > 48 || entries < 12000)) return false;
    return (update && replicas <= 32) || entries * replicas * (2 * kappa + 8) < 240000000;
}

// Whether an edge chunk of `rows` local rows holds anything in slot s, which is 16 of them.
constexpr bool slot_used(int rows, int s) { return 16 * s < rows; }

// Aggregation: entries of a chunk's message per lane of the wave that adds it, 0: one replica after the other by one wave, for
// messages that would take too many registers.  A kernel is made for a plan's kappa; an edge chunk that holds fewer elements
// than kappa takes the way of its own messages in it (mean over 17 replicas, 4000 chunks of 100 elements: kappa 512 35.9 -> 20.9
// us, 256 22.2 -> 20.3; of 40: kappa 512 26.1 -> 19.2, 130 21.3 -> 18.9).
constexpr int entries_per_lane(uint32_t entries) { return entries <= 64 ? 1 : (entries <= 128 ? 2 : (entries <= 256 ? 4 : 0)); }

// Aggregation: workgroups that share a compute unit (0: all that fit, eight) and, with the outer update, whether theta is read
// only after the messages have been added (late: the reads of some workgroups then meet the writes of others) or with the
// first of them (its latency then hides behind theirs).  The dense mean alone is a stream of writes that waits for
// messages, and wants all workgroups that fit; with theta read as well, memory is kept busiest by four or five.  Time,
// MI355X, us, messages not in a cache, all that fit / five, early / five, late / four, late:
//   update, quantised, flat: 72,400 chunks, kappa 32: 3 replicas 403 / 395 / 368 / 371, 8: 409 / 395 / 379 / 400, 12: 406 / 394 /
//     435 / 469, 16: 414 / 401 / 393 / 435, 20: 422 / 406 / 436 / 481, 24: 420 / 417 / 423 / 472; kappa 64, 12: 426 / 421 / 419 / 471,
//     16: 448 / 440 / 425 / 440, 20: 460 / 445 / 438 / 485, 24: 462 / 456 / 458 / 487; 32: 481 / 474 / 477 / 507; kappa 128, 12: 472 / 461 /
//     449 / 475, 24: 529 / 514 / 499 / 549; 205,000 chunks, kappa 32, 3: 1165 / 1128 / 1069 / 1030, 8: 1179 / 1167 / 1083 / 1121;
//     5000 and 8400 chunks: within 3 % of each other; kappa 256, 16: 513 / 520 / 541 / 570;
//   unquantised, flat: 72,400, kappa 32, 4 replicas 409 / 404 / 377 / 381, 16: 481 / 468 / 442 / 466, 32: 528 / 526 / 507 / 507; kappa 64,
//     8: 483 / 481 / 460 / 446, 16: 539 / 531 / 516 / 503; kappa 128, 5: 862 / 780 / 756 / 763 (128,000), 32: 755 / 756 / 755 / 736;
//   tiles of 2050 columns, which share cache lines: 69,000, kappa 32, 4: 473 / 456 / 452 / 449, 16: 503 / 484 / 501 / 514, 32: 529 / 514 /
//     550 / 556; 25,600, kappa 32, 4: 173 / 167 / 170 / 172, 64, 24: 201 / 197 / 214 / 218;
//   mean only, all that fit / five / four: 225,000 chunks, kappa 64, 8 replicas 724 / 840 / 919; unquantised, kappa 32, 8: 739 / 849 / 941;
//     70,000 chunks, kappa 64, 8: 311 / 282 / 324, 9: 294 / 309 / 354, 17: 336 / 343 / 383, 32: 408 / 410 / 426; kappa 128, 8: 350 / 324 / 313,
//     12: 363 / 356 / 375, 17: 411 / 415 / 433, 32: 562 / 556 / 568; kappa 200, 27: - / 685 / 749; 25,000, kappa 64, 17: 138 / 133 / 142;
//     messages in a cache, 70,000, kappa 64, 17: 295 / 313 / 356, kappa 128, 17: 373 / 374 / 399.
struct AggregatePace { int groups_per_unit; bool theta_late; };
constexpr AggregatePace aggregate_pace(int64_t chunks, int replicas, int kappa, bool quantised, bool flat, bool update) {
    if (chunks < kFewStreams) return AggregatePace{0, false};
    const bool heavy = !quantised && replicas >= 8 && kappa >= 64;       // messages of the order of the chunk itself
    if (!update) return AggregatePace{heavy ? (replicas == 8 && kappa >= 128 ? 4 : 5) : 0, false};
    if (kappa > 128) return AggregatePace{0, false};
    const bool late = flat && (!quantised || replicas <= 8 || (kappa >= 64 && replicas <= 24));
    return AggregatePace{flat && heavy ? 4 : 5, late};
}

// How the mean alone is divided and stored in a complete chunk; the results are the same.
//   in_turn: a vector is read from the accumulator, divided and stored, and then the next one; a power of two by the
//     multiplication with its inverse;
//   together: the sixteen divisions of a lane stand in front of its four stores.  With divisions between them the stores of a row
//     come apart, and lines that two waves or two tiles write leave the L2 in parts;
//   divided: in turn, and powers of two are divided too.  With one message or two there is little to wait for, and writes that
//     come as fast as a multiplication lets them get in each other's way.
// Time, MI355X, messages in no cache (profiles/aggregate_pace_measured.txt), M no power of two, in turn over together:
//   tiles of 330 to 2050 columns, kappa * M from 192 on: 12,000 chunks 1.00 ... 1.16, 25,000 1.05 ... 1.17, 40,000 1.02 ... 1.26, 70,000 1.02 ...
//     1.20; 96: 0.91 ... 1.11 (median 0.99); 2048 chunks 0.94 ... 1.01;
//   flat: 12,000 chunks 0.98 ... 1.03, 40,000 0.97 ... 1.09; 2048 0.96 ... 0.98.
// Flat, M one or two, kappa * M up to 64, multiplied over divided: 8192 chunks 0.97 ... 1.05, 12,000 0.98 ... 1.05, 45,000 1.07 ... 1.16, 150,000
//   1.09 ... 1.15, messages in a cache 0.98 ... 1.04; four and eight messages 0.84 ... 1.07; tiles of 2048 columns 0.88 ... 1.03.
enum class MeanStores { in_turn, together, divided };
constexpr MeanStores mean_stores(int64_t chunks, int replicas, int kappa, bool flat) {
    if (chunks < kFewStreams) return MeanStores::in_turn;
    if (replicas <= 2) return flat && kappa * replicas <= 64 ? MeanStores::divided : MeanStores::in_turn;
    return (replicas & (replicas - 1)) != 0 && (int64_t)kappa * replicas >= 192 ? MeanStores::together : MeanStores::in_turn;
}

// Whether no two of these address ranges [first, second) share a byte; empty ranges share none.
inline bool disjoint(std::vector<std::pair<uintptr_t, uintptr_t>> ranges) {
    std::sort(ranges.begin(), ranges.end());
    uintptr_t end = 0;
    for (const auto& r : ranges) {
        if (r.first >= r.second) continue;
        if (r.first < end) return false;
        end = r.second;
    }
    return true;
}

}  // namespace splc
