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
