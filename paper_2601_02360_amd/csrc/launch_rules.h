// Rules of the launches and kernels that are plain integer arithmetic: compiled into the library's host and device
// code, and by themselves into a CPU test.
#pragma once

namespace splc {

// A product walks the rows of a row-major `rows` x `width` operand in tiles of `tile_rows`, every lane loading `floats`
// consecutive floats per row from a column that is a multiple of `floats` and below `width` (or from column 0).  A lane
// that straddles the last column reads up to floats - 1 floats of the rows that follow: (floats - 1) / width of them,
// rounded up -- more than one where the operand is narrower than a load.  Returns how many leading tiles have those
// rows behind them, so that their loads need no guard.
constexpr int unguarded_tiles(int rows, int width, int floats, int tile_rows) {
    const int spare = width % floats == 0 ? 0 : (floats - 1 + width - 1) / width;
    return rows > spare ? (rows - spare) / tile_rows : 0;
}

}  // namespace splc
