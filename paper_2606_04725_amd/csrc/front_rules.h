// Index rules of the front kernels that a program without a device can check:
// plain constant expressions, the same on the host and in the kernels.
#pragma once

#include <cstddef>
#include <cstdint>

namespace nmpc {

// One-workgroup fronts.  A panel of 16 pivot columns is factored by waves that
// each hold the pivot rows in 16 lanes and rows of their own in the others; there
// is no second round, so the smallest workgroup must hold every row of the front.
constexpr int kCholWave = 64;
constexpr int kRowsPerWave = kCholWave - 16;
constexpr int kFactorThreads[] = {256, 512};   // workgroups of the factor kernel by variant
constexpr int kSolveThreads = 256;             // of the one-workgroup solves: a thread per column
// first and last + 1 of the rows below the pivot rows kb that a wave holds
// (wave 0 also stores the pivot rows)
constexpr int panel_wave_begin(int kb, int wave) { return kb + kRowsPerWave * wave + 16; }
constexpr int panel_wave_end(int kb, int wave) { return kb + kRowsPerWave * wave + kCholWave; }
constexpr int panel_rows(int threads) { return panel_wave_end(0, threads / kCholWave - 1); }

// Shared memory of a one-workgroup front: the packed lower triangle of one more
// row, the fused forward solve's.
constexpr size_t front_bytes(int64_t rows) { return (size_t)((rows + 1) * (rows + 2) / 2) * sizeof(double); }
constexpr bool one_workgroup_front(int64_t rows, size_t lds) {
    return front_bytes(rows) <= lds && rows + 1 <= panel_rows(kFactorThreads[0]);
}
// And of its solves: the panel, the solution of the rows, two vectors of its columns.
constexpr size_t front_solve_bytes(int64_t rows, int64_t w) {
    return (size_t)(rows * (w | 1) + rows + 2 * w) * sizeof(double);
}
constexpr bool one_workgroup_solve(int64_t rows, int64_t w, size_t lds) {
    return front_solve_bytes(rows, w) <= lds && w <= kSolveThreads;
}

// Large fronts.

constexpr int kPanelRowWaves = 4;                  // waves of a panel launch that solve rows, 16 rows each
constexpr int kRowBlock = 16 * kPanelRowWaves;     // rows below a panel per workgroup

// First of the 16 rows whose panel entries a wave of k_big_panel loads, columns
// [kb, kb + pw) of a front, row block b.  Waves 1 .. kPanelRowWaves solve theirs;
// wave 0 solves none and loads the first wave's, as it takes the same
// instructions: counted from its own number they began 16 rows before the block,
// before the front's storage where a front has fewer than 16 columns.
constexpr int panel_first_row(int kb, int pw, int b, int wave) {
    return kb + pw + b * kRowBlock + 16 * (wave >= 1 ? wave - 1 : 0);
}

}  // namespace nmpc
