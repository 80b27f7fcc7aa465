// Index rules of the front kernels that a program without a device can check:
// plain constant expressions, the same on the host and in the kernels.
#pragma once

namespace nmpc {

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
