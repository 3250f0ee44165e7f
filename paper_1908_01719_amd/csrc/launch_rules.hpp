// Rules on sizes that the host and the kernels share. No device code, so that
// they can be checked on the CPU.
#pragma once

#include <algorithm>
#include <cstdint>

namespace dmri {

// Persistent solver with its rows in memory: the rows of wavefront `wave` of
// block `block` start here, and its next ones are a step further. `waves` is
// what the blocks of the launch really have.
constexpr int persist_first_row(int block, int waves, int wave, int rows_per_wave) {
    return (block * waves + wave) * rows_per_wave;
}
constexpr int persist_row_step(int blocks, int waves, int rows_per_wave) {
    return blocks * waves * rows_per_wave;
}

}  // namespace dmri
