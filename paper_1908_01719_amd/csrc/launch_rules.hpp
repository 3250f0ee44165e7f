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

// Row queues (option queue): whether wavefront `wave` of block `block` of
// `blocks` takes rows of an item of `rows` rows in n grabs. One wavefront a
// grab does, and one for four passes over R rows each; more of them only queue
// up at the item's counter to find it spent, and with few row slots an item has
// blocks enough for several times as many. Counted across the blocks, so that
// all CUs take part. FP64 at 26^3, 10 steps: 12 pairs 36.8 ms with every
// wavefront, 28.9 this way; 32 pairs 46.6 and 38.3; 16 pairs 35.4 and 28.8.
constexpr bool queue_taker(int block, int blocks, int wave, int n, int rows, int R) {
    const int by_rows = (rows + 4 * R - 1) / (4 * R);
    return wave * blocks + block < (n < by_rows ? n : by_rows);
}

// Tile width of a batch: the narrowest tile that holds all its systems, up to
// 64. One tile reads the matrix once where two half-filled tiles of half the
// width read it twice for the same padded batch, and a 64-wide tile's rows are
// wavefront-uniform (its SpMV stages their matrix entries in LDS). FP64,
// cylinder meshes, 30 steps: 40 pairs at 26^3 131.7 ms as two 32-wide tiles,
// 86.2 ms as one of 64 (40^3: 488 and 350 ms); 12 pairs at 26^3 78.2 ms as two
// of 8, 68.6 ms as one of 16. Mixed precision, 10 steps: 40 pairs at 40^3 104
// and 67 ms.
inline int auto_tile(int64_t n_sys) {
    for (int S = 8; S < 64; S *= 2)
        if (n_sys <= S) return S;
    return 64;
}

// The widest tile not wider than the batch, for solvers that one wide tile
// does not serve: the persistent solver and several-mesh batches, whose
// 64-wide tiles have no wavefront-uniform fast path (40 pairs at 12^3 in the
// persistent solver: 20.9 ms as two 32-wide tiles, 22.3 ms as one of 64), and
// GMRES, which adds the dot products of a tile in one block, each group of its
// threads over every 1024 / S-th partial (10 steps at 26^3: 40 pairs 217 ms as
// two 32-wide tiles, 790 ms as one of 64; 20 pairs 117 ms as two of 16, 237 ms
// as one of 32).
inline int auto_tile_filled(int64_t n_sys) {
    if (n_sys >= 64) return 64;
    if (n_sys >= 32) return 32;
    if (n_sys >= 16) return 16;
    return 8;
}

inline int tile_of_batch(int64_t n_sys, bool persistent, bool gmres) {
    return persistent || gmres ? auto_tile_filled(n_sys) : auto_tile(n_sys);
}

}  // namespace dmri
