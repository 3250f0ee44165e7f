// Rules on sizes that the host and the kernels share. No device code, so that
// they can be checked on the CPU.
#pragma once

#include <algorithm>
#include <cstdint>

namespace dmri {

// Persistent solver: one kernel keeps a (row, system) element in every lane's
// registers, the other its rows in memory. All blocks of all tiles are resident
// together, at most one per CU.
constexpr int kPersistBlock = 512;

struct PersistPlan {
    bool lanes;       // an element per lane
    int32_t threads;  // per block
    int32_t nbt;      // blocks per tile
};

// False where it cannot run: a tile of `rows` rows of S systems must stay below
// 2^31 bytes (its directions are addressed through one buffer resource).
inline bool persist_plan(int64_t rows, int64_t S, int64_t n_tiles, int64_t n_cu, PersistPlan& p) {
    if (rows * S * 16 >= (int64_t(1) << 31)) return false;
    const int64_t per_wave = std::max<int64_t>(1, 64 / S);
    const int64_t groups = (rows + per_wave - 1) / per_wave;  // wavefronts
    const int64_t most = n_cu / n_tiles;                      // blocks a tile can have
    if (most < 1) return false;
    // One element per lane: 4 wavefronts a block while that fits (the gathers
    // of a block's wavefronts share its CU's L1), else 8.
    p.lanes = true;
    p.threads = (groups + 3) / 4 <= most ? kPersistBlock / 2 : kPersistBlock;
    if ((groups + p.threads / 64 - 1) / (p.threads / 64) > most) {
        p.lanes = false;
        p.threads = kPersistBlock;
    }
    const int64_t waves = p.threads / 64;
    p.nbt = static_cast<int32_t>(std::min(most, (groups + waves - 1) / waves));
    return true;
}

// Whether every block reads the `vals` sums of all blocks itself (one hop), or
// each value is added by one block and its total read in turn (two hops, but
// nbt * vals words read in all instead of by every block).
constexpr bool persist_direct(int nbt, int vals) { return nbt * vals <= 2048; }

// Its kernel with rows in memory: the rows of wavefront `wave` of block `block`
// start here, and its next ones are a step further. `waves` is what the blocks
// of the launch really have.
constexpr int persist_first_row(int block, int waves, int wave, int rows_per_wave) {
    return (block * waves + wave) * rows_per_wave;
}
constexpr int persist_row_step(int blocks, int waves, int rows_per_wave) {
    return blocks * waves * rows_per_wave;
}

// Blocks per XCD that sweep a part of `chunks` chunks in a launch whose tiles
// (of S systems) are split into n_parts parts; bpx is option blocks_per_xcd,
// whose default value stands for the rule below and every other for itself.
// Chunks are the 8 to 32 rows of a block's sweep (GMRES's kernels: 16 to 128).
//
// By default one generation of resident blocks (32 CUs x 4 blocks): the fewest
// partials to add, no tail of a last, nearly empty generation, and blocks that
// keep together and share their gathers in the XCD's L2. A tile split over 4
// or 8 XCDs wants that at any length (chunks a part; ms with 128 / 512 / 1,024
// blocks, 10 to 3 steps):
//   200 pairs mixed, 48^3  3.7k 164 / 175 / 183   66^3  9.5k 556 / 574 / 588
//    24 pairs FP64,  57^3  3.1k 110 / 117 / 130   90^3 11.9k 505 / 521 / 538
//    64 pairs FP64,  64^3  4.4k 209 / 218 / 226   80^3  8.4k 496 / 510 / 519
// Where an XCD sweeps a whole tile or half of one, long parts let the blocks
// drift apart, and more of them cover that:
//   200 pairs FP64,  48^3  7.4k 279 / 279 / 276   57^3 12.3k 556 / 550 / 539
//  1024 pairs FP64,  36^3  6.5k 390 / 387 / 380   512 pairs, 48^3 14.9k 622 / 612 / 604
// so there the line lies at 4,096 chunks, and at twice that for the paired
// tiles of mixed precision, which gather half the bytes a row (512 pairs at
// 40^3, 4.4k chunks, with 128 / 512 blocks: 163 / 170; 1,024 at 66^3, 38.1k,
// with 128 / 512 / 1,024: 1,693 / 1,648 / 1,637). 512 is best nowhere.
constexpr int32_t kDefaultBlocks = 512;
constexpr int32_t kResidentBlocks = 128;
constexpr int32_t kResidentChunks = 4096;

inline int32_t blocks_per_xcd_of(int32_t bpx, int32_t chunks, int32_t n_parts, int32_t S) {
    int32_t cap = bpx;
    if (bpx == kDefaultBlocks) {
        const int32_t line = S > 64 ? 2 * kResidentChunks : kResidentChunks;
        cap = n_parts >= 4 || chunks <= line ? kResidentBlocks : 8 * kResidentBlocks;
    }
    return std::max(1, std::min(cap, chunks));
}

// Row queues (option queue): whether wavefront `wave` of block `block` of
// `blocks` takes rows of an item of `rows` rows in n grabs. One wavefront a
// grab does, and one for four passes over R rows each; more of them only queue
// up at the item's counter to find it spent, and with few row slots an item has
// blocks enough for several times as many. Counted across the blocks, so that
// all CUs take part; callers turn the wavefronts from item to item, so that an
// XCD's next item starts beside the last. FP64 at 26^3, 10 steps: 12 pairs
// 36.8 ms with every wavefront, 28.0 this way; 32 pairs 46.6 and 38.3; 16 pairs
// 35.4 and 28.3; 173 pairs in 8-wide tiles 155 without the turn, 131 with it.
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
// threads over every 1024 / S-th partial (10 steps at 26^3: 40 pairs 230 ms as
// two 32-wide tiles, 802 ms as one of 64; 20 pairs 131 ms as two of 16, 251 ms
// as one of 32; 12 pairs 86 ms as two of 8, 115 ms as one of 16).
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
