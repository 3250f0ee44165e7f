// Checks launch_rules.hpp on the CPU. Each check prints what failed.
#include <cstdio>
#include <numeric>
#include <vector>

#include "../../paper_1908_01719_amd/csrc/launch_rules.hpp"

using namespace dmri;

namespace {

int failed = 0;

#define CHECK(cond, ...)                            \
    do {                                            \
        if (!(cond)) {                              \
            std::printf("%s:%d: ", #cond, __LINE__); \
            std::printf(__VA_ARGS__);               \
            std::puts("");                          \
            ++failed;                               \
        }                                           \
    } while (0)

// Every row of a tile belongs to one wavefront, whatever a block's size: a plan
// of 256-thread blocks that is given fewer blocks runs this kernel too.
void persistent_rows() {
    for (int waves : {1, 4, 8})
        for (int blocks : {1, 3, 71, 256})
            for (int R : {1, 2, 4, 8})
                for (int rows : {1, 7, 1000, 17576}) {
                    std::vector<int> seen(static_cast<size_t>(rows), 0);
                    for (int b = 0; b < blocks; ++b)
                        for (int w = 0; w < waves; ++w)
                            for (int l = 0; l < R; ++l)
                                for (int row = persist_first_row(b, waves, w, R) + l; row < rows;
                                     row += persist_row_step(blocks, waves, R))
                                    ++seen[static_cast<size_t>(row)];
                    int bad = 0;
                    for (int s : seen) bad += s != 1;
                    CHECK(bad == 0, "%d of %d rows, %d blocks of %d wavefronts, %d rows each", bad,
                          rows, blocks, waves, R);
                }
}

// The tile width of every batch: GMRES and the persistent solver fill their
// tiles; the chunked CG and COCG take one tile up to 64 systems.
void tiles() {
    for (int64_t n = 1; n <= 200; ++n) {
        const int filled = n >= 64 ? 64 : n >= 32 ? 32 : n >= 16 ? 16 : 8;
        const int one = n <= 8 ? 8 : n <= 16 ? 16 : n <= 32 ? 32 : 64;
        CHECK(tile_of_batch(n, false, true) == filled, "GMRES, %d systems", int(n));
        CHECK(tile_of_batch(n, true, false) == filled, "persistent, %d systems", int(n));
        CHECK(tile_of_batch(n, false, false) == one, "chunked, %d systems", int(n));
    }
}

// Row queues: never more wavefronts than grabs, never none, and spread over the
// blocks.
void queue_takers() {
    for (int blocks : {1, 3, 128, 512})
        for (int R : {1, 2, 4, 8})
            for (int rows : {1, 7, 300, 2200, 100000})
                for (int grab : {1, 4, 16}) {
                    const int per = grab * 2 * R, n = (rows + per - 1) / per;
                    const int want = std::min(std::min(n, (rows + 4 * R - 1) / (4 * R)), 4 * blocks);
                    int takers = 0, most = 0, least = 1 << 30;
                    for (int b = 0; b < blocks; ++b) {
                        int here = 0;
                        for (int w = 0; w < 4; ++w) here += queue_taker(b, blocks, w, n, rows, R);
                        takers += here;
                        most = std::max(most, here);
                        least = std::min(least, here);
                    }
                    CHECK(takers == want && takers >= 1, "%d takers of %d grabs, %d rows, %d blocks",
                          takers, n, rows, blocks);
                    CHECK(most - least <= 1, "%d to %d takers a block", least, most);
                }
}

// Blocks per XCD: the default on both sides of its lines, a count that is asked
// for taken as it is, and launches restricted to some tiles (up to 8 parts a
// tile) never with more blocks than the batch's own, for which the partial sums
// have room.
void blocks() {
    constexpr int kAuto = kDefaultBlocks;
    for (int S : {8, 64, 128})
        for (int chunks : {1, 127, 128, 4096, 4097, 8192, 8193, 40000}) {
            const int line = S == 128 ? 8192 : 4096;
            for (int parts : {1, 2})
                CHECK(blocks_per_xcd_of(kAuto, chunks, parts, S) ==
                          std::min(chunks, chunks <= line ? 128 : 1024),
                      "%d chunks, %d parts, tiles of %d", chunks, parts, S);
            for (int parts : {4, 8})
                CHECK(blocks_per_xcd_of(kAuto, chunks, parts, S) == std::min(chunks, 128),
                      "%d chunks, %d parts, tiles of %d", chunks, parts, S);
            for (int bpx : {1, 3, 128, 256, 511, 513, 1024, 4096})
                CHECK(blocks_per_xcd_of(bpx, chunks, 2, S) == std::min(bpx, chunks), "%d asked", bpx);
        }
    for (int bpx : {kAuto, 64, 4096})
        for (int S : {8, 64, 128}) {
            const int chunk_rows = S == 8 ? 32 : 8;
            for (int tiles = 1; tiles <= 33; ++tiles)
                for (int rows = 50; rows < 3000000; rows = rows * 5 / 4 + 1) {
                    const int parts = 8 / std::gcd(tiles, 8);
                    auto of = [&](int n_parts) {
                        const int pr = (rows + n_parts - 1) / n_parts;
                        return blocks_per_xcd_of(bpx, (pr + chunk_rows - 1) / chunk_rows, n_parts, S);
                    };
                    for (int n = 1; n < tiles; ++n) {
                        const int p = std::max(parts, 8 / std::gcd(n, 8));
                        CHECK(of(p) <= of(parts), "%d rows, %d of %d tiles", rows, n, tiles);
                    }
                }
        }
}

// The persistent kernel that a batch runs on 256 CUs: the parameter rows of the
// GPU tests of the persistent solver reach each of them, with both exchanges
// (direct: all blocks read all words; sums of 2 and 3 values a system).
void persistent_variants() {
    struct {
        int rows, S, tiles;
        bool lanes;
        int threads, nbt;
        bool direct;
    } const table[] = {
        {312, 8, 1, true, 256, 10, true},      {312, 16, 1, true, 256, 20, true},
        {312, 64, 1, true, 256, 78, false},    {312, 32, 2, true, 256, 39, false},
        {2160, 8, 3, true, 256, 68, true},     {4928, 32, 1, false, 512, 256, false},
        {4928, 64, 1, false, 512, 256, false}, {9440, 64, 1, false, 512, 256, false},
        {9440, 8, 1, true, 512, 148, false},   {6768, 16, 1, true, 512, 212, false},
        {6768, 8, 2, true, 512, 106, false},   {6768, 8, 3, false, 512, 85, true},
        {19864, 8, 1, false, 512, 256, false},
    };
    for (const auto& t : table) {
        PersistPlan p{};
        CHECK(persist_plan(t.rows, t.S, t.tiles, 256, p), "%d rows", t.rows);
        CHECK(p.lanes == t.lanes && p.threads == t.threads && p.nbt == t.nbt,
              "%d rows, %d tiles of %d: lanes %d, %d threads, %d blocks", t.rows, t.tiles, t.S, p.lanes,
              p.threads, p.nbt);
        CHECK(persist_direct(p.nbt, 3 * t.S) == t.direct, "%d blocks, tiles of %d", p.nbt, t.S);
    }
    // Any batch: enough lanes or rows for all, never more blocks than CUs.
    for (int S : {8, 16, 32, 64})
        for (int tiles = 1; tiles * S <= 64; ++tiles)
            for (int n_cu : {32, 256, 304})
                for (int64_t rows = 1; rows < 200000; rows = rows * 9 / 8 + 1) {
                    PersistPlan p{};
                    CHECK(persist_plan(rows, S, tiles, n_cu, p), "%d rows", int(rows));
                    CHECK(p.nbt >= 1 && p.nbt * tiles <= n_cu, "%d blocks", p.nbt);
                    CHECK(!p.lanes || int64_t(p.nbt) * p.threads >= rows * S, "%d rows", int(rows));
                }
    PersistPlan p{};
    CHECK(!persist_plan(int64_t(1) << 21, 64, 1, 256, p), "a tile of 2^31 bytes");
    CHECK(!persist_plan(100, 8, 8, 4, p), "fewer CUs than tiles");
}

}  // namespace

int main() {
    persistent_variants();
    blocks();
    persistent_rows();
    tiles();
    queue_takers();
    std::puts(failed ? "failed" : "ok");
    return failed ? 1 : 0;
}
