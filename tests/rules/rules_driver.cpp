// Checks launch_rules.hpp on the CPU. Each check prints what failed.
#include <cstdio>
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

}  // namespace

int main() {
    persistent_rows();
    tiles();
    std::puts(failed ? "failed" : "ok");
    return failed ? 1 : 0;
}
