// Checks residency.hpp on the CPU: whatever runs are admitted together, every
// one of their blocks finds room under any placement that the hardware might
// choose, and runs are admitted in order.
#include <atomic>
#include <cstdio>
#include <random>
#include <thread>
#include <vector>

#include "../../paper_1908_01719_amd/csrc/residency.hpp"

using namespace dmri;

namespace {

struct Run {
    int64_t n;
    bool half;
    std::vector<int> cu;  // CU of each placed block (xcd * cus + index)
};

// Deals a run's blocks to the XCDs in turn from a random one on; each lies on
// a random CU of its XCD with room. free[cu] in half CUs. False: no room.
bool place(Run& r, std::vector<int>& free, int cus, std::mt19937& rng) {
    const int need = r.half ? 1 : 2;
    const int first = static_cast<int>(rng() % kXcds);
    for (int64_t b = 0; b < r.n; ++b) {
        const int xcd = static_cast<int>((first + b) % kXcds);
        std::vector<int> ok;
        for (int c = 0; c < cus; ++c)
            if (free[xcd * cus + c] >= need) ok.push_back(xcd * cus + c);
        if (ok.empty()) return false;
        const int cu = ok[rng() % ok.size()];
        free[cu] -= need;
        r.cu.push_back(cu);
    }
    return true;
}

bool placements(int cus, unsigned seed) {
    std::mt19937 rng(seed);
    std::vector<int> free(kXcds * cus, 2);
    std::vector<Run> in;
    ResidentBlocks used;
    int64_t joined = 0, together = 0;
    for (int step = 0; step < 400; ++step) {
        Run r{1 + static_cast<int64_t>(rng() % (kXcds * cus)), (rng() & 1) != 0, {}};
        if (rng() % 3 == 0) r.n = 1 + r.n % 20;
        const ResidentBlocks rb = resident_blocks(r.n, r.half);
        while (!may_join(used, rb, cus)) {  // a random run ends
            const size_t k = rng() % in.size();
            for (int cu : in[k].cu) free[cu] += in[k].half ? 1 : 2;
            const ResidentBlocks o = resident_blocks(in[k].n, in[k].half);
            used.whole -= o.whole;
            used.half -= o.half;
            in.erase(in.begin() + static_cast<long>(k));
        }
        if (!place(r, free, cus, rng)) {
            std::printf("no room: %lld %s blocks beside %zu runs, %d CUs an XCD\n",
                        static_cast<long long>(r.n), r.half ? "half" : "whole", in.size(), cus);
            return false;
        }
        used.whole += rb.whole;
        used.half += rb.half;
        in.push_back(r);
        ++joined;
        together += in.size() > 1;
    }
    return joined == 400 && together > 40;  // runs do share the device
}

// A run of the whole device asks while small ones keep coming: it is admitted
// before they end, and none of them runs beside it.
bool in_order() {
    constexpr int kThreads = 4, kRuns = 3000, kCus = 32;
    ResidencyGate gate;
    std::atomic<int> done{0}, inside{0}, at{-1};
    std::atomic<bool> over{false};
    std::vector<std::thread> th;
    for (int t = 0; t < kThreads; ++t)
        th.emplace_back([&] {
            const ResidentBlocks rb = resident_blocks(24, true);
            for (int i = 0; i < kRuns; ++i) {
                gate.enter(rb, kCus);
                ++inside;
                std::this_thread::yield();
                --inside;
                gate.leave(rb);
                ++done;
            }
        });
    std::thread big([&] {
        const ResidentBlocks rb = resident_blocks(kXcds * kCus, false);
        while (done < 100) std::this_thread::yield();
        gate.enter(rb, kCus);
        at = done.load();
        std::this_thread::yield();
        if (inside != 0) over = true;  // somebody ran beside a run of the whole device
        gate.leave(rb);
    });
    for (auto& t : th) t.join();
    big.join();
    std::printf("whole-device run admitted after %d of %d small runs\n", at.load(), kThreads * kRuns);
    return done == kThreads * kRuns && !over && at < kThreads * kRuns;
}

}  // namespace

int main() {
    bool ok = true;
    for (int cus : {4, 32, 38})
        for (unsigned seed = 1; seed <= 20; ++seed) ok = placements(cus, seed) && ok;
    ok = in_order() && ok;
    std::puts(ok ? "ok" : "failed");
    return ok ? 0 : 1;
}
