// Which persistent solves may be in flight together on one device. Host only.
//
// The blocks of a persistent solve wait for each other, so every block of
// every such launch in flight has to be resident. Blocks are dealt to the 8
// XCDs in turn, hence n blocks put at most ceil(n / 8) on any one, and there
// each of them lies on any CU with room for it:
//  - a block that needs a CU to itself ("whole") finds one as long as the
//    whole blocks and the CUs that smaller blocks may have touched together
//    are no more than the XCD's CUs: smaller blocks count a CU each;
//  - with no whole block in flight, two smaller blocks share a CU.
// Both hold wherever the hardware puts the blocks. Runs are admitted in the
// order in which they ask, so one that needs the whole device does not wait
// behind later, smaller ones for ever.
#pragma once

#include <algorithm>
#include <condition_variable>
#include <cstdint>
#include <mutex>

namespace dmri {

constexpr int kXcds = 8;

// Blocks per XCD of the runs admitted on a device, or of one run.
struct ResidentBlocks {
    int64_t whole = 0, half = 0;
};

// A run of n blocks, two of which fit a CU (half) or not.
inline ResidentBlocks resident_blocks(int64_t n, bool half) {
    const int64_t per_xcd = (n + kXcds - 1) / kXcds;
    return half ? ResidentBlocks{0, per_xcd} : ResidentBlocks{per_xcd, 0};
}

// Whether a run may join the admitted ones on XCDs of `cus` CUs. A run alone
// always may: its own plan has checked that it fits.
inline bool may_join(const ResidentBlocks& in, const ResidentBlocks& run, int64_t cus) {
    if (in.whole + in.half == 0) return true;
    const int64_t w = in.whole + run.whole, h = in.half + run.half;
    return w == 0 ? h <= 2 * cus : w + h <= cus;
}

// Admission on one device, for runs of any threads.
class ResidencyGate {
public:
    void enter(const ResidentBlocks& run, int64_t cus) {
        std::unique_lock<std::mutex> lock(mu_);
        const uint64_t ticket = next_++;
        cv_.wait(lock, [&] { return ticket == head_ && may_join(in_, run, cus); });
        ++head_;
        in_.whole += run.whole;
        in_.half += run.half;
        lock.unlock();
        cv_.notify_all();  // the next in line may fit beside this one
    }
    void leave(const ResidentBlocks& run) {
        {
            std::lock_guard<std::mutex> lock(mu_);
            in_.whole -= run.whole;
            in_.half -= run.half;
        }
        cv_.notify_all();
    }

private:
    std::mutex mu_;
    std::condition_variable cv_;
    uint64_t next_ = 0, head_ = 0;
    ResidentBlocks in_;
};

}  // namespace dmri
