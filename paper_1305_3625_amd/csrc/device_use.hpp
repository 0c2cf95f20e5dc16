// What this process has in flight on each device, by which a solve chooses
// what it runs.
//
// A resident solve keeps its CUs for the whole solve, and a good part of their
// registers.  A pass whose workgroups do not fit beside it waits for its end
// with every launch (workgroups go to the XCDs in turn and do not move), and
// loses the race against the next resident solve again.  When resident solves
// took any free XCD, passes beside them starved (each per second, with that
// rule -> with the one below; threads that solve or multiply without a pause):
//   mixed L = 4096 solves beside two threads of L = 128 solves   1.2 -> 27
//   preconditioned L = 1024 beside FP64 L = 512                   15 -> 600
//   FP64 L = 512, four threads together                          640 -> 1,150
//   preconditioned FP64 L = 512, four threads                  1,240 -> 2,210
//   FP64 products of L = 2048 beside FP64 L = 512                315 -> 7,100
// The passes above M = 1024 need what a resident workgroup takes (70 to 144 KB
// of LDS a workgroup, or four waves a SIMD of 121 registers for their
// barrier), so no resident solve starts beside them.  The passes up to M =
// 1024 take at most 220 registers of a SIMD (the FP64 column pass of M = 1024)
// and 70 KB; they fit, or nearly fit, beside the resident kernel up to M = 512
// and beside the plain FP32 one of M = 1024 (272 of 512 registers), which
// therefore start beside solves, servers and products of that size: those run
// as fast as beside passes, and the resident solve twice as fast (L = 128 mixed
// beside a server of eight mixed L = 512: 2,390 and 1,360 per second, as passes
// 930 and 1,390; beside FP64 products of L = 512: 2,530 and 46,000, as passes
// 1,050 and 45,400).  At M = 1024 in FP64 or preconditioned the resident kernel
// takes 290 to 512 registers and runs alone.
//
// Grid-wide barriers: the sum of the shares of the device that the grids in
// flight take is kept to one, a grid that fills the device asks for it alone,
// and barriers above the resident kernel's grids stay away from resident
// solves: no two grids then each hold a part of the device that the other
// waits for (such a wait ends after 20 ms, and the plan keeps the separate
// update).  Two threads of preconditioned L = 2048 solves: 310 solves a
// second with one of them at the barrier, 355 with neither.
#pragma once
#include <mutex>

namespace fftcg {

class DeviceUse {
public:
    enum Kind { SMALL, LARGE };  // passes of M <= 1024, above
    static Kind kind(int M) { return M <= 1024 ? SMALL : LARGE; }

    explicit DeviceUse(int device) : dev_(device >= 0 && device < kDevices ? device : -1) {}
    ~DeviceUse() { end(); }
    DeviceUse(const DeviceUse&) = delete;
    DeviceUse& operator=(const DeviceUse&) = delete;

    // A resident solve on `xcds` XCDs (1 or 8) that may start beside the small
    // passes of `beside` solves and servers: whether it may start.
    bool resident(int xcds, int beside) {
        if (dev_ < 0) return false;
        std::lock_guard<std::mutex> lk(mu_);
        Device& d = use_[dev_];
        if (d.large > 0 || d.small > beside) return false;
        if (xcds == 8) {
            if (d.xcds == 0) mask_ = 0xff;
        } else {
            for (int i = 0; i < 8 && !mask_; ++i)
                if (!(d.xcds & (1u << i))) mask_ = 1u << i;
        }
        d.xcds |= mask_;
        return mask_ != 0;
    }
    int first_xcd() const { return mask_ ? __builtin_ctz(mask_) : 0; }

    // Launched passes; fits: grids of their barrier that the device holds at
    // once (0: no barrier).  Whether they may use the barrier.
    bool passes(Kind kind, int fits) {
        if (dev_ < 0) return fits > 0;
        std::lock_guard<std::mutex> lk(mu_);
        Device& d = use_[dev_];
        const bool alone = d.small + d.large == 0;
        passes_ = true;
        kind_ = kind;
        (kind == SMALL ? d.small : d.large) += 1;
        if (fits <= 0 || (fits == 1 && !alone) || (kind == LARGE && d.xcds != 0) ||
            d.share + 1.0 / fits > 1.0 + 1e-9)
            return false;
        share_ = 1.0 / fits;
        d.share += share_;
        return true;
    }
    void end() {
        if (!mask_ && !passes_) return;
        std::lock_guard<std::mutex> lk(mu_);
        Device& d = use_[dev_];
        d.xcds &= ~mask_;
        if (passes_) (kind_ == SMALL ? d.small : d.large) -= 1;
        d.share -= share_;
        if (d.small + d.large == 0) d.share = 0.0;  // (no rounding left behind)
        mask_ = 0;
        passes_ = false;
        share_ = 0.0;
    }

private:
    static constexpr int kDevices = 64;
    struct Device {
        unsigned xcds;  // XCDs that resident solves hold, a bit each, by their hardware number
        int small;      // solves that run the passes, and servers at work,
        int large;      // by kind
        double share;   // of the device, by grids with a barrier
    };
    static inline std::mutex mu_;
    static inline Device use_[kDevices];
    int dev_;
    unsigned mask_ = 0;
    bool passes_ = false;
    Kind kind_ = LARGE;
    double share_ = 0.0;
};

}  // namespace fftcg
