// Which on-chip preconditioners (launch_cheb_res) may run on a device at once.
#pragma once

#include <algorithm>
#include <condition_variable>
#include <cstdint>
#include <mutex>

namespace cuth {

// Compute units of a device held by one solve.  All tiles of an on-chip launch
// must run at the same time, so the solves of the process that use such launches
// share the device's units: each takes as many as its widest launch has
// workgroups, in whole rows of 8 (workgroups go to the 8 XCDs in turn), and waits
// where they are taken, in the order of arrival.  So a call computes the same
// whatever other threads do; ordinary launches of theirs end by themselves and
// hold up nothing.  Who holds units must not wait for another thread's solve: the
// caller's earlier work on the stream is waited for first, and a solve waits for
// its own launches before it returns and gives the units back.
class ResLease {
public:
    ResLease() = default;
    ResLease(const ResLease &) = delete;
    ResLease &operator=(const ResLease &) = delete;
    ~ResLease() {
        if (!pool_) return;
        std::lock_guard<std::mutex> lock(pool_->mu);
        pool_->used -= held_;
        pool_->freed.notify_all();
    }
    // Waits for `width` of the device's `units` (false: a device out of range).
    bool acquire(int device, int width, int units) {
        // (never destroyed: a thread may still wait here when the process ends)
        static Pool *const pools = new Pool[kDevices];
        if (device < 0 || device >= kDevices || units <= 0) return false;
        Pool &p = pools[device];
        const int need = std::min((width + 7) / 8 * 8, units);
        std::unique_lock<std::mutex> lock(p.mu);
        const uint64_t ticket = p.arrived++;
        p.freed.wait(lock, [&] { return p.serving == ticket && p.used + need <= units; });
        p.used += need;
        ++p.serving;
        p.freed.notify_all();
        pool_ = &p;
        held_ = need;
        return true;
    }

    bool held() const { return pool_ != nullptr; }

private:
    struct Pool {
        std::mutex mu;
        std::condition_variable freed;
        int used = 0;
        uint64_t arrived = 0, serving = 0;
    };
    static constexpr int kDevices = 64;
    Pool *pool_ = nullptr;
    int held_ = 0;
};

}  // namespace cuth
