// Which on-chip preconditioners (launch_cheb_res) may run on a device at once.
#pragma once

#include <algorithm>
#include <condition_variable>
#include <cstdint>
#include <mutex>

namespace cuth {

// The compute units of a device, shared by the solves of the process.  All tiles of
// an on-chip launch must run at the same time, so such launches of different
// streams may be in flight together only if the device has a unit for each of
// their workgroups.  A solve enters with the workgroups of its widest launch, in
// whole rows of 8 (workgroups go to the 8 XCDs in turn), takes that many units for
// each run of launches that it enqueues and then waits for, and gives them back.  Who
// finds them taken waits, in the order of arrival, so that a call computes the same
// whatever other threads do.  Where the solves under way want more than there are
// (crowded), they take turns of a few iterations: a small solve does not wait for
// the end of a long one.  Ordinary launches need no units: they end by themselves.
// While it holds units a thread waits for its own launches only.
class ResLease {
public:
    ResLease() = default;
    ResLease(const ResLease &) = delete;
    ResLease &operator=(const ResLease &) = delete;
    ~ResLease() {
        give();
        if (!pool_) return;
        std::lock_guard<std::mutex> lock(pool_->mu);
        pool_->wanted -= need_;
    }
    // A solve with launches of up to `width` workgroups begins (false: a device out of
    // range).
    bool enter(int device, int width, int units) {
        // (never destroyed: a thread may still wait here when the process ends)
        static Pool *const pools = new Pool[kDevices];
        if (pool_ || device < 0 || device >= kDevices || units <= 0) return false;
        pool_ = &pools[device];
        need_ = std::min((width + 7) / 8 * 8, units);
        units_ = units;
        std::lock_guard<std::mutex> lock(pool_->mu);
        pool_->wanted += need_;
        return true;
    }
    bool entered() const { return pool_ != nullptr; }
    // Waits for the units (nothing if they are held already).
    void take() {
        if (!pool_ || held_) return;
        std::unique_lock<std::mutex> lock(pool_->mu);
        const uint64_t ticket = pool_->arrived++;
        pool_->freed.wait(lock, [&] { return pool_->serving == ticket && pool_->used + need_ <= units_; });
        pool_->used += need_;
        ++pool_->serving;
        held_ = true;
        pool_->freed.notify_all();
    }
    void give() {
        if (!held_) return;
        std::lock_guard<std::mutex> lock(pool_->mu);
        pool_->used -= need_;
        held_ = false;
        pool_->freed.notify_all();
    }
    // Not all solves under way can hold their units at once.
    bool crowded() const {
        if (!pool_) return false;
        std::lock_guard<std::mutex> lock(pool_->mu);
        return pool_->wanted > units_;
    }

private:
    struct Pool {
        std::mutex mu;
        std::condition_variable freed;
        int64_t wanted = 0;
        int used = 0;
        uint64_t arrived = 0, serving = 0;
    };
    static constexpr int kDevices = 64;
    Pool *pool_ = nullptr;
    int need_ = 0, units_ = 0;
    bool held_ = false;
};

}  // namespace cuth
