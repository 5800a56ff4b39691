// Threads that share compute units through ResLease (no device): prints "ok" or what
// went wrong.
#include "res_lease.hpp"

#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <thread>
#include <vector>

constexpr int kUnits = 256, kThreads = 8, kTurns = 400;

static int need_of(int width) { return std::min((width + 7) / 8 * 8, kUnits); }

// Solves of random widths, each of a few turns.
static int share() {
    std::atomic<int> held{0}, wide{0}, together{0}, over{0}, refused{0}, crowded{0};
    std::vector<std::thread> threads;
    for (int t = 0; t < kThreads; ++t)
        threads.emplace_back([&, t] {
            std::mt19937 rng(t);
            const int widths[] = {1, 8, 60, 128, 200, 256, 300};   // (more than there are: all of them)
            for (int q = 0; q < kTurns / 4; ++q) {
                const int w = widths[rng() % 7], need = need_of(w);
                cuth::ResLease lease;
                if (!lease.enter(0, w, kUnits)) ++refused;
                for (int turn = 0; turn < 4; ++turn) {
                    lease.take();
                    lease.take();   // (held already)
                    const int now = held += need;
                    if (now > kUnits) ++over;
                    if (now > need) ++together;
                    if (need == kUnits) ++wide;
                    if (lease.crowded()) ++crowded;
                    std::this_thread::sleep_for(std::chrono::microseconds(rng() % 50));
                    held -= need;
                    if (turn < 3) lease.give();   // (the last by the destructor)
                }
            }
        });
    for (auto &t : threads) t.join();
    cuth::ResLease none, alone;
    alone.enter(0, 256, kUnits);
    const bool ok = !over && !refused && together && wide && crowded && !alone.crowded() &&
                    !none.enter(-1, 8, kUnits) && !none.enter(64, 8, kUnits);
    if (!ok)
        std::printf("over %d refused %d together %d wide %d crowded %d\n", over.load(), refused.load(),
                    together.load(), wide.load(), crowded.load());
    return ok;
}

// A solve of many turns on all units, and a small one: it has its turn after the one
// under way, and then sees that it need not hurry alone.
static int in_turn() {
    std::atomic<int> turns{0};
    std::atomic<bool> stop{false};
    std::thread big([&] {
        cuth::ResLease lease;
        lease.enter(1, kUnits, kUnits);
        while (!stop) {
            lease.take();
            ++turns;
            std::this_thread::sleep_for(std::chrono::milliseconds(2));
            lease.give();
        }
    });
    while (turns < 3) std::this_thread::yield();
    int worst = 0;
    {
        cuth::ResLease small;
        small.enter(1, 8, kUnits);
        for (int q = 0; q < 20; ++q) {
            const int before = turns;
            small.take();
            worst = std::max(worst, turns - before);
            small.give();
        }
    }
    stop = true;
    big.join();
    // (the turn under way, and at most one that began before the small solve's ticket)
    if (worst > 2) std::printf("%d turns before the small solve's\n", worst);
    return worst <= 2;
}

int main(int argc, char **) {
    if (argc > 1) {   // the process ends while a thread waits
        auto *all = new cuth::ResLease;   // (held to the end)
        all->enter(0, kUnits, kUnits);
        all->take();
        std::thread([] {
            cuth::ResLease more;
            more.enter(0, 8, kUnits);
            more.take();
        }).detach();
        std::this_thread::sleep_for(std::chrono::milliseconds(200));
        std::printf("ok\n");
        std::fflush(stdout);
        std::exit(0);
    }
    if (share() && in_turn()) std::printf("ok\n");
    return 0;
}
