// Threads that take compute units from ResLease (no device): prints "ok" or what
// went wrong.
#include "res_lease.hpp"

#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <thread>
#include <vector>

int main(int argc, char **) {
    if (argc > 1) {   // the process ends while a thread waits
        auto *all = new cuth::ResLease;   // (held to the end)
        (void)all->acquire(0, 256, 256);
        std::thread([] {
            cuth::ResLease more;
            (void)more.acquire(0, 8, 256);
        }).detach();
        std::this_thread::sleep_for(std::chrono::milliseconds(200));
        std::printf("ok\n");
        std::fflush(stdout);
        std::exit(0);
    }
    constexpr int kUnits = 256, kThreads = 8, kTurns = 400;
    std::atomic<int> held{0}, wide{0}, together{0}, over{0}, refused{0};
    std::vector<std::thread> threads;
    for (int t = 0; t < kThreads; ++t)
        threads.emplace_back([&, t] {
            std::mt19937 rng(t);
            const int widths[] = {1, 8, 60, 128, 200, 256, 300};   // (more than there are: all of them)
            for (int q = 0; q < kTurns; ++q) {
                const int w = widths[rng() % 7], need = std::min((w + 7) / 8 * 8, kUnits);
                cuth::ResLease lease;
                if (!lease.acquire(0, w, kUnits)) ++refused;
                const int now = held += need;
                if (now > kUnits) ++over;
                if (now > need) ++together;
                if (need == kUnits) ++wide;
                std::this_thread::sleep_for(std::chrono::microseconds(rng() % 50));
                held -= need;
            }
        });
    for (auto &t : threads) t.join();
    cuth::ResLease none;
    if (over || refused || !together || !wide || none.acquire(-1, 8, kUnits) || none.acquire(64, 8, kUnits))
        std::printf("over %d refused %d together %d wide %d\n", over.load(), refused.load(), together.load(), wide.load());
    else
        std::printf("ok\n");
    return 0;
}
