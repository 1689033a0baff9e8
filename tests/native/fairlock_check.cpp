// csrc/fairlock.h: while one thread takes the lock again and again, with
// nothing in between, another one that comes for it gets it within a turn or two
// (the median of 21 tries, so that a scheduler's pause does not matter), and no
// two threads have it at once.
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cstdio>
#include <thread>
#include <vector>

#include "fairlock.h"

#ifndef LOCK
#define LOCK hub::FairLock
#endif

int main() {
    LOCK lock;
    std::atomic<bool> stop{false};
    std::atomic<int> turns{0}, inside{0}, clashes{0};
    auto hold = [&](std::chrono::microseconds t) {
        if (inside.fetch_add(1) != 0) ++clashes;
        const auto end = std::chrono::steady_clock::now() + t;
        while (std::chrono::steady_clock::now() < end) {
        }
        inside.fetch_sub(1);
    };
    std::thread busy([&] {
        while (!stop) {
            lock.lock();
            hold(std::chrono::microseconds(1000));
            ++turns;
            lock.unlock();
        }
    });
    while (turns == 0) std::this_thread::yield();
    std::vector<int> waited;
    for (int k = 0; k < 21; ++k) {
        const int before = turns;
        lock.lock();
        waited.push_back(turns - before);
        hold(std::chrono::microseconds(100));
        lock.unlock();
        std::this_thread::sleep_for(std::chrono::microseconds(1500));
    }
    stop = true;
    busy.join();
    std::sort(waited.begin(), waited.end());
    std::printf("%s: waited for %d turns (median), %d at most, %d clashes\n",
                waited[10] <= 2 && clashes == 0 ? "ok" : "FAIL", waited[10], waited[20],
                clashes.load());
    return waited[10] <= 2 && clashes == 0 ? 0 : 1;
}
