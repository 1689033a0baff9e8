// A lock whose waiters get it in the order in which they came.  A solve that
// stays on the chip takes it for every one of its launches, with next to
// nothing in between: with std::mutex it had it again before a thread that
// waits was awake, and a short solve of another thread waited for the whole of
// a long one (5^3 x 20 beside 16^3 x 128: 33 ms, by itself 1.4).
#pragma once

#include <condition_variable>
#include <cstdint>
#include <mutex>

namespace hub {

class FairLock {
    std::mutex m_;
    std::condition_variable turn_;
    uint64_t next_ = 0, serving_ = 0;

  public:
    void lock() {
        std::unique_lock<std::mutex> lk(m_);
        const uint64_t mine = next_++;
        turn_.wait(lk, [&] { return serving_ == mine; });
    }
    void unlock() {
        {
            std::lock_guard<std::mutex> lk(m_);
            ++serving_;
        }
        turn_.notify_all();
    }
};

}  // namespace hub
