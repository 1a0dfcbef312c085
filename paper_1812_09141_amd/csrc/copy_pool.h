// Copies between host buffers by several threads.
#pragma once

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstring>
#include <mutex>
#include <thread>
#include <vector>

namespace ssj {

// Copies from pageable to pinned memory run at about 30 GB/s in one thread,
// little more than half of what the link to the device takes.  The pool's
// threads share the parts of a copy with its caller.  They start with the first
// large copy and look out for the next one for a short while before they sleep
// (requests come in bursts, and a wake-up takes as long as a part).  One copy at
// a time is shared: a caller that finds the pool busy copies alone.
class CopyPool {
public:
    ~CopyPool() {
        {
            std::lock_guard<std::mutex> g(m_);
            stop_ = true;
            seq_.fetch_add(1);
        }
        cv_.notify_all();
        for (auto& t : threads_) t.join();
    }

    void copy(void* dst, const void* src, size_t bytes) {
        std::unique_lock<std::mutex> mine(use_, std::defer_lock);
        if (bytes < kLeast || !mine.try_lock() || !start()) {
            std::memcpy(dst, src, bytes);
            return;
        }
        {
            std::lock_guard<std::mutex> g(m_);
            dst_ = static_cast<char*>(dst);
            src_ = static_cast<const char*>(src);
            bytes_ = bytes;
            next_.store(0);
            open_ = true;
            seq_.fetch_add(1);
        }
        cv_.notify_all();
        parts(dst_, src_, bytes_);
        std::unique_lock<std::mutex> g(m_);
        open_ = false;
        done_.wait(g, [&] { return active_ == 0; });
    }

private:
    static constexpr size_t kPart = (size_t)128 << 10, kLeast = 4 * kPart;
    static constexpr int kThreads = 3, kLooks = 2000;

    bool start() {  // use_ held
        if (threads_.empty()) {
            const unsigned hw = std::max(1u, std::thread::hardware_concurrency());
            try {
                for (int k = 0; k < std::min<int>(kThreads, (int)hw - 1); ++k) threads_.emplace_back([this] { serve(); });
            } catch (...) {  // no (further) thread
            }
        }
        return !threads_.empty();
    }

    void parts(char* dst, const char* src, size_t bytes) {
        for (;;) {
            const size_t b = next_.fetch_add(kPart);
            if (b >= bytes) return;
            std::memcpy(dst + b, src + b, std::min(kPart, bytes - b));
        }
    }

    void serve() {
        unsigned long long seen = 0;
        for (;;) {
            for (int k = 0; k < kLooks && seq_.load() == seen; ++k) __builtin_ia32_pause();
            std::unique_lock<std::mutex> g(m_);
            cv_.wait(g, [&] { return stop_ || seq_.load() != seen; });
            if (stop_) return;
            seen = seq_.load();
            if (!open_) continue;
            ++active_;
            char* dst = dst_;
            const char* src = src_;
            const size_t bytes = bytes_;
            g.unlock();
            parts(dst, src, bytes);
            g.lock();
            if (--active_ == 0) done_.notify_one();
        }
    }

    std::mutex use_;                       // the copy being shared
    std::mutex m_;                         // the fields below
    std::condition_variable cv_, done_;
    std::atomic<unsigned long long> seq_{0};  // copies begun
    std::atomic<size_t> next_{0};          // first byte that no thread has taken
    char* dst_ = nullptr;
    const char* src_ = nullptr;
    size_t bytes_ = 0;
    int active_ = 0;                       // threads at work on the copy
    bool open_ = false, stop_ = false;
    std::vector<std::thread> threads_;
};

}  // namespace ssj
