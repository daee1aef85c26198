// Host copies split over a few threads (plain C++).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstring>
#include <mutex>
#include <thread>
#include <vector>

namespace pll {

// Copies between request arrays and the slots' pinned staging, split over
// the scheduler and a few helper threads.  A full batch moves 8 MiB in and
// 4 MiB out, and one thread's copies (about 20 GB/s) took longer than the
// device: 2,000 requests of 11.8 M pairs on R-MAT 262,144 took 7.5 ms, 6.0 with
// three helpers and 5.7 with six.  Small sets stay on the scheduler's thread.
// A thread takes a part at a time, of kPart bytes: large copies are cut into
// parts and small ones gathered, so that the requests' size does not set how
// often the threads meet: 2,000 requests of 200 pairs on R-MAT 65,536 took 2.4
// ms on one thread, 2.4 to 3.4 with each request's copies handed out on their
// own, 2.0 to 2.4 in parts; the 11.8 M pairs 5.9 and 5.3 ms.
constexpr uint32_t kCopyHelpers = 6;

class CopyPool {
public:
    static constexpr size_t kPart = 128u << 10, kShare = 1u << 20;

    CopyPool() = default;
    CopyPool(const CopyPool&) = delete;
    CopyPool& operator=(const CopyPool&) = delete;

    // As many helpers as start; with none the caller copies alone.
    void start(uint32_t helpers) {
        try {
            for (uint32_t i = 0; i < helpers; ++i) threads_.emplace_back([this] { loop(); });
        } catch (...) {
        }
    }
    ~CopyPool() {
        {
            std::lock_guard<std::mutex> lk(mu_);
            stop_ = true;
        }
        cv_.notify_all();
        for (std::thread& t : threads_) t.join();
    }
    void add(void* dst, const void* src, size_t bytes) {
        total_ += bytes;
        for (size_t at = 0; at < bytes; at += kPart) {
            const size_t k = std::min(kPart, bytes - at);
            jobs_.push_back(Job{static_cast<char*>(dst) + at, static_cast<const char*>(src) + at, k});
            part_bytes_ += k;
            if (part_bytes_ >= kPart) close_part();
        }
    }
    // Run what was added (one thread adds and runs; returns when all is
    // copied); the number of parts it was handed out in.
    size_t run() {
        if (part_bytes_) close_part();
        const size_t parts = ends_.size();
        next_.store(0, std::memory_order_relaxed);
        const bool share = total_ >= kShare && !threads_.empty();
        if (share) {
            {
                std::lock_guard<std::mutex> lk(mu_);
                ++generation_;
                open_ = true;
            }
            cv_.notify_all();
        }
        work();
        if (share) {  // every part is taken: wait for the helpers still copying
            std::unique_lock<std::mutex> lk(mu_);
            open_ = false;
            idle_.wait(lk, [this] { return inside_ == 0; });
        }
        jobs_.clear();
        ends_.clear();
        total_ = 0;
        return parts;
    }

private:
    struct Job {
        void* dst;
        const void* src;
        size_t bytes;
    };
    void close_part() {
        ends_.push_back(jobs_.size());
        part_bytes_ = 0;
    }
    void work() {
        for (;;) {
            const size_t p = next_.fetch_add(1, std::memory_order_relaxed);
            if (p >= ends_.size()) return;
            for (size_t i = p ? ends_[p - 1] : 0; i < ends_[p]; ++i)
                std::memcpy(jobs_[i].dst, jobs_[i].src, jobs_[i].bytes);
        }
    }
    void loop() {
        uint64_t seen = 0;
        std::unique_lock<std::mutex> lk(mu_);
        for (;;) {
            cv_.wait(lk, [&] { return stop_ || (open_ && generation_ != seen); });
            if (stop_) return;
            seen = generation_;
            ++inside_;
            lk.unlock();
            work();
            lk.lock();
            if (--inside_ == 0) idle_.notify_one();
        }
    }
    std::vector<std::thread> threads_;
    std::mutex mu_;
    std::condition_variable cv_, idle_;
    std::vector<Job> jobs_;     // these two are fixed while open_
    std::vector<size_t> ends_;  // part p: jobs [ends_[p - 1], ends_[p])
    size_t part_bytes_ = 0;     // of the part being filled
    std::atomic<size_t> next_{0};
    size_t total_ = 0;
    uint64_t generation_ = 0;
    uint32_t inside_ = 0;
    bool open_ = false, stop_ = false;
};

}  // namespace pll
