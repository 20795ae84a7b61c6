// Copies of large results out of pinned memory.
//
// A result goes into memory that the caller has usually just allocated, so the
// copy takes a page fault every 4 KiB (or 2 MiB) beside the traffic: one thread
// moves 13 MB in 0.45 ms and 420 MB in 35-60, where the device produces the
// latter in 12.  Faults of different pages and the traffic itself go in
// parallel, so a large copy gets helper threads, started for this copy and joined
// before it returns (about 15 us each); the calling thread copies too, and alone
// where none can be started.  The 420 MB take 14 ms then (the device's 12 and the
// ends), a served result of 13 MB 0.57 ms where it took 0.78.
#pragma once

#include <algorithm>
#include <condition_variable>
#include <cstddef>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <exception>
#include <thread>
#include <vector>

namespace bem {

// Helper threads for a copy of so many bytes: one for each 2 MiB past the first.
inline int copy_helpers(size_t bytes, int most) { return (int)std::min<size_t>((size_t)most, bytes >> 21); }

// Work items 0, 1, ..., done by helpers and by the caller in help(); item i may
// be taken once release(m) has been called with m > i.
template <class Do>
class CopyCrew {
public:
    static constexpr int kMost = 7;

    CopyCrew(int helpers, Do item) : do_(item)
    {
        for (int64_t &i : open_) i = INT64_MAX;
        try {
            threads_.reserve((size_t)helpers);
            for (int i = 0; i < std::min(helpers, kMost); ++i) threads_.emplace_back([this, i] { work(i + 1); });
        } catch (const std::exception &) {
            // fewer helpers
        }
    }
    ~CopyCrew()
    {
        {
            std::lock_guard<std::mutex> g(mu_);
            stop_ = true;
        }
        cv_.notify_all();
        for (std::thread &t : threads_) t.join();
    }
    CopyCrew(const CopyCrew &) = delete;
    CopyCrew &operator=(const CopyCrew &) = delete;

    void release(int64_t m)
    {
        {
            std::lock_guard<std::mutex> g(mu_);
            ready_ = m;
        }
        cv_.notify_all();
    }
    // Returns once the first m items (all released) are done.
    void help(int64_t m)
    {
        std::unique_lock<std::mutex> lk(mu_);
        while (next_ < m) one(lk, 0);
        idle_.wait(lk, [&] { return lowest() >= m; });
    }

private:
    // every item below this one is done
    int64_t lowest() const
    {
        int64_t v = next_;
        for (int64_t i : open_) v = std::min(v, i);
        return v;
    }
    void one(std::unique_lock<std::mutex> &lk, int me)
    {
        const int64_t i = open_[me] = next_++;
        lk.unlock();
        do_(i);
        lk.lock();
        open_[me] = INT64_MAX;
        idle_.notify_all();
    }
    void work(int me)
    {
        std::unique_lock<std::mutex> lk(mu_);
        for (;;) {
            cv_.wait(lk, [&] { return stop_ || next_ < ready_; });
            if (next_ >= ready_) return;
            one(lk, me);
        }
    }

    Do do_;
    std::mutex mu_;
    std::condition_variable cv_, idle_;
    int64_t next_ = 0, ready_ = 0;
    bool stop_ = false;
    int64_t open_[kMost + 1];   // per thread the item it is at
    std::vector<std::thread> threads_;
};

// memcpy with up to three helpers, a MiB at a time.
inline void copy_large(void *dst, const void *src, size_t bytes)
{
    const int helpers = copy_helpers(bytes, 3);
    if (helpers == 0) {
        std::memcpy(dst, src, bytes);
        return;
    }
    constexpr size_t kPart = size_t(1) << 20;
    const int64_t n = (int64_t)((bytes + kPart - 1) / kPart);
    auto part = [=](int64_t i) {
        const size_t at = (size_t)i * kPart;
        std::memcpy(static_cast<char *>(dst) + at, static_cast<const char *>(src) + at, std::min(kPart, bytes - at));
    };
    CopyCrew<decltype(part)> crew(helpers, part);
    crew.release(n);
    crew.help(n);
}

}  // namespace bem
