// Host threads of one library call: started when the call has enough to do, joined before it returns.
#pragma once

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstdint>
#include <exception>
#include <functional>
#include <mutex>
#include <thread>
#include <vector>

namespace vbrk {

// A team of `size` threads, the caller being the first of them.  run(f) calls f(member) on all of them and
// returns when every one is through; the first exception any of them throws is thrown again here.  A
// team of one starts no thread.  When the system refuses a thread the team is smaller.
class Team {
public:
    explicit Team(int size)
    {
        for (int t = 1; t < size; ++t) {
            try {
                workers_.emplace_back([this, t] { work(t); });
            } catch (const std::exception &) {
                break;
            }
        }
    }
    ~Team()
    {
        {
            std::lock_guard<std::mutex> g(m_);
            stop_ = true;
        }
        start_.notify_all();
        for (std::thread &t : workers_) t.join();
    }
    Team(const Team &) = delete;
    Team &operator=(const Team &) = delete;

    int size() const { return (int)workers_.size() + 1; }

    void run(const std::function<void(int)> &f)
    {
        if (workers_.empty()) { f(0); return; }
        {
            std::lock_guard<std::mutex> g(m_);
            job_ = &f;
            pending_ = (int)workers_.size();
            error_ = nullptr;
            ++round_;
        }
        start_.notify_all();
        call(f, 0);
        std::unique_lock<std::mutex> g(m_);
        done_.wait(g, [this] { return pending_ == 0; });
        if (error_) std::rethrow_exception(error_);
    }

    // f(begin, end) over [0, n) in pieces of `piece`, dealt to whoever is free
    template <class F>
    void each(int64_t n, int64_t piece, F f)
    {
        if (workers_.empty() || n <= piece) {
            if (n > 0) f((int64_t)0, n);
            return;
        }
        std::atomic<int64_t> next(0);
        run([&](int) {
            for (;;) {
                const int64_t b = next.fetch_add(piece);
                if (b >= n) break;
                f(b, std::min(n, b + piece));
            }
        });
    }

private:
    void call(const std::function<void(int)> &f, int member)
    {
        try {
            f(member);
        } catch (...) {
            std::lock_guard<std::mutex> g(m_);
            if (!error_) error_ = std::current_exception();
        }
    }
    void work(int member)
    {
        uint64_t seen = 0;
        for (;;) {
            const std::function<void(int)> *f;
            {
                std::unique_lock<std::mutex> g(m_);
                start_.wait(g, [&] { return stop_ || round_ != seen; });
                if (stop_) return;
                seen = round_;
                f = job_;
            }
            call(*f, member);
            {
                std::lock_guard<std::mutex> g(m_);
                if (--pending_ == 0) done_.notify_one();
            }
        }
    }
    std::vector<std::thread> workers_;
    std::mutex m_;
    std::condition_variable start_, done_;
    const std::function<void(int)> *job_ = nullptr;
    std::exception_ptr error_;
    uint64_t round_ = 0;
    int pending_ = 0;
    bool stop_ = false;
};

// Threads worth starting for about `work` elementary steps: one for every `per_thread` of them, at most the host's
// cores and 32 (starting and joining a thread costs some tens of microseconds).
inline int threads_for(int64_t work, int64_t per_thread)
{
    const int64_t hw = std::max(1u, std::min(std::thread::hardware_concurrency(), 32u));
    return (int)std::max<int64_t>(1, std::min(hw, work / per_thread));
}

}  // namespace vbrk
