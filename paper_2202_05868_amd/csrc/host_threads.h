// Host threads of the library's calls: kept between calls, asleep, and ended when they have been idle for some seconds.
#pragma once

#include <linux/futex.h>
#include <errno.h>
#include <pthread.h>
#include <sys/syscall.h>
#include <time.h>
#include <unistd.h>

#include <algorithm>
#include <atomic>
#include <cstdint>
#include <exception>
#include <functional>
#include <memory>
#include <mutex>
#include <thread>

namespace vbrk {

// Threads that wait for jobs.  A job is offered, not assigned: whoever is there in time joins it, and the caller, who
// works on it too, waits only for those who did, so a thread that takes long to wake up delays nobody.  Waiting threads
// look for the next job for some twenty microseconds before they sleep.  (Starting and joining 16 threads took 0.5 ms
// a call, and handing them a job 39 us, most of it waking them one after the other.)
class Gang {
public:
    // at least n threads from now on, as far as the system grants them
    static void grow(const std::shared_ptr<Gang> &g, int n)
    {
        while (g->threads_.load() < n) {
            g->threads_.fetch_add(1);
            try {
                std::thread([g] { g->work(); }).detach();
            } catch (const std::exception &) {
                g->threads_.fetch_sub(1);
                return;
            }
        }
    }

    // f(0) here, f(1) .. f(others) on as many threads as join before f(0) is done; one job at a time
    void run(const std::function<void(int)> &f, int others)
    {
        job_ = &f;
        error_ = nullptr;
        finished_.store(0);
        state_.store(kOpen | ((uint64_t)others << 32));
        round_.fetch_add(1);
        wake(4);                                             // each of them wakes two more
        call(f, 0);
        const int started = (int)(state_.fetch_and(~kOpen) & kStarted);
        for (int spin = 0; finished_.load(std::memory_order_acquire) != started;) {
            __builtin_ia32_pause();
            if (++spin > 4000) { std::this_thread::yield(); spin = 0; }
        }
        if (error_) std::rethrow_exception(error_);
    }

    void stop()
    {
        stop_.store(true);
        round_.fetch_add(1);
        syscall(SYS_futex, reinterpret_cast<uint32_t *>(&round_), FUTEX_WAKE_PRIVATE, INT32_MAX, nullptr, nullptr, 0);
    }

private:
    static constexpr uint64_t kOpen = (uint64_t)1 << 63, kStarted = 0xffffffffu;
    static constexpr int kSpins = 500, kIdleSeconds = 5;

    void wake(int n)
    {
        if (sleepers_.load() > 0) syscall(SYS_futex, reinterpret_cast<uint32_t *>(&round_), FUTEX_WAKE_PRIVATE, n, nullptr, nullptr, 0);
    }
    void call(const std::function<void(int)> &f, int member)
    {
        try {
            f(member);
        } catch (...) {
            std::lock_guard<std::mutex> g(m_);
            if (!error_) error_ = std::current_exception();
        }
    }
    void work()
    {
        uint32_t seen = round_.load();
        join();
        for (;;) {
            for (int i = 0; i < kSpins && round_.load(std::memory_order_relaxed) == seen; ++i) __builtin_ia32_pause();
            bool slept = false, idle = false;
            if (round_.load() == seen) {
                slept = true;
                sleepers_.fetch_add(1);
                const timespec limit = {kIdleSeconds, 0};
                const long rc = syscall(SYS_futex, reinterpret_cast<uint32_t *>(&round_), FUTEX_WAIT_PRIVATE, seen, &limit, nullptr, 0);
                idle = rc != 0 && errno == ETIMEDOUT && round_.load() == seen;
                sleepers_.fetch_sub(1);
            }
            if (idle || stop_.load()) {
                threads_.fetch_sub(1);
                return;
            }
            seen = round_.load();
            if (slept) wake(2);
            join();
        }
    }
    void join()
    {
        uint64_t s = state_.load();
        while ((s & kOpen) && (s & kStarted) < (s >> 32 & 0x7fffffffu)) {
            if (!state_.compare_exchange_weak(s, s + 1)) continue;
            call(*job_, (int)(s & kStarted) + 1);
            finished_.fetch_add(1, std::memory_order_release);
            return;
        }
    }

    std::atomic<uint32_t> round_{0};
    std::atomic<uint64_t> state_{0};         // open, most others, others started
    std::atomic<int> finished_{0}, sleepers_{0}, threads_{0};
    std::atomic<bool> stop_{false};
    const std::function<void(int)> *job_ = nullptr;
    std::mutex m_;
    std::exception_ptr error_;
};

// The gang calls share, one call at a time; never destroyed (its threads may outlive static objects), and left behind
// by a forked child, which has none of its threads.
struct SharedGang {
    std::shared_ptr<Gang> gang = std::make_shared<Gang>();
    std::atomic<bool> taken{false};
    static std::atomic<SharedGang *> &slot()
    {
        static std::atomic<SharedGang *> current([] {
            pthread_atfork(nullptr, nullptr, [] { slot().store(new SharedGang()); });
            return new SharedGang();
        }());
        return current;
    }
};

// Up to `size` threads for one call, the caller being the first of them.  Team::run(f) calls f(member), member < size(), on
// the caller and on those that come in time; f takes its share of the work from a common counter.  The first exception
// any of them throws is thrown again here.  A call that finds the shared gang taken by another has threads of its own.
class Team {
public:
    explicit Team(int size) : size_(std::max(1, size))
    {
        if (size_ == 1) return;
        SharedGang *s = SharedGang::slot().load();
        if (!s->taken.exchange(true)) {
            shared_ = s;
            gang_ = s->gang;
        } else {
            gang_ = std::make_shared<Gang>();
        }
        Gang::grow(gang_, size_ - 1);
    }
    ~Team()
    {
        if (shared_) shared_->taken.store(false);
        else if (gang_) gang_->stop();
    }
    Team(const Team &) = delete;
    Team &operator=(const Team &) = delete;

    int size() const { return size_; }

    void run(const std::function<void(int)> &f)
    {
        if (size_ == 1) f(0);
        else gang_->run(f, size_ - 1);
    }

    // f(begin, end) over [0, n) in pieces of `piece`, dealt to whoever is free
    template <class F>
    void each(int64_t n, int64_t piece, F f)
    {
        if (size_ == 1 || n <= piece) {
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
    const int size_;
    SharedGang *shared_ = nullptr;
    std::shared_ptr<Gang> gang_;
};

// Threads worth asking for about `work` elementary steps: one for every `per_thread` of them, at most the host's
// cores and 32.
inline int threads_for(int64_t work, int64_t per_thread)
{
    const int64_t hw = std::max(1u, std::min(std::thread::hardware_concurrency(), 32u));
    return (int)std::max<int64_t>(1, std::min(hw, work / per_thread));
}

}  // namespace vbrk
