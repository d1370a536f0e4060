// A team of host threads for the length of one library call.
#pragma once
#include <sched.h>

#include <algorithm>
#include <atomic>
#include <condition_variable>
#include <cstdint>
#include <exception>
#include <mutex>
#include <thread>
#include <vector>

namespace cl {

// Started when a call has enough work for more than one thread, joined when it ends: no
// thread outlives the call, so nothing is shared between callers and a forked child
// misses none.  A call runs several loops one after the other, and the threads wait in
// between instead of being started for each (about 15 us a thread).
class Team {
public:
    static constexpr int kMaxThreads = 16;

    // As many threads as the process may run on, up to kMaxThreads and one per
    // `grain` units of the call's work.
    Team(int64_t work, int64_t grain)
    {
        int64_t n = std::min<int64_t>(kMaxThreads, work / std::max<int64_t>(1, grain));
        if (n > 1) {
            cpu_set_t set;
            const int cpus = sched_getaffinity(0, sizeof set, &set) == 0 ? CPU_COUNT(&set) : (int)std::thread::hardware_concurrency();
            n = std::min<int64_t>(n, std::max(1, cpus));
        }
        threads_.reserve((size_t)std::max<int64_t>(0, n - 1));
        try {
            for (int64_t i = 1; i < n; ++i) threads_.emplace_back([this] { serve(); });
        } catch (...) {      // (no thread, no memory for one) fewer than asked for: the work is shared among those there are
        }
    }

    ~Team()
    {
        {
            std::lock_guard<std::mutex> g(m_);
            stop_ = true;
        }
        wake_.notify_all();
        for (auto &t : threads_) t.join();
    }

    Team(const Team &) = delete;
    Team &operator=(const Team &) = delete;

    int size() const { return (int)threads_.size() + 1; }

    // f(i) for every i in [0, n), each once, in no particular order over threads; returns when
    // all are done.  The first exception of any f is thrown again here.
    template <class F>
    void each(int64_t n, F &&f)
    {
        if (threads_.empty() || n < 2) {
            for (int64_t i = 0; i < n; ++i) f(i);
            return;
        }
        std::atomic<int64_t> next{0};
        auto body = [&] {
            for (int64_t i; (i = next.fetch_add(1, std::memory_order_relaxed)) < n;) f(i);
        };
        auto call = [](void *p) { (*(decltype(body) *)p)(); };
        {
            std::lock_guard<std::mutex> g(m_);
            call_ = call;
            arg_ = &body;
            running_ = (int)threads_.size();
            ++round_;
        }
        wake_.notify_all();
        run_one(call, &body);
        std::unique_lock<std::mutex> l(m_);
        done_.wait(l, [&] { return running_ == 0; });
        if (error_) {
            std::exception_ptr e = error_;
            error_ = nullptr;
            std::rethrow_exception(e);
        }
    }

private:
    void run_one(void (*call)(void *), void *arg)
    {
        try {
            call(arg);
        } catch (...) {
            std::lock_guard<std::mutex> g(m_);
            if (!error_) error_ = std::current_exception();
        }
    }

    void serve()
    {
        uint64_t seen = 0;
        for (;;) {
            void (*call)(void *);
            void *arg;
            {
                std::unique_lock<std::mutex> l(m_);
                wake_.wait(l, [&] { return stop_ || round_ != seen; });
                if (stop_) return;
                seen = round_;
                call = call_;
                arg = arg_;
            }
            run_one(call, arg);
            std::lock_guard<std::mutex> g(m_);
            if (--running_ == 0) done_.notify_one();
        }
    }

    std::vector<std::thread> threads_;
    std::mutex m_;
    std::condition_variable wake_, done_;
    void (*call_)(void *) = nullptr;
    void *arg_ = nullptr;
    std::exception_ptr error_;
    uint64_t round_ = 0;
    int running_ = 0;
    bool stop_ = false;
};

}  // namespace cl
