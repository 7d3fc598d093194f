// A few worker threads for the length of one encode call.  run(parts, f) calls f(0) .. f(parts - 1),
// each once, on the calling thread and the workers, and returns when all are done.  The workers are
// started by the first run (after its parts are up for grabs, so that starting them overlaps with the
// work) and joined by the destructor: nothing outlives the call, calls on several threads share nothing.
#ifndef HAC_TEAM_H
#define HAC_TEAM_H

#include <sched.h>

#include <atomic>
#include <condition_variable>
#include <cstdint>
#include <functional>
#include <mutex>
#include <new>
#include <system_error>
#include <thread>
#include <vector>

namespace hac_internal {

class Team {
public:
    // one thread per `grain` units of work, at most 16 and at most the CPUs this process may use
    Team(uint64_t work, uint64_t grain) : size_(1)
    {
        cpu_set_t set;
        int cpus = 1;
        if (sched_getaffinity(0, sizeof set, &set) == 0) cpus = CPU_COUNT(&set);
        const uint64_t want = work / grain;
        size_ = (unsigned)(want < 1 ? 1 : want > 16 ? 16 : want);
        if (size_ > (unsigned)cpus) size_ = (unsigned)cpus;
    }
    ~Team()
    {
        if (workers_.empty()) return;
        { std::lock_guard<std::mutex> hold(lock_); stop_ = true; }
        wake_.notify_all();
        for (std::thread& w : workers_) w.join();
    }
    Team(const Team&) = delete;
    Team& operator=(const Team&) = delete;

    unsigned size() const { return size_; }

    void run(uint64_t parts, const std::function<void(uint64_t)>& f)
    {
        if (size_ == 1 || parts <= 1) {
            for (uint64_t i = 0; i < parts; ++i) f(i);
            return;
        }
        {
            std::lock_guard<std::mutex> hold(lock_);
            job_ = &f; parts_ = parts; next_.store(0); left_.store(parts); failed_.store(false);
            ++round_;
        }
        wake_.notify_all();
        if (workers_.empty()) {
            try {
                workers_.reserve(size_ - 1);
                for (unsigned i = 1; i < size_; ++i) workers_.emplace_back([this] { serve(); });
            } catch (const std::system_error&) {             // no more threads to be had: fewer will do
            } catch (const std::bad_alloc&) {
            }
        }
        work(f, parts);
        while (left_.load(std::memory_order_acquire)) std::this_thread::yield();
        {   // a worker that has not looked yet must not see this job (f ends with this call)
            std::unique_lock<std::mutex> hold(lock_);
            job_ = nullptr;
            idle_.wait(hold, [this] { return busy_ == 0; });
        }
        if (failed_.load()) throw std::bad_alloc();
    }

private:
    void work(const std::function<void(uint64_t)>& f, uint64_t parts)
    {
        for (;;) {
            const uint64_t i = next_.fetch_add(1);
            if (i >= parts) return;
            try {
                if (!failed_.load(std::memory_order_relaxed)) f(i);
            } catch (const std::bad_alloc&) {
                failed_.store(true);
            }
            left_.fetch_sub(1, std::memory_order_release);
        }
    }
    void serve()
    {
        uint64_t seen = 0;
        std::unique_lock<std::mutex> hold(lock_);
        for (;;) {
            wake_.wait(hold, [&] { return stop_ || (round_ != seen && job_); });
            if (stop_) return;
            seen = round_;
            const std::function<void(uint64_t)>* f = job_;
            const uint64_t parts = parts_;
            ++busy_;
            hold.unlock();
            work(*f, parts);
            hold.lock();
            if (--busy_ == 0) idle_.notify_all();
        }
    }

    unsigned size_;
    std::vector<std::thread> workers_;
    std::mutex lock_;
    std::condition_variable wake_, idle_;
    const std::function<void(uint64_t)>* job_ = nullptr;
    uint64_t parts_ = 0, round_ = 0;
    unsigned busy_ = 0;
    bool stop_ = false;
    std::atomic<uint64_t> next_{0}, left_{0};
    std::atomic<bool> failed_{false};
};

} // namespace hac_internal

#endif
