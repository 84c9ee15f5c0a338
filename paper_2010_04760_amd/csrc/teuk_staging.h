// Large results to the host through a few pinned chunks: who moves which chunk when,
// the pool of the chunk sets and the number of threads.  Host code without HIP calls (the
// transfers and the sets' memory are the caller's), so that it can be tested without a GPU.
#pragma once

#include <sched.h>

#include <algorithm>
#include <condition_variable>
#include <cstddef>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <thread>
#include <vector>

namespace teuk {

// CPUs that a cgroup's quota leaves (0: no quota), from the files of version 2 and 1.
inline int quota_cpus(const char* v2 = "/sys/fs/cgroup/cpu.max",
                      const char* v1_quota = "/sys/fs/cgroup/cpu/cpu.cfs_quota_us",
                      const char* v1_period = "/sys/fs/cgroup/cpu/cpu.cfs_period_us")
{
    long long quota = -1, period = 0;
    if (FILE* f = std::fopen(v2, "r")) {
        if (std::fscanf(f, "%lld %lld", &quota, &period) != 2) quota = -1;      // "max" where there is none
        std::fclose(f);
    } else if (FILE* q = std::fopen(v1_quota, "r")) {
        if (std::fscanf(q, "%lld", &quota) != 1) quota = -1;
        std::fclose(q);
        if (FILE* p = std::fopen(v1_period, "r")) {
            if (std::fscanf(p, "%lld", &period) != 1) period = 0;
            std::fclose(p);
        }
    }
    if (quota <= 0 || period <= 0) return 0;
    return (int)std::min<long long>(std::max<long long>(quota / period, 1), 1 << 20);
}

// CPUs this process may run on at once (1 if unknown).
inline int usable_cpus()
{
    static const int quota = quota_cpus();
    cpu_set_t set;
    CPU_ZERO(&set);
    const int n = sched_getaffinity(0, sizeof(set), &set) == 0 ? std::max(1, CPU_COUNT(&set)) : 1;
    return quota > 0 ? std::min(n, quota) : n;
}

// Chunk sets, at most kMax in the process: handed to one copy at a time, kept between
// copies while any user (solver) is alive, released with the last one.  A copy on a
// device without an idle set takes the place of another device's.
template <class Set, int kMax>
class SetPool {
public:
    void user_made()
    {
        std::lock_guard<std::mutex> lock(mutex_);
        ++users_;
    }
    template <class Free>
    void user_gone(Free free)
    {
        Set* drop[kMax];
        int n = 0;
        {
            std::lock_guard<std::mutex> lock(mutex_);
            if (--users_ == 0) {
                for (; n < nidle_; ++n) drop[n] = idle_[n];
                nidle_ = 0;
                made_ -= n;
            }
        }
        for (int i = 0; i < n; ++i) free(drop[i]);
    }
    // A set of `device`, or null: kMax are in use, or make() gave none.
    template <class Make, class Free>
    Set* take(int device, Make make, Free free)
    {
        Set* other = nullptr;
        {
            std::lock_guard<std::mutex> lock(mutex_);
            for (int i = 0; i < nidle_; ++i)
                if (idle_[i]->device == device) {
                    Set* s = idle_[i];
                    idle_[i] = idle_[--nidle_];
                    return s;
                }
            if (made_ < kMax) ++made_;
            else if (nidle_ > 0) other = idle_[--nidle_];
            else return nullptr;
        }
        if (other) free(other);
        Set* s = make();
        if (s) return s;
        std::lock_guard<std::mutex> lock(mutex_);
        --made_;
        return nullptr;
    }
    template <class Free>
    void give(Set* s, Free free)
    {
        {
            std::lock_guard<std::mutex> lock(mutex_);
            if (users_ > 0) {
                idle_[nidle_++] = s;
                return;
            }
            --made_;
        }
        free(s);
    }

private:
    std::mutex mutex_;
    Set* idle_[kMax] = {};
    int nidle_ = 0, made_ = 0;
    long long users_ = 0;
};

// Move `bytes` to dst through `buffers` buffers of `chunk` bytes at mem: issue(c, b, n)
// starts the arrival of chunk c (n bytes) in buffer b, landed(b) waits for it (both 0 or
// an error), at most half of the buffers under way at a time; `workers` threads move the
// chunks on, asleep while they have none.  Returns the first error; *started is false, and
// nothing was issued, if the threads could not be had.  (Nothing here throws: it is
// called below a C interface.)
constexpr int kMaxMovers = 16, kMaxBuffers = 32;
template <class Issue, class Landed>
int move_chunks(char* dst, const char* mem, size_t bytes, size_t chunk, int buffers, int workers, Issue issue,
                Landed landed, bool* started)
{
    const long long n = (long long)((bytes + chunk - 1) / chunk);
    std::mutex mutex;
    std::condition_variable wake[kMaxMovers];     // each worker's
    std::condition_variable freed;                // a buffer has been moved on
    long long ready = 0;                          // chunks that have arrived; n + 1: give up
    long long moved[kMaxBuffers] = {};            // per buffer: the last chunk moved out of it, plus 1
    workers = std::min(workers, kMaxMovers);
    buffers = std::min(buffers, kMaxBuffers);
    auto size_of = [&](long long c) { return std::min(chunk, bytes - (size_t)c * chunk); };
    auto work = [&](int w) {
        for (long long c = w; c < n; c += workers) {
            {
                std::unique_lock<std::mutex> lock(mutex);
                wake[w].wait(lock, [&] { return ready > c; });
                if (ready > n) return;
            }
            const size_t b = (size_t)(c % buffers);
            std::memcpy(dst + (size_t)c * chunk, mem + b * chunk, size_of(c));
            {
                std::lock_guard<std::mutex> lock(mutex);
                moved[b] = c + 1;
            }
            freed.notify_one();
        }
    };
    std::vector<std::thread> threads;
    *started = true;
    try {
        threads.reserve((size_t)workers);
        for (int w = 0; w < workers; ++w) threads.emplace_back(work, w);
    } catch (...) {
        *started = false;
    }
    int e = 0;
    long long issued = 0;
    for (long long here = 0; *started && here < n && !e;) {
        while (issued < n && issued - here < buffers / 2 && !e) {
            // the buffer's chunk before this one has been moved on (wait only if nothing is under way)
            const size_t b = (size_t)(issued % buffers);
            if (issued >= buffers) {
                std::unique_lock<std::mutex> lock(mutex);
                auto is_free = [&] { return moved[b] == issued - buffers + 1; };
                if (issued > here) {
                    if (!is_free()) break;
                } else {
                    freed.wait(lock, is_free);
                }
            }
            e = issue(issued, (int)b, size_of(issued));
            ++issued;
        }
        if (!e) e = landed((int)(here % buffers));
        if (!e) {
            std::lock_guard<std::mutex> lock(mutex);
            ready = here + 1;
        }
        if (!e) wake[here++ % workers].notify_one();
    }
    if (!*started || e) {
        std::lock_guard<std::mutex> lock(mutex);
        ready = n + 1;
    }
    for (std::condition_variable& w : wake) w.notify_one();
    for (std::thread& t : threads) t.join();
    return e;
}

}  // namespace teuk
