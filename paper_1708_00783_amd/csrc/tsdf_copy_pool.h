// tsdf_copy_pool.h -- the threads that copy blocks beside the calling one.
// Host code only, with no use of the HIP runtime.  Internal.
#pragma once

#include <emmintrin.h>
#include <sched.h>
#include <stdint.h>
#include <unistd.h>

#include <atomic>
#include <condition_variable>
#include <memory>
#include <mutex>
#include <new>
#include <thread>
#include <vector>

namespace tsdf {

// Copies of single blocks by the calling thread and up to kHelpers others.  A
// block is 1.5 KB somewhere in a store of hundreds of megabytes, so one thread
// moves them at what its own cache misses allow: 17 GB/s, 280 us for 3000
// blocks, twice their time on the link.  The helpers sleep between jobs:
// start() wakes them, each goes back to sleep when a job has no more blocks to
// take, and finish() returns only once each has put the job down.
class CopyPool {
public:
    static constexpr uint32_t kHelpers = 3, kParts = 8, kGrab = 16;

    struct Job {
        virtual ~Job() {}
        virtual uint32_t size() const = 0;        // blocks of the job
        virtual void block(uint32_t k) = 0;       // copy block k; waits until it can be
        uint32_t per = ~0u;                       // blocks per part
        std::atomic<uint32_t> next{0};            // first block nobody has taken
        std::atomic<uint32_t> done[kParts] = {};  // blocks copied, by part
    };

    // One turn of a wait for another thread or the device: a pause for some tens
    // of microseconds, then sleep.  What is waited for is due within that; where
    // it is not (a busy device, a container short of CPU time), a thread that
    // goes on spinning takes the time from those that get on with the work.
    struct Turn {
        uint32_t n = 0;
        void operator()()
        {
            if (++n < 1024u)
                _mm_pause();
            else
                usleep(20);
        }
    };

    ~CopyPool()
    {
        if (!s_) return;
        // a forked child has the handles but not the threads, and the condition
        // variable, as it was copied, still counts them as waiters: its end
        // would wait for them for good
        if (getpid() != s_->pid) {
            (void)s_.release();
            return;
        }
        {
            std::lock_guard<std::mutex> g(s_->m);
            s_->stop = true;
        }
        s_->cv.notify_all();
        for (std::thread &t : s_->th) t.join();
    }

    void start(Job &job)
    {
        if (s_ && getpid() != s_->pid) (void)s_.release();
        if (!s_) {
            s_.reset(new (std::nothrow) Shared());
            if (!s_) return;   // the caller copies it all
            Shared *s = s_.get();
            cpu_set_t set;
            const int cpus = sched_getaffinity(0, sizeof(set), &set) == 0 ? CPU_COUNT(&set) : 1;
            try {
                for (int k = 0; k < (int)kHelpers && k < cpus - 1; ++k) s->th.emplace_back([s] { helper(*s); });
            } catch (...) {   // no more threads to be had: the caller copies what they would have
            }
        }
        {
            std::lock_guard<std::mutex> g(s_->m);
            s_->job = &job;
            ++s_->jobs;
        }
        s_->cv.notify_all();
    }

    // the next few blocks of a job, if there are any
    static bool take(Job &job)
    {
        uint32_t i = job.next.load(std::memory_order_relaxed);
        const uint32_t n = job.size();
        if (i >= n) return false;
        const uint32_t part = i / job.per, rest = job.per - i % job.per;
        const uint32_t cnt = rest < n - i ? (rest < kGrab ? rest : kGrab) : (n - i < kGrab ? n - i : kGrab);
        if (!job.next.compare_exchange_weak(i, i + cnt, std::memory_order_acq_rel)) return true;
        for (uint32_t k = i; k < i + cnt; ++k) job.block(k);
        job.done[part].fetch_add(cnt, std::memory_order_release);
        return true;
    }

    // returns when the `blocks` blocks of a part are copied
    static void finish_part(Job &job, uint32_t part, uint32_t blocks)
    {
        Turn turn;
        while (job.done[part].load(std::memory_order_acquire) < blocks)
            if (!take(job)) turn();
    }

    void finish()
    {
        if (!s_) return;
        {
            std::lock_guard<std::mutex> g(s_->m);
            s_->job = nullptr;
        }
        for (Turn turn; s_->busy.load(std::memory_order_acquire) != 0;) turn();
    }

private:
    // what the helpers hold on to: apart from the pool, so that a forked child can leave it behind
    struct Shared {
        std::vector<std::thread> th;
        std::mutex m;
        std::condition_variable cv;
        bool stop = false;
        const pid_t pid = getpid();
        Job *job = nullptr;
        uint64_t jobs = 0;           // jobs started
        std::atomic<int> busy{0};    // helpers that hold the job
    };

    static void helper(Shared &s)
    {
        for (uint64_t seen = 0;;) {
            Job *job;
            {
                std::unique_lock<std::mutex> g(s.m);
                s.cv.wait(g, [&] { return s.stop || (s.job && s.jobs != seen); });
                if (s.stop) return;
                seen = s.jobs;
                job = s.job;
                s.busy.fetch_add(1, std::memory_order_relaxed);   // under the lock: finish() sees it or we see no job
            }
            while (take(*job)) {}
            s.busy.fetch_sub(1, std::memory_order_release);
        }
    }

    std::unique_ptr<Shared> s_;
};

}  // namespace tsdf
