// tsdf_swap.h -- host side of block swapping: the note kernels leave for the
// host, the transfer buffer, and the threads that move blocks between it and
// the host store.  Internal.
#pragma once

#include <emmintrin.h>
#include <sched.h>
#include <stdint.h>
#include <string.h>
#include <unistd.h>

#include <atomic>
#include <condition_variable>
#include <mutex>
#include <thread>
#include <vector>

#include "tsdf.h"
#include "tsdf_internal.h"

namespace tsdf {

// Copies of single blocks by the calling thread and up to kHelpers others.  A
// block is 1.5 KB somewhere in a store of hundreds of megabytes, so one thread
// moves them at what its own cache misses allow: 17 GB/s, 280 us for 3000
// blocks, twice their time on the link.  The helpers sleep between jobs:
// start() wakes them (they may wait for the job's size there) and finish()
// returns only once each has put the job down.
class CopyPool {
public:
    static constexpr uint32_t kHelpers = 3, kParts = 8, kGrab = 16;

    struct Job {
        virtual ~Job() {}
        virtual uint32_t size() const = 0;        // blocks of the job; 0 while that is not known
        virtual void block(uint32_t k) = 0;       // copy block k; waits until it can be
        uint32_t per = ~0u;                       // blocks per part
        std::atomic<uint32_t> next{0};            // first block nobody has taken
        std::atomic<uint32_t> done[kParts] = {};  // blocks copied, by part
    };

    ~CopyPool()
    {
        if (th_.empty()) return;
        if (getpid() != pid_) {   // a forked child has the handles but not the threads
            for (std::thread &t : th_) t.detach();
            return;
        }
        {
            std::lock_guard<std::mutex> g(m_);
            stop_ = true;
        }
        cv_.notify_all();
        for (std::thread &t : th_) t.join();
    }

    void start(Job &job)
    {
        if (!tried_) {
            tried_ = true;
            pid_ = getpid();
            cpu_set_t set;
            const int cpus = sched_getaffinity(0, sizeof(set), &set) == 0 ? CPU_COUNT(&set) : 1;
            try {
                for (int k = 0; k < (int)kHelpers && k < cpus - 1; ++k) th_.emplace_back([this] { helper(); });
            } catch (...) {   // no more threads to be had: the caller copies what they would have
            }
        }
        {
            std::lock_guard<std::mutex> g(m_);
            job_.store(&job, std::memory_order_seq_cst);
        }
        cv_.notify_all();
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
        while (job.done[part].load(std::memory_order_acquire) < blocks)
            if (!take(job)) _mm_pause();
    }

    void finish()
    {
        job_.store(nullptr, std::memory_order_seq_cst);
        while (busy_.load(std::memory_order_seq_cst) != 0) _mm_pause();
    }

private:
    void helper()
    {
        for (;;) {
            {
                std::unique_lock<std::mutex> g(m_);
                cv_.wait(g, [this] { return stop_ || job_.load(std::memory_order_seq_cst); });
                if (stop_) return;
            }
            // announced before the look at job_, so that finish() waits for whoever saw a job
            busy_.fetch_add(1, std::memory_order_seq_cst);
            while (Job *job = job_.load(std::memory_order_seq_cst))
                if (!take(*job)) _mm_pause();
            busy_.fetch_sub(1, std::memory_order_seq_cst);
        }
    }

    std::vector<std::thread> th_;
    std::mutex m_;
    std::condition_variable cv_;
    bool stop_ = false, tried_ = false;
    pid_t pid_ = 0;
    std::atomic<Job *> job_{nullptr};
    std::atomic<int> busy_{0};
};

// swap-in: store blocks idx[k] into slots k of the transfer buffer
struct SwapInCopy : CopyPool::Job {
    std::atomic<uint32_t> n{0};
    const int32_t *idx = nullptr;
    const uint8_t *store = nullptr;
    uint8_t *vox = nullptr;
    uint32_t size() const override { return n.load(std::memory_order_acquire); }
    void block(uint32_t k) override
    {
        memcpy(vox + (size_t)k * kBlockBytes, store + (size_t)idx[k] * kBlockBytes, kBlockBytes);
    }
};

// swap-out: slots k of the transfer buffer into the store, each as soon as the
// gather has noted it (or, at the latest, when the stream is done), except
// blocks the store already holds.  A note word is entry | call << 32.
struct SwapOutCopy : CopyPool::Job {
    const uint64_t *note = nullptr;
    uint32_t call = 0, cap = 0;
    const uint8_t *held = nullptr;
    uint8_t *store = nullptr;
    const uint8_t *vox = nullptr;
    std::atomic<bool> synced{false}, lost{false};
    static uint64_t word(const uint64_t *p) { return __atomic_load_n(p, __ATOMIC_ACQUIRE); }
    uint32_t size() const override
    {
        const uint64_t w = word(note);
        return (uint32_t)(w >> 32) == call ? ((uint32_t)w < cap ? (uint32_t)w : cap) : 0u;
    }
    void block(uint32_t k) override
    {
        uint64_t w;
        for (;;) {
            const bool last = synced.load(std::memory_order_acquire);
            w = word(note + 1 + k);
            if ((uint32_t)(w >> 32) == call) break;
            if (last) {
                lost.store(true, std::memory_order_relaxed);
                return;
            }
            _mm_pause();
        }
        const size_t e = (uint32_t)w;
        if (!held[e]) memcpy(store + e * kBlockBytes, vox + (size_t)k * kBlockBytes, kBlockBytes);
    }
};

struct SwapHost {
    uint64_t *note = nullptr;   // pinned: [0] candidates, then their entries
    uint8_t *vox = nullptr;     // the transfer buffer: blocks, then entry indices
    int32_t *idx = nullptr;
    void *own = nullptr;        // it, where the caller's is not one the device can use
    uint32_t call = 0;          // of swap-out, in the words of its note
    uint32_t last_in = 0, last_out = 0;   // blocks the last call moved
    CopyPool pool;
    pid_t pid = getpid();

    // blocks per part of a swap-in of n: a part below 256 (10 us) costs more in its launch than it overlaps
    static uint32_t part(uint32_t n)
    {
        const uint32_t per = (n + CopyPool::kParts - 1) / CopyPool::kParts;
        return per < 256u ? 256u : per;
    }

    // helpers are woken ahead of a wait for the device that is likely to end in as many blocks again
    static bool many(uint32_t blocks) { return blocks >= 8 * CopyPool::kGrab; }

    hipError_t init(const tf_params &p, void *h_transfer, size_t bytes, Vol &v)
    {
        void *d = nullptr;
        // a note of candidates: visible blocks (swap-in), or a transfer (swap-out)
        const size_t most = p.n_blocks > p.swap_transfer_blocks ? p.n_blocks : p.swap_transfer_blocks;
        hipError_t e = hipHostMalloc((void **)&note, 8 * (1 + most), hipHostMallocCoherent);
        if (e == hipSuccess) e = hipHostGetDevicePointer(&d, note, 0);
        if (e != hipSuccess) return e;
        memset(note, 0, 8 * (1 + most));
        v.note = (unsigned long long *)d;
        // kernels write and read the transfer buffer as vectors: the caller's
        // if it is pinned and aligned, else one of its size
        hipPointerAttribute_t a;
        d = nullptr;
        if (hipPointerGetAttributes(&a, h_transfer) == hipSuccess && a.type == hipMemoryTypeHost)
            d = a.devicePointer;
        else
            (void)hipGetLastError();
        vox = (uint8_t *)h_transfer;
        if (!d || ((uintptr_t)d & 15u) || ((uintptr_t)h_transfer & 15u)) {
            e = hipHostMalloc(&own, bytes, hipHostMallocDefault);
            if (e == hipSuccess) e = hipHostGetDevicePointer(&d, own, 0);
            if (e != hipSuccess) return e;
            vox = (uint8_t *)own;
        }
        const size_t at = (size_t)p.swap_transfer_blocks * kBlockBytes;
        idx = (int32_t *)(vox + at);
        v.hx_vox = (uint8_t *)d;
        v.hx_idx = (int32_t *)(v.hx_vox + at);
        return hipSuccess;
    }
    ~SwapHost()
    {
        if (getpid() != pid) return;   // a forked child: the parent's to give back
        if (own) (void)hipHostFree(own);
        if (note) (void)hipHostFree(note);
    }
};

}  // namespace tsdf
