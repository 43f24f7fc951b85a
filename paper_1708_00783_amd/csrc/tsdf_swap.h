// tsdf_swap.h -- host side of block swapping: the note kernels leave for the
// host, the transfer buffer, and the copies between it and the host store.
// Internal.
#pragma once

#include <emmintrin.h>
#include <stdint.h>
#include <string.h>
#include <unistd.h>

#include <atomic>

#include "tsdf.h"
#include "tsdf_copy_pool.h"
#include "tsdf_internal.h"

namespace tsdf {

// swap-in: store blocks idx[k] into slots k of the transfer buffer
struct SwapInCopy : CopyPool::Job {
    uint32_t n = 0;
    const int32_t *idx = nullptr;
    const uint8_t *store = nullptr;
    uint8_t *vox = nullptr;
    uint32_t size() const override { return n; }
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
    uint32_t call = 0, n = 0;
    const uint8_t *held = nullptr;
    uint8_t *store = nullptr;
    const uint8_t *vox = nullptr;
    std::atomic<bool> synced{false}, lost{false};
    static uint64_t word(const uint64_t *p) { return __atomic_load_n(p, __ATOMIC_ACQUIRE); }
    uint32_t size() const override { return n; }
    void block(uint32_t k) override
    {
        uint64_t w;
        for (CopyPool::Turn turn;;) {
            const bool last = synced.load(std::memory_order_acquire);
            w = word(note + 1 + k);
            if ((uint32_t)(w >> 32) == call) break;
            if (last) {
                lost.store(true, std::memory_order_relaxed);
                return;
            }
            turn();
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
    hipEvent_t counted = nullptr;   // swap-out: the note has the number of blocks
    CopyPool pool;
    pid_t pid = getpid();

    // blocks per part of a swap-in of n: a part below 256 (10 us) costs more in its launch than it overlaps
    static uint32_t part(uint32_t n)
    {
        const uint32_t per = (n + CopyPool::kParts - 1) / CopyPool::kParts;
        return per < 256u ? 256u : per;
    }

    // blocks that are worth waking the helpers for
    static bool many(uint32_t blocks) { return blocks >= 8 * CopyPool::kGrab; }

    hipError_t init(const tf_params &p, void *h_transfer, size_t bytes, Vol &v)
    {
        void *d = nullptr;
        // a note of candidates: visible blocks (swap-in), or a transfer (swap-out)
        const size_t most = p.n_blocks > p.swap_transfer_blocks ? p.n_blocks : p.swap_transfer_blocks;
        hipError_t e = hipHostMalloc((void **)&note, 8 * (1 + most), hipHostMallocCoherent);
        if (e == hipSuccess) e = hipHostGetDevicePointer(&d, note, 0);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&counted, hipEventDisableTiming);
        if (e != hipSuccess) return e;
        memset(note, 0, 8 * (1 + most));
        v.note = (unsigned long long *)d;
        // Kernels write and read the transfer buffer as vectors, while the host
        // reads other blocks of it, and writes other parts: the caller's if it is
        // pinned, coherent (as hipHostMalloc's default is) and aligned, else one
        // of its size.
        hipPointerAttribute_t a;
        unsigned flags = hipHostMallocNonCoherent;
        d = nullptr;
        if (hipPointerGetAttributes(&a, h_transfer) == hipSuccess && a.type == hipMemoryTypeHost &&
            hipHostGetFlags(&flags, h_transfer) == hipSuccess &&
            (flags == hipHostMallocDefault || ((flags & hipHostMallocCoherent) && !(flags & hipHostMallocNonCoherent))))
            d = a.devicePointer;
        else
            (void)hipGetLastError();
        vox = (uint8_t *)h_transfer;
        if (!d || ((uintptr_t)d & 15u) || ((uintptr_t)h_transfer & 15u)) {
            e = hipHostMalloc(&own, bytes, hipHostMallocCoherent);
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
        if (counted) (void)hipEventDestroy(counted);
    }
};

}  // namespace tsdf
