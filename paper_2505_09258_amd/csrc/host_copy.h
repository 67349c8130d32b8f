// Reading tables back into the caller's memory.
//
// Measured on a bucket of five million edges that reads its table of 1M x 100 floats back: 140.1 ms by hipMemcpy, 112.6 ms
// this way (120 001 x 128 floats: 11.5 and 7.5 ms).
// One hipMemcpy into pageable memory moves 10 to 16 GB/s here: a single host thread copies out of the runtime's
// staging buffer, and where the destination is fresh memory it also takes every page fault.  The link itself moves about
// 50 GB/s.  So a large read goes through a ring of pinned blocks: the calling thread enqueues the device copies in
// order, a few short-lived threads wait for each block and copy it out (the faults are spread over them).  Parts that
// lie in the host tier already are copied by the same threads.
// The ring belongs to one context (one caller at a time, like the context itself) and is freed with it.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <cstring>
#include <thread>
#include <vector>

namespace legend {

struct HostCopyPart {
    char* dst;
    const char* src;
    size_t bytes;
    bool on_device;
};

class HostCopyRing {
public:
    static constexpr size_t kBlock = (size_t)1 << 20;
    static constexpr int kSlots = 8;
    static constexpr int kMaxThreads = 8;
    // A context's first large read also pays for pinning the ring, about 0.1 ms a MB (with 24 MB of ring a first read of 24 MB was
    // slower than hipMemcpy); 32 MB take hipMemcpy 2 to 3 ms.
    static constexpr size_t kMinBytes = (size_t)32 << 20;

    // pinned memory and events on first use; false (nothing kept) where the host cannot give them
    bool prepare() {
        if (mem_) return true;
        void* p = nullptr;
        if (hipHostMalloc(&p, kBlock * kSlots, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
        mem_ = static_cast<char*>(p);
        for (hipEvent_t& e : ready_) {
            if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) {
                (void)hipGetLastError();
                release();
                return false;
            }
        }
        return true;
    }

    void release() {
        for (hipEvent_t& e : ready_) {
            if (e) (void)hipEventDestroy(e);
            e = nullptr;
        }
        if (mem_) (void)hipHostFree(mem_);
        mem_ = nullptr;
    }

    // Copies every part; the device parts on `st`.  Returns when all of it has arrived.  May throw std::bad_alloc
    // before anything has started.
    hipError_t run(const std::vector<HostCopyPart>& parts, int device, hipStream_t st) {
        struct Block {
            char* dst;
            const char* src;
            size_t bytes;
            int64_t dev;                 // running number among the device blocks, -1: host memory
        };
        std::vector<Block> blocks;
        std::vector<size_t> dev_block;
        for (const HostCopyPart& p : parts)
            for (size_t o = 0; o < p.bytes; o += kBlock) {
                if (p.on_device) dev_block.push_back(blocks.size());
                blocks.push_back({p.dst + o, p.src + o, p.bytes - o < kBlock ? p.bytes - o : kBlock,
                                  p.on_device ? (int64_t)dev_block.size() - 1 : -1});
            }
        std::vector<std::thread> threads;
        threads.reserve(kMaxThreads);
        std::vector<std::atomic<char>> drained(dev_block.size());
        for (auto& x : drained) x.store(0, std::memory_order_relaxed);
        std::atomic<size_t> next{0};
        std::atomic<int64_t> issued{0};
        std::atomic<int> err{(int)hipSuccess};

        // every wait below also ends on an error, which the thread that meets it publishes
        auto failed = [&] { return err.load(std::memory_order_acquire) != (int)hipSuccess; };
        auto copy_block = [&](const Block& b) {
            if (b.dev < 0) {
                std::memcpy(b.dst, b.src, b.bytes);
                return;
            }
            while (issued.load(std::memory_order_acquire) <= b.dev) {
                if (failed()) return;
                std::this_thread::yield();
            }
            const int slot = (int)(b.dev % kSlots);
            const hipError_t e = hipEventSynchronize(ready_[slot]);
            if (e != hipSuccess) {
                err.store((int)e, std::memory_order_release);
                return;
            }
            std::memcpy(b.dst, mem_ + (size_t)slot * kBlock, b.bytes);
            drained[(size_t)b.dev].store(1, std::memory_order_release);
        };
        auto work = [&] {
            const hipError_t e = hipSetDevice(device);           // a thread's own setting
            if (e != hipSuccess) err.store((int)e, std::memory_order_release);
            for (size_t k; !failed() && (k = next.fetch_add(1, std::memory_order_relaxed)) < blocks.size();) copy_block(blocks[k]);
        };
        const size_t want = blocks.size() < (size_t)kMaxThreads ? blocks.size() : (size_t)kMaxThreads;
        for (size_t t = 0; t < want; ++t) {
            try {
                threads.emplace_back(work);
            } catch (...) {
                break;                   // no more threads to be had: fewer, or none
            }
        }
        auto enqueue = [&](size_t k) {
            const Block& b = blocks[dev_block[k]];
            const int slot = (int)(k % kSlots);
            hipError_t e = hipMemcpyAsync(mem_ + (size_t)slot * kBlock, b.src, b.bytes, hipMemcpyDeviceToHost, st);
            if (e == hipSuccess) e = hipEventRecord(ready_[slot], st);
            if (e != hipSuccess) err.store((int)e, std::memory_order_release);
            else issued.store((int64_t)k + 1, std::memory_order_release);
        };
        // a full ring: the calling thread lends a hand with the oldest block nobody has taken, or waits
        for (size_t k = 0; k < dev_block.size() && !failed(); ++k) {
            while (k >= (size_t)kSlots && !drained[k - kSlots].load(std::memory_order_acquire) && !failed()) {
                if (threads.empty()) {
                    const size_t b = next.fetch_add(1, std::memory_order_relaxed);
                    if (b < blocks.size()) copy_block(blocks[b]);
                } else {
                    std::this_thread::yield();
                }
            }
            if (!failed()) enqueue(k);
        }
        work();
        for (std::thread& t : threads) t.join();
        // after an error a copy into the ring may still be on its way
        if (failed()) (void)hipStreamSynchronize(st);
        return (hipError_t)err.load(std::memory_order_acquire);
    }

private:
    char* mem_ = nullptr;
    hipEvent_t ready_[kSlots] = {};
};

// Memory that the runtime neither allocated nor page-locked.
inline bool is_pageable(const void* p) {
    hipPointerAttribute_t a{};
    if (hipPointerGetAttributes(&a, p) != hipSuccess) {
        (void)hipGetLastError();
        return true;
    }
    return a.type == hipMemoryTypeUnregistered;
}

// Device and host-tier memory into the caller's buffer, which the parts fill from its beginning; every stream that could write
// the parts is idle.  Large reads into pageable memory take the ring.  Everything else takes plain copies: into page-locked
// memory one hipMemcpy runs at the link's rate (1M x 100 floats: 7.0 ms, through the ring 12.7; into pageable memory 22 to 38
// and 13), memory of the device the processor does not write, and of a small read the ring's set-up is the larger part.
inline hipError_t copy_parts(HostCopyRing& ring, const std::vector<HostCopyPart>& parts, int device, hipStream_t st) {
    size_t total = 0;
    for (const HostCopyPart& p : parts) total += p.bytes;
    if (total >= HostCopyRing::kMinBytes && is_pageable(parts[0].dst) && ring.prepare()) return ring.run(parts, device, st);
    for (const HostCopyPart& p : parts) {
        if (!p.on_device) {
            std::memcpy(p.dst, p.src, p.bytes);
            continue;
        }
        const hipError_t e = hipMemcpy(p.dst, p.src, p.bytes, hipMemcpyDeviceToHost);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace legend
