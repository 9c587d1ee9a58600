// Device memory of freed plaintext and ciphertext handles, kept for the next handle of about the same size: freeing a large
// block costs a quarter of a millisecond.  Bounded (KEEP_EACH, KEEP_ALL); emptied when the context is freed, or when an
// allocation of the library fails.  Shared by the context and its handles, which may outlive it, and safe with several threads.  The
// release of a block waits for nothing; taking one waits for the device, as hipFree did when the block was freed.
#pragma once
#include <hip/hip_runtime_api.h>
#include <stddef.h>

#include <map>
#include <mutex>
#include <new>

struct DevPool {
    static constexpr size_t KEEP_EACH = (size_t)256 << 20, KEEP_ALL = (size_t)1 << 30;
    std::mutex mu;
    std::multimap<size_t, void *> blocks;  // by size
    size_t held = 0;
    bool closed = false;

    // hipMalloc, with the kept blocks given back first if the card is full
    hipError_t alloc(void **p, size_t bytes) {
        void *block = nullptr;
        hipError_t e = hipMalloc(&block, bytes);
        if (e == hipErrorOutOfMemory) {
            release();
            (void)hipGetLastError();
            e = hipMalloc(&block, bytes);  // also where nothing was kept: another thread may just have given it back
        }
        if (e != hipSuccess) (void)hipGetLastError();  // the caller has it: a later call that asks for launch errors must not find it
        *p = block;
        return e;
    }
    // A kept block, or a new one; *got: its size.
    hipError_t take(void **p, size_t bytes, size_t *got) {
        void *block = nullptr;
        {
            std::lock_guard<std::mutex> lock(mu);
            auto it = blocks.lower_bound(bytes);
            if (it != blocks.end() && it->first <= bytes + bytes / 8) {
                block = it->second;
                *got = it->first;
                held -= it->first;
                blocks.erase(it);
            }
        }
        if (block) {
            if (hipDeviceSynchronize() == hipSuccess) {
                *p = block;
                return hipSuccess;
            }
            // the device cannot be waited for now (a stream of this thread is being captured): the block stays, a new one serves
            (void)hipGetLastError();
            give(block, *got);
        }
        *got = bytes;
        return alloc(p, bytes);
    }
    void give(void *p, size_t bytes) {
        try {
            std::lock_guard<std::mutex> lock(mu);
            if (!closed && bytes <= KEEP_EACH && held + bytes <= KEEP_ALL) {
                blocks.emplace(bytes, p);
                held += bytes;
                return;
            }
        } catch (const std::bad_alloc &) {  // no host memory to note the block down: handles are freed from C, where nothing may throw
        }
        (void)hipFree(p);
    }
    void release() {
        std::lock_guard<std::mutex> lock(mu);
        for (auto &b : blocks) (void)hipFree(b.second);
        blocks.clear();
        held = 0;
    }
    void close() {
        {
            std::lock_guard<std::mutex> lock(mu);
            closed = true;
        }
        release();
    }
    ~DevPool() { close(); }
};
