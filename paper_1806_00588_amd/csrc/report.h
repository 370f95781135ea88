// Pinned host words that a build's kernels report to (a copy of them from the device, and the wait for the copy, was
// 10 us of a build).  One page for the life of the process serves the builds that run at the same time; what it does
// not hold has memory of its own.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cstring>
#include <mutex>

namespace lshbeam {

struct Report {
    static constexpr int kPlaces = 16, kWords = 64;   // places of the page; words of a place, one per workgroup that may report
    uint32_t* words = nullptr;
    int place = -1;
    bool idle = true;   // no kernel that may write to it is under way
    inline static std::mutex mu;
    inline static uint32_t* page = nullptr;
    inline static uint32_t used = 0;   // bit i: place i
    hipError_t take() {
        constexpr size_t n = kWords * sizeof(uint32_t);
        {
            std::lock_guard<std::mutex> lock(mu);
            if (!page) {
                const hipError_t e = hipHostMalloc((void**)&page, kPlaces * n, hipHostMallocPortable);
                if (e != hipSuccess) { page = nullptr; return e; }
            }
            for (int i = 0; i < kPlaces && place < 0; ++i)
                if (!(used >> i & 1u)) { used |= 1u << i; place = i; words = page + (size_t)i * kWords; }
        }
        if (place < 0) {
            const hipError_t e = hipHostMalloc((void**)&words, n, hipHostMallocPortable);
            if (e != hipSuccess) { words = nullptr; return e; }
        }
        std::memset(words, 0, n);
        return hipSuccess;
    }
    ~Report() {
        if (words && place < 0) (void)hipHostFree(words);   // (waits)
        if (place < 0 || !idle) return;                     // (a build that failed with kernels under way: the place is lost)
        std::lock_guard<std::mutex> lock(mu);
        used &= ~(1u << place);
    }
};

}  // namespace lshbeam
