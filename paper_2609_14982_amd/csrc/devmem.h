// Several device arrays of one owner.
#pragma once

#include <hip/hip_runtime.h>

#include <vector>

namespace fm {

struct Part {
    void** p;
    size_t bytes;
};

// An array of up to 2 MB is an allocation of its own, which the runtime takes
// from its pool (1 us, 1 us to free); the larger ones are one allocation
// together, since each would cost 270 us from 4 MB on, one at a time whichever
// thread asks.  (All in one, 18 arrays of 42,000 nodes cost 360 us where 115 do;
// each alone, 8 sources on 101x101x51 spent 54 of 165 ms in 215 frees.)
struct DevBlocks {
    std::vector<void*> blocks;

    hipError_t take(const std::vector<Part>& parts) {
        constexpr size_t kPool = size_t(2) << 20;
        auto whole = [](size_t n) { return (n + 255) & ~size_t(255); };
        size_t rest = 0;
        for (const Part& x : parts) {
            if (x.bytes > kPool) {
                rest += whole(x.bytes);
                continue;
            }
            const hipError_t e = add(x.p, x.bytes);
            if (e != hipSuccess) return e;
        }
        if (!rest) return hipSuccess;
        void* block = nullptr;
        const hipError_t e = add(&block, rest);
        if (e != hipSuccess) return e;
        char* at = (char*)block;
        for (const Part& x : parts)
            if (x.bytes > kPool) {
                *x.p = at;
                at += whole(x.bytes);
            }
        return hipSuccess;
    }

    void release() {
        for (void* p : blocks) (void)hipFree(p);
        blocks.clear();
    }

private:
    hipError_t add(void** p, size_t bytes) {
        blocks.reserve(blocks.size() + 1);
        const hipError_t e = hipMalloc(p, bytes > 256 ? bytes : 256);
        if (e != hipSuccess) {
            *p = nullptr;
            return e;
        }
        blocks.push_back(*p);
        return hipSuccess;
    }
};

}  // namespace fm
