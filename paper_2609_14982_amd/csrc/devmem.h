// Several device arrays of one owner.
#pragma once

#include <hip/hip_runtime.h>

#include <vector>

namespace fm {

struct Part {
    void** p;
    size_t bytes;
};

// Arrays of up to 2 MB, 4 MB of them together, are allocations of their own,
// which the runtime takes from its pool (1 us each, 1 us to free); all others are
// one allocation, since each costs 270 us from 4 MB on, one at a time whichever
// thread asks, and the pool grows by chunks of 2 MB at a cost of their own.
// (All in one, 18 arrays of 42,000 nodes cost 360 us where 115 do; all alone,
// 8 sources on 101x101x51 spent 54 of 165 ms in 215 frees; up to 2 MB alone without
// the second limit, one source on 112x42x33 took 14.1 ms for 13.0.)
struct DevBlocks {
    std::vector<void*> blocks;

    hipError_t take(const std::vector<Part>& parts) {
        auto whole = [](size_t n) { return (n + 255) & ~size_t(255); };
        size_t small = 0;
        for (const Part& x : parts) small += x.bytes > kAlone ? 0 : whole(x.bytes);
        const size_t alone = small > 2 * kAlone ? 0 : kAlone;
        size_t rest = 0;
        for (const Part& x : parts) {
            if (x.bytes > alone) {
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
            if (x.bytes > alone) {
                *x.p = at;
                at += whole(x.bytes);
            }
        return hipSuccess;
    }

    void release() {
        for (void* p : blocks) (void)hipFree(p);
        blocks.clear();
    }

    static constexpr size_t kAlone = size_t(2) << 20;

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
