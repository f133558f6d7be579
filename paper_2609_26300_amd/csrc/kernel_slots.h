// kernel_slots.h -- the occupancy of a kernel, asked for once per kernel and device (host code, plain C++).
#pragma once

#include <atomic>
#include <cstdint>

namespace compkv {

struct Occupancy {
    int per_cu, cus;  // workgroups that fit a compute unit, compute units
};

// The occupancy of `Kern` on device `dev`; `query(Occupancy&)` asks the runtime and says whether it answered.
// Each kernel has words of its own, one per device, that hold a whole answer: threads that ask at once repeat the
// query and store the same word, and no kernel's answer takes another's place. A query that failed is
// not kept ({1, 1} for this call); devices past the array are asked each time.
template <auto Kern, typename Query>
Occupancy kernel_occupancy(int dev, Query query) {
    constexpr int kDevices = 16;
    static std::atomic<uint32_t> known[kDevices];
    const bool kept = dev >= 0 && dev < kDevices;
    if (kept) {
        const uint32_t w = known[dev].load(std::memory_order_relaxed);
        if (w != 0) return {(int)(w >> 16), (int)(w & 0xFFFFu)};
    }
    Occupancy o{1, 1};
    if (!query(o) || o.per_cu < 1 || o.cus < 1) return {1, 1};
    if (kept && o.per_cu < 0x10000 && o.cus < 0x10000)
        known[dev].store((uint32_t)o.per_cu << 16 | (uint32_t)o.cus, std::memory_order_relaxed);
    return o;
}

}  // namespace compkv
