// Work-groups per CU of one kernel by launch shape.
#pragma once
#include <stdint.h>

#include <algorithm>
#include <atomic>

namespace nbb {

// The answers for the last few (LDS bytes, threads) asked for, from any number
// of host threads: descriptors of one kernel have LDS sizes of their own, and
// with one answer kept two of them stepped in turn asked on every launch (3.43
// to 3.57 us of host time per call, 3.32 to 3.45 with these; one descriptor
// alone 3.3 to 3.4).  A full table replaces its entries in turn; a lost race
// only asks again.
class OccupancyCache {
   public:
    // 1..255, or what `query(&value)` returns where that is an error (not 0).
    template <typename Query>
    auto get(uint32_t lds, uint32_t threads, int *per_cu, Query query) -> decltype(query(per_cu)) {
        const uint64_t key = uint64_t(lds) << 32 | uint64_t(threads) << 8;
        for (const std::atomic<uint64_t> &s : slot_) {
            const uint64_t v = s.load(std::memory_order_relaxed);
            if ((v & ~uint64_t(0xFF)) == key && (v & 0xFF)) {
                *per_cu = int(v & 0xFF);
                return decltype(query(per_cu))(0);
            }
        }
        const auto e = query(per_cu);
        if (int(e) != 0) return e;
        *per_cu = std::max(1, std::min(*per_cu, 255));
        slot_[next_.fetch_add(1, std::memory_order_relaxed) % kSlots].store(key | uint64_t(*per_cu),
                                                                            std::memory_order_relaxed);
        return e;
    }

   private:
    static constexpr uint32_t kSlots = 8;
    std::atomic<uint64_t> slot_[kSlots] = {};
    std::atomic<uint32_t> next_{0};
};

}  // namespace nbb
