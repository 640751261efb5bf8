// What a launcher finds out once per device (a raised kernel limit, a count of compute units) and keeps for the process.
// Plain C++.
#pragma once

#include <atomic>

namespace drc {

struct PerDevice {
    static constexpr int kSlots = 32;
    std::atomic<int> known[kSlots] = {};

    // The number kept for `dev`, found by find(&n) (0 on success, n > 0) on the first call for it.  Concurrent first calls
    // both look: same answer.  A failure is passed on and not kept; a device beyond the slots is looked up every time.
    template <typename F> int get(int dev, int* out, F find) {
        const bool kept = dev >= 0 && dev < kSlots;
        int n = kept ? known[dev].load(std::memory_order_acquire) : 0;
        if (n == 0) {
            if (const int rc = find(&n)) return rc;
            if (kept) known[dev].store(n, std::memory_order_release);
        }
        *out = n;
        return 0;
    }
};

}  // namespace drc
