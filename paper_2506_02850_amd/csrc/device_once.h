// Something that is done once for every device of the process, in plain C++.
#pragma once

#include <stdint.h>

#include <atomic>

namespace metok {

// Calls `act` unless an earlier call for this device has succeeded; several threads may call at once, and `act` may then run in each of
// them.  false: no such device, or `act` failed, which the next call tries again.
template <typename Act>
bool once_per_device(std::atomic<uint64_t>& done, int device, Act act) {
    if (device < 0 || device >= 64) return false;
    const uint64_t bit = static_cast<uint64_t>(1) << device;
    if (done.load(std::memory_order_acquire) & bit) return true;
    if (!act()) return false;
    done.fetch_or(bit, std::memory_order_release);
    return true;
}

}  // namespace metok
