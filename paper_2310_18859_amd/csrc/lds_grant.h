// A kernel's permission to be launched with more dynamic LDS than 64 KiB.  Host code, checked without a GPU.
#pragma once

#include <atomic>
#include <cstdint>

namespace sida {

// The runtime holds the permission per device: it is asked for by the first launch on each, and again by the
// next launch where that failed.  Launches may come from several threads (asking twice does no harm).
class LdsGrant {
public:
    // ask() returns 0 when the permission has been given on the current device, which is `device`.
    template <class Ask>
    int on(int device, Ask &&ask)
    {
        const uint64_t bit = device >= 0 && device < 64 ? uint64_t(1) << device : 0;   // others ask every time
        if (given_.load(std::memory_order_acquire) & bit) return 0;
        const int rc = ask();
        if (rc == 0) given_.fetch_or(bit, std::memory_order_release);
        return rc;
    }

private:
    std::atomic<uint64_t> given_{0};
};

}  // namespace sida
