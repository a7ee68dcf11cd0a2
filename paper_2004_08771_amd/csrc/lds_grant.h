// More than 64 KB of dynamic LDS has to be asked for per kernel and device before the launch.
#pragma once

#include <stddef.h>

#include <mutex>

namespace hb {

// What has been granted to one kernel (or several that are launched with the same size), by device.  Handles on different
// host threads launch concurrently.
class LdsGrant {
public:
    // ask() -> error code, 0 if granted; called when `device` has not granted `bytes` yet
    template <typename Ask>
    auto ensure(int device, size_t bytes, Ask ask) -> decltype(ask())
    {
        if (device < 0 || device >= DEVICES) return ask();
        std::lock_guard<std::mutex> lk(mu_);
        if (bytes <= granted_[device]) return decltype(ask())(0);
        const auto e = ask();
        if (e == decltype(ask())(0)) granted_[device] = bytes;
        return e;
    }

private:
    static constexpr int DEVICES = 64;
    std::mutex mu_;
    size_t granted_[DEVICES] = {};
};

}  // namespace hb
