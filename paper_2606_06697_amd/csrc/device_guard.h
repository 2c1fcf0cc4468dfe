// Makes a HIP device current for the lifetime of the object and restores the previous one.
#pragma once
#include <hip/hip_runtime.h>

namespace agile {

struct DeviceGuard {
    int prev = -1;
    bool ok = false, changed = false;
    explicit DeviceGuard(int dev) {
        if (hipGetDevice(&prev) != hipSuccess) return;
        changed = prev != dev;
        ok = !changed || hipSetDevice(dev) == hipSuccess;
    }
    ~DeviceGuard() {
        if (changed) (void)hipSetDevice(prev);
    }
    DeviceGuard(const DeviceGuard&) = delete;
    DeviceGuard& operator=(const DeviceGuard&) = delete;
};

}  // namespace agile
