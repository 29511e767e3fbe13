// Makes a device current for the lifetime of an object.
#pragma once

#include <hip/hip_runtime_api.h>

namespace cube {

struct DeviceGuard {
  int cur = -1, dev;
  explicit DeviceGuard(int d) : dev(d) {
    if (hipGetDevice(&cur) != hipSuccess) cur = dev;
    if (cur != dev) (void)hipSetDevice(dev);
  }
  ~DeviceGuard() {
    if (cur != dev) (void)hipSetDevice(cur);
  }
  DeviceGuard(const DeviceGuard&) = delete;
  DeviceGuard& operator=(const DeviceGuard&) = delete;
};

}  // namespace cube
