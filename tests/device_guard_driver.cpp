// Test-only driver of csrc/device_guard.h over a fake device runtime.
#include "../paper_1712_06121_amd/csrc/device_guard.h"

static int current = 0, fails = 0;

hipError_t hipGetDevice(int* d) {
  if (fails) return hipErrorUnknown;
  *d = current;
  return hipSuccess;
}
hipError_t hipSetDevice(int d) {
  current = d;
  return hipSuccess;
}

// the device that is current inside a guard for `dev`, and behind it
extern "C" int inside(int before, int dev, int no_answer, int* after) {
  current = before;
  fails = no_answer;
  int in = -1;
  {
    cube::DeviceGuard on(dev);
    in = current;
  }
  *after = current;
  return in;
}
