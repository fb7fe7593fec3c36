// Host build of what the device code does with the step counter
// (wcnst_device.hpp).
#include <hip/hip_runtime.h>

#include "wcnst_device.hpp"

extern "C" {

int sc_speed_slot(long long n) { return wcnst::speed_slot(n); }

}  // extern "C"
