// Host build of what the device code does with the step counter
// (wcnst_device.hpp).
#include <hip/hip_runtime.h>

#include "wcnst_device.hpp"

extern "C" {

int sc_speed_slot(long long n) { return wcnst::speed_slot(n); }

// of the key that a stage of step `failed` leaves at cell c
unsigned sc_bad_stage(long long failed, int stage, long long c, long long n)
{
    const unsigned long long key = ((unsigned long long)(failed * 3 + stage) << 36) | (unsigned long long)c;
    return wcnst::bad_stage_of(key, n);
}

}  // extern "C"
