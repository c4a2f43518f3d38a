// Largest of two values where a NaN of either stays a NaN: a running maximum that
// starts from finite values is NaN at the end if any value was.  (With "if (!(x <= m)) m
// = x" a NaN enters m but leaves it again at the next finite value, since every
// comparison with NaN is false.)  Host and device.
#pragma once

#if defined(__HIPCC__)
#define DF_HOST_DEVICE __host__ __device__
#else
#define DF_HOST_DEVICE
#endif

namespace df {

DF_HOST_DEVICE inline float max_nan(float a, float b) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_elementwise_maximum(a, b);   // v_maximum3_f32
#else
    return (a != a || a >= b) ? a : b;            // (b a NaN: a >= b is false)
#endif
}

}  // namespace df
