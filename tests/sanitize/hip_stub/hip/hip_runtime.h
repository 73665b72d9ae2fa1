/* The few HIP names that the library's headers use, for host builds of device code that
 * consists of plain loads and stores. */
#pragma once
#include <cstdint>
#include <cstring>

#define __device__
#define __host__
#define __forceinline__ inline
#define __global__

typedef int hipError_t;
typedef void *hipStream_t;
struct int2 { int x, y; };
struct alignas(16) int4 { int x, y, z, w; };

inline uint32_t __umulhi(uint32_t a, uint32_t b) { return uint32_t((uint64_t(a) * b) >> 32); }
inline float __uint_as_float(uint32_t u) {
    float f;
    std::memcpy(&f, &u, 4);
    return f;
}
