// Host stand-ins for what the device building blocks take from HIP and from
// the compiler's gfx950 builtins, so that the arithmetic of physics.h runs
// on the CPU.  The estimates carry the hardware's accuracy and range: FP64
// ones about 24 correct bits; FP32 ones flush denormal arguments and results.
#pragma once

#include <cmath>
#include <cstdint>
#include <cstring>
#include <limits>

#define __device__
#define __forceinline__ inline

static inline uint64_t __ballot(int b) { return b != 0; }   // a wavefront of one lane

static inline double bits24(double x)
{
    if (!(std::fabs(x) < std::numeric_limits<double>::infinity())) return x;
    uint64_t u;
    std::memcpy(&u, &x, 8);
    u &= ~((1ull << 28) - 1);
    std::memcpy(&x, &u, 8);
    return x;
}
static inline float flush(float x) { return std::fabs(x) < std::numeric_limits<float>::min() ? std::copysign(0.0f, x) : x; }

static inline double __builtin_amdgcn_rcp(double x) { return bits24(1.0 / x); }
static inline double __builtin_amdgcn_rsq(double x) { return bits24(1.0 / std::sqrt(x)); }
static inline float __builtin_amdgcn_rcpf(float x) { return flush(1.0f / flush(x)); }
static inline float __builtin_amdgcn_rsqf(float x) { return (float)(1.0 / std::sqrt((double)flush(x))); }
static inline float __builtin_amdgcn_sqrtf(float x) { return std::sqrt(flush(x)); }

// the class mask's bits: 0x1 and 0x2 NaN, then from negative to positive
// infinity -inf 0x4, normal 0x8, denormal 0x10, -0 0x20, +0 0x40 and so on
template <class T>
static inline bool in_class(T x, int mask)
{
    int k;   // bits from the middle
    switch (std::fpclassify(x)) {
    case FP_NAN: return (mask & 0x3) != 0;
    case FP_ZERO: k = 0; break;
    case FP_SUBNORMAL: k = 1; break;
    case FP_NORMAL: k = 2; break;
    default: k = 3;
    }
    return (mask & (std::signbit(x) ? 0x20 >> k : 0x40 << k)) != 0;
}
static inline bool __builtin_amdgcn_class(double x, int mask) { return in_class(x, mask); }
static inline bool __builtin_amdgcn_classf(float x, int mask) { return in_class(x, mask); }

// median of three; with a NaN among them the smallest of the others
static inline float __builtin_amdgcn_fmed3f(float a, float b, float c)
{
    if (std::isnan(a) || std::isnan(b) || std::isnan(c)) return std::fmin(a, std::fmin(b, c));
    return std::fmax(std::fmin(a, b), std::fmin(std::fmax(a, b), c));
}
