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

// the class mask's bits of finite nonzero values: 0x8 negative normal, 0x10
// negative denormal, 0x80 positive denormal, 0x100 positive normal
template <class T>
static inline bool in_class(T x, int mask)
{
    if (std::fpclassify(x) == FP_NORMAL) return (mask & (x > T(0) ? 0x100 : 0x8)) != 0;
    return std::fpclassify(x) == FP_SUBNORMAL && (mask & (x > T(0) ? 0x80 : 0x10)) != 0;
}
static inline bool __builtin_amdgcn_class(double x, int mask) { return in_class(x, mask); }
static inline bool __builtin_amdgcn_classf(float x, int mask) { return in_class(x, mask); }

// median of three; with a NaN among them the smallest of the others
static inline float __builtin_amdgcn_fmed3f(float a, float b, float c)
{
    if (std::isnan(a) || std::isnan(b) || std::isnan(c)) return std::fmin(a, std::fmin(b, c));
    return std::fmax(std::fmin(a, b), std::fmin(std::fmax(a, b), c));
}
