// Host stand-in for the few HIP names that csrc/device_math.hpp uses, so that
// its arithmetic can be checked on the CPU.  The hardware estimates of a
// reciprocal and a reciprocal square root are the exact values off by a
// relative error of up to 4.5e-8 (gfx950: below 5e-8) that depends on the bits.
#pragma once
#include <cmath>
#include <cstdint>
#include <cstring>

#define __device__
#define __host__
#define __forceinline__ inline

using std::fma;

static inline double off(double x) {
    uint64_t b;
    std::memcpy(&b, &x, 8);
    b *= 0x9e3779b97f4a7c15ull;
    b = (b ^ (b >> 29)) * 0xbf58476d1ce4e5b9ull;
    return 1.0 + 4.5e-8 * (double((b ^ (b >> 32)) >> 11) * 0x1p-52 - 1.0);
}
static inline double __builtin_amdgcn_rcp(double x) { return 1.0 / x * off(x); }
static inline double __builtin_amdgcn_rsq(double x) { return 1.0 / std::sqrt(x) * off(x); }
static inline float __builtin_amdgcn_rcpf(float x) { return 1.0f / x; }
static inline float __builtin_amdgcn_rsqf(float x) { return 1.0f / std::sqrt(x); }
static inline float __builtin_amdgcn_sqrtf(float x) { return std::sqrt(x); }
static inline float __builtin_amdgcn_fmed3f(float a, float b, float c) {
    return std::fmax(std::fmin(a, b), std::fmin(std::fmax(a, b), c));
}
static inline int __double2hiint(double x) {
    uint64_t b;
    std::memcpy(&b, &x, 8);
    return int(b >> 32);
}
static inline unsigned long long __shfl_xor(unsigned long long v, int, int) { return v; }
