// Stand-in for the HIP header in host builds of device code: the qualifiers, the
// bit casts and the instructions that csrc/math64.hpp uses. The reciprocal and the
// reciprocal square root are the exact ones moved by `seed_error`, the largest
// relative error their instructions are documented with (2^29 ulp).
#pragma once
#include <cmath>
#include <cstdint>
#include <cstring>

#define __device__
#define __forceinline__ inline

struct HostIndex {
    int x;
};
static HostIndex threadIdx{0}, blockDim{1};
static double seed_error = 0.0;

inline uint64_t host_bits(double x) { uint64_t u; std::memcpy(&u, &x, 8); return u; }
inline double host_double(uint64_t u) { double x; std::memcpy(&x, &u, 8); return x; }
inline int __double2hiint(double x) { return (int)(host_bits(x) >> 32); }
inline int __double2loint(double x) { return (int)host_bits(x); }
inline double __hiloint2double(int h, int l) { return host_double(((uint64_t)(uint32_t)h << 32) | (uint32_t)l); }
inline long long __double_as_longlong(double x) { return (long long)host_bits(x); }
inline double __longlong_as_double(long long b) { return host_double((uint64_t)b); }

inline double host_rsq(double x) { return 1.0 / std::sqrt(x) * (1.0 + seed_error); }
inline double host_rcp(double x) { return 1.0 / x * (1.0 + seed_error); }
#define __builtin_amdgcn_rsq host_rsq
#define __builtin_amdgcn_rcp host_rcp
#define __builtin_amdgcn_ldexp(x, e) std::ldexp(x, e)
#define __builtin_amdgcn_class(x, mask) ((x) == 0.0 || (x) == INFINITY) /* mask 0x260 */
