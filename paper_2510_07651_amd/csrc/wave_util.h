// Reductions across the lanes of a wave without trips through LDS: data-parallel-primitive lane controls inside a row
// of 16 lanes, register exchanges between rows and halves (a shuffle is an LDS instruction with its latency; a chain of
// six of them is most of a short kernel).  Every lane must be active; all lanes end with the same bits.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace obc {

// x of the lane that the control pairs this lane with.  0xB1, 0x4E: neighbours, neighbouring pairs (quad permutes 1032
// and 2301); 0x141, 0x140: mirror image inside 8 and inside 16 lanes; 0x128: the lane 8 further in the row of 16.
template <int kCtrl>
__device__ __forceinline__ uint32_t dpp_pair(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kCtrl, 0xf, 0xf, false);
}
template <int kCtrl>
__device__ __forceinline__ float dpp_pair(float x) { return __uint_as_float(dpp_pair<kCtrl>(__float_as_uint(x))); }
template <int kCtrl>
__device__ __forceinline__ unsigned long long dpp_pair(unsigned long long x) {
    return ((unsigned long long)dpp_pair<kCtrl>((uint32_t)(x >> 32)) << 32) | dpp_pair<kCtrl>((uint32_t)x);
}

template <int kCtrl>
__device__ __forceinline__ double dpp_pair(double x) { return __longlong_as_double((long long)dpp_pair<kCtrl>((unsigned long long)__double_as_longlong(x))); }

// The values of the two lanes that differ in bit 4 (16) or 5 (32) of their index, lower one first.
template <int kBit>
__device__ __forceinline__ void both_of_pair(uint32_t x, uint32_t &lower, uint32_t &upper) {
    const auto r = kBit == 16 ? __builtin_amdgcn_permlane16_swap(x, x, false, false) : __builtin_amdgcn_permlane32_swap(x, x, false, false);
    lower = r[0];
    upper = r[1];
}
template <int kBit>
__device__ __forceinline__ void both_of_pair(float x, float &lower, float &upper) {
    uint32_t a, b;
    both_of_pair<kBit>(__float_as_uint(x), a, b);
    lower = __uint_as_float(a);
    upper = __uint_as_float(b);
}
template <int kBit>
__device__ __forceinline__ void both_of_pair(unsigned long long x, unsigned long long &lower, unsigned long long &upper) {
    uint32_t lh, uh, ll, ul;
    both_of_pair<kBit>((uint32_t)(x >> 32), lh, uh);
    both_of_pair<kBit>((uint32_t)x, ll, ul);
    lower = ((unsigned long long)lh << 32) | ll;
    upper = ((unsigned long long)uh << 32) | ul;
}

template <int kBit>
__device__ __forceinline__ void both_of_pair(double x, double &lower, double &upper) {
    unsigned long long a, b;
    both_of_pair<kBit>((unsigned long long)__double_as_longlong(x), a, b);
    lower = __longlong_as_double((long long)a);
    upper = __longlong_as_double((long long)b);
}

__device__ __forceinline__ unsigned long long min64(unsigned long long a, unsigned long long b) { return a < b ? a : b; }
struct SumOp { template <typename T> __device__ __forceinline__ T operator()(T a, T b) const { return a + b; } };
struct MaxOp { __device__ __forceinline__ float operator()(float a, float b) const { return fmaxf(a, b); } };
struct MinOp { __device__ __forceinline__ uint32_t operator()(uint32_t a, uint32_t b) const { return a < b ? a : b; } };

struct Min64Op { __device__ __forceinline__ unsigned long long operator()(unsigned long long a, unsigned long long b) const { return min64(a, b); } };

// Over each row of 16 lanes.
template <typename Op, typename T>
__device__ __forceinline__ T row16_reduce(T x) {
    const Op op;
    x = op(x, dpp_pair<0xB1>(x));
    x = op(x, dpp_pair<0x4E>(x));
    x = op(x, dpp_pair<0x141>(x));
    return op(x, dpp_pair<0x140>(x));
}
// Over the lanes of equal position in their row of 16.
template <typename Op, typename T>
__device__ __forceinline__ T across_rows(T x) {
    const Op op;
    T a, b;
    both_of_pair<16>(x, a, b);
    x = op(a, b);
    both_of_pair<32>(x, a, b);
    return op(a, b);
}
template <typename Op, typename T>
__device__ __forceinline__ T wave_reduce(T x) { return across_rows<Op>(row16_reduce<Op>(x)); }

// Unsigned 64-bit minimum: the high words first, then the low words of the lanes that hold it.
__device__ __forceinline__ unsigned long long wave_min(unsigned long long x) {
    const uint32_t hi = (uint32_t)(x >> 32), best = wave_reduce<MinOp>(hi);
    const uint32_t lo = wave_reduce<MinOp>(hi == best ? (uint32_t)x : 0xffffffffu);
    return ((unsigned long long)best << 32) | lo;
}

}  // namespace obc
