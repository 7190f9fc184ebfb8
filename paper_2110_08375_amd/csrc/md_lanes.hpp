// md_lanes.hpp -- one multiple-double scalar spread over the lanes of a wave.
//
// The panel's chain forms a few scalars per column (a square root and two reciprocals) that every lane
// would otherwise compute alike, thousands of instructions one after the other.  Here a value is a row of
// digits, lane k holding d_k with value sum_k d_k 2^(-24 k) (times a power of two the caller keeps), each
// d_k an integer of at most 24 bits and sign in a double, so that a product's columns c_k = sum_i a_i
// b_(k-i) are exact in double (at most 20 products below 2^47): one broadcast, one FMA and one shift by a
// lane per digit of a.  Fixed point: the digits reach 2^-456, below the last limb of an od value in [1/4, 4).
// (qd keeps the limbs: its scalars are short enough that the spread form was 5% slower.)  A product takes about 130 instructions in place of 970, the square
// root with its reciprocal 1.1 K in place of 6 K, and the code is short enough to stay in the instruction
// cache.
#pragma once

#include "mdls_kernels.hpp"

namespace mdk {
namespace lanes {

constexpr int kDigits = 20;  // digit 0 is the integer part
constexpr double kBase = 16777216.0;  // 2^24

// lane k takes lane k - 1's value (lane 0 zero), and lane k + 1's (the last lane zero): DPP shifts
// of the whole wave by one
__device__ __forceinline__ double shift_up(double x)
{
    const long long b = __double_as_longlong(x);
    const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x138, 0xf, 0xf, true);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x138, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

__device__ __forceinline__ double shift_down(double x)
{
    const long long b = __double_as_longlong(x);
    const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)b, 0x130, 0xf, 0xf, true);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x130, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

__device__ __forceinline__ double lane_value(double x, int k)
{
    const long long b = __double_as_longlong(x);
    const unsigned lo = __builtin_amdgcn_readlane((int)b, k);
    const unsigned hi = __builtin_amdgcn_readlane((int)(b >> 32), k);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Carries moved up: columns below 2^52 come out as digits of at most 2^23 + 2^5 (lane 0 keeps what it gets).
__device__ __forceinline__ double carry(double c, int lane)
{
    const double inv = lane == 0 ? 0.0 : 1.0 / kBase;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        const double q = __builtin_rint(c * inv);
        c = __builtin_fma(-kBase, q, c) + shift_down(q);
    }
    return c;
}

// a b with the first N digits of a; carried
template <int N>
__device__ __forceinline__ double mul(double a, double b, int lane)
{
    double c = 0.0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        c = __builtin_fma(lane_value(a, i), b, c);
        if (i + 1 < N) b = shift_up(b);
    }
    return carry(c, lane);
}

// digits of x 2^-e, |x 2^-e| < 2^22: every limb rounded to each digit's grid, less what the digits above took
template <int NL>
__device__ __forceinline__ double digits(const double *x, int e, int lane)
{
    double d = 0.0;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const double a = lane < kDigits ? __builtin_rint(__builtin_ldexp(x[i], 24 * lane - e)) : 0.0;
        const double up = shift_up(a);
        d += lane < kDigits ? __builtin_fma(-kBase, up, a) : 0.0;
    }
    return d;
}

// the value of carried digits times 2^e as P limbs, in every lane.  Two digits make an exact double, and those
// do not overlap, so FastTwoSum is exact (a zero above a nonzero one included).
template <int P>
__device__ __forceinline__ V<P> limbs(double d, int e)
{
    constexpr int N = kDigits / 2;
    const double v = __builtin_fma(shift_down(d), 1.0 / kBase, d);
    double x[N];
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = __builtin_ldexp(lane_value(v, 2 * i), e - 48 * i);
    // limb k: the rest summed from the bottom, its errors the rest of limb k + 1 (one pass from the top would
    // leave two limbs where a sum comes out exact)
    V<P> r;
#pragma unroll
    for (int k = 0; k < P; ++k) {
        double s = x[N - 1];
#pragma unroll
        for (int i = N - 2; i >= k; --i) {
            if (k < P - 1)
                fast_two_sum(x[i], s, s, x[i + 1]);
            else
                s = x[i] + s;
        }
        r.x[k] = s;
    }
    return r;
}

// 1/sqrt(Q) for Q in [1, 4), q its leading double.  y (1 + e/2 + 3 e^2/8) with e = 1 - Q y^2 triples the bits:
// 52 -> 154 -> 460.  e/2 + 3 e^2/8 is kept as eighths, and the product's eighths are brought back to whole digits
// one lane further down (2^-3 = 2^21 2^-24).
__device__ __forceinline__ double rsqrt(double Q, double q, int lane)
{
    const double y0 = 1.0 / sqrt(q);
    double y = digits<1>(&y0, 0, lane);
    auto refine = [&](auto n, auto m, auto k) __attribute__((always_inline)) {
        const double t = mul<decltype(m)::value>(mul<decltype(n)::value>(y, y, lane), Q, lane);
        const double e = (lane == 0 ? 1.0 : 0.0) - t;
        const double u = carry(__builtin_fma(3.0, mul<decltype(k)::value>(e, e, lane), 4.0 * e), lane);
        const double v = mul<decltype(n)::value>(y, u, lane);
        y = carry(y + carry(shift_up(v * 2097152.0), lane), lane);
    };
    refine(std::integral_constant<int, 4>{}, std::integral_constant<int, 8>{}, std::integral_constant<int, 8>{});
    y = lane < 8 ? y : 0.0;
    refine(std::integral_constant<int, 8>{}, std::integral_constant<int, 16>{}, std::integral_constant<int, 14>{});
    return y;
}

// 1/X for X in [1, 4), x its leading double: z (1 + r + r^2) with r = 1 - X z
__device__ __forceinline__ double recip(double X, double x, int lane)
{
    const double z0 = 1.0 / x;
    double z = digits<1>(&z0, 0, lane);
    auto refine = [&](auto n, auto k) __attribute__((always_inline)) {
        const double r = (lane == 0 ? 1.0 : 0.0) - mul<decltype(n)::value>(z, X, lane);
        const double u = carry(r + mul<decltype(k)::value>(r, r, lane), lane);
        z = carry(z + mul<decltype(n)::value>(z, u, lane), lane);
    };
    refine(std::integral_constant<int, 4>{}, std::integral_constant<int, 8>{});
    z = lane < 8 ? z : 0.0;
    refine(std::integral_constant<int, 8>{}, std::integral_constant<int, 14>{});
    return z;
}

}  // namespace lanes
}  // namespace mdk
