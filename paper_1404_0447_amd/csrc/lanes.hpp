// Device helpers for kernels that keep a 16 x 16 block in one wave's
// registers: lane (m, g) = (l % 16, l / 16).
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

namespace selinv {

// f(integral_constant<int, I>) for I = I0 .. N - 1, each call with its own
// compile-time index (register arrays indexed by it stay in registers)
template <int I0, int N>
struct StaticFor {
    template <class Fn>
    __device__ __forceinline__ static void run(Fn&& f)
    {
        f(std::integral_constant<int, I0>{});
        StaticFor<I0 + 1, N>::run(f);
    }
};
template <int N>
struct StaticFor<N, N> {
    template <class Fn>
    __device__ __forceinline__ static void run(Fn&&)
    {
    }
};

// x of lane J of each row of 16 lanes, in every lane of the row
template <int J>
__device__ __forceinline__ double row_lane(double x)
{
    return __longlong_as_double(__builtin_amdgcn_update_dpp(0ll, __double_as_longlong(x), 0x150 + J, 0xF, 0xF, true));
}

// row G (of the wave's four rows of 16 lanes) of x in every row.  Rows of the
// two halves h, l of x side by side: swapping neighbouring rows gives
// (h0 l0 h2 l2) and (h1 l1 h3 l3); swapping halves with a copy (hG lG hG lG);
// swapping rows with a copy every h and every l.
template <int G>
__device__ __forceinline__ double row_copy(double x)
{
    const auto a = __builtin_amdgcn_permlane16_swap((unsigned)__double2hiint(x), (unsigned)__double2loint(x), false, false);
    const unsigned y = a[G & 1];
    const auto b = __builtin_amdgcn_permlane32_swap(y, y, false, false);
    const unsigned z = b[G >> 1];
    const auto c = __builtin_amdgcn_permlane16_swap(z, z, false, false);
    return __hiloint2double((int)c[0], (int)c[1]);
}

// the power of two s with |d| s in [1, 4), from d's exponent bits; 2^1023 for 0
__device__ __forceinline__ double pow2_scale(double d)
{
    return __hiloint2double(max(0x7FE00000 - (__double2hiint(d) & 0x7FF00000), 0x00100000), 0);
}
// 1 / f: one third-order step from the hardware's estimate, which is within
// 2^-24 of it (measured over [1, 4): the result within 2^-53)
__device__ __forceinline__ double recip3(double f)
{
    const double y = __builtin_amdgcn_rcp(f), h = fma(-f, y, 1.0);
    return fma(y, fma(h, h, h), y);
}

// one wave's LDS writes before its own reads of other lanes' values
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace selinv
