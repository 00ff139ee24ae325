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

// row G (of the wave's four rows of 16 lanes) in every row: halves, then
// neighbouring rows swapped between two copies
template <int G>
__device__ __forceinline__ unsigned row_copy32(unsigned x)
{
    const auto a = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    const unsigned y = (G & 2) ? a[1] : a[0];
    const auto b = __builtin_amdgcn_permlane16_swap(y, y, false, false);
    return (G & 1) ? b[1] : b[0];
}
template <int G>
__device__ __forceinline__ double row_copy(double x)
{
    return __hiloint2double((int)row_copy32<G>((unsigned)__double2hiint(x)),
                            (int)row_copy32<G>((unsigned)__double2loint(x)));
}

}  // namespace selinv
