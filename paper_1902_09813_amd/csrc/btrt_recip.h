// 1/d of the moment forms' per-node K1 with the bits of an IEEE division.
#pragma once

#include <hip/hip_runtime.h>

namespace btrtk {

// 1/d: the hardware reciprocal and Newton steps with fused multiply-adds, and the division's own handling of
// infinities, zeros and NaN (det M overflows to 1/d = 0). FP32 takes one step: measured on gfx950 over every
// significand, d up to 2^126, it is the IEEE quotient each time (above, where the quotient is subnormal, 0).
// FP64 takes three: two leave it within half an ulp and 2^-40, and from there the third rounds correctly (P.
// Markstein, IBM J. Res. Dev. 34 (1990): if it starts within an ulp of 1/d, for any significand but the all-ones
// one); over 6e9 divisors (log-uniform from 2^-3 up, around powers of two, just below them and around reciprocals
// of midpoints) it is the IEEE quotient each time, where two steps miss 3085 of the 5e8 just below a power of two.
// Instructions: 4 and 8, against about 10 and 12 of a division.
template <typename T>
__host__ __device__ __forceinline__ T quotient(T d)
{
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (sizeof(T) == 4) {
        const T r = __builtin_amdgcn_rcpf(d);
        return __builtin_amdgcn_div_fixupf(fmaf(r, fmaf(-d, r, T(1)), r), d, T(1));
    } else {
        T r = __builtin_amdgcn_rcp(d);
        r = fma(r, fma(-d, r, T(1)), r);
        r = fma(r, fma(-d, r, T(1)), r);
        return __builtin_amdgcn_div_fixup(fma(r, fma(-d, r, T(1)), r), d, T(1));
    }
#else
    return T(1) / d;
#endif
}

}  // namespace btrtk
