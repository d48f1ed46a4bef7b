// Data moved between the lanes of a wave without LDS.
#pragma once

#include <hip/hip_runtime.h>

namespace csph {

// The value of the lane N places on among the lane's row of 16 (every lane active).
template <int N>
__device__ __forceinline__ int row_ror(int v) {
    return __builtin_amdgcn_mov_dpp(v, 0x120 + N, 0xf, 0xf, true);
}
template <int N>
__device__ __forceinline__ double row_ror(double v) {
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)row_ror<N>((int)(unsigned)b);
    const unsigned hi = (unsigned)row_ror<N>((int)(unsigned)(b >> 32));
    return __longlong_as_double((long long)((unsigned long long)hi << 32 | lo));
}

}  // namespace csph
