// A pixel's depths spread over a row of sixteen lanes (four pixels per
// wavefront): lane q holds the NP consecutive depths NP q .. NP q + NP - 1 and
// the segments that end at them.  Row shifts and reductions for float32 and
// float64, and the host's choice of NP.
#pragma once

#include "pz_internal.h"

namespace pz {

template <int CTRL>
__device__ __forceinline__ float row_move(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double row_move(double x) {
    const unsigned long long u = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)u, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
// shr<n> takes the value n lanes below, shl<n> n lanes above, within the row; zero enters.
template <int n, class T>
__device__ __forceinline__ T shr(T x) {
    return row_move<0x110 + n>(x);
}
template <int n, class T>
__device__ __forceinline__ T shl(T x) {
    return row_move<0x100 + n>(x);
}

// Sum and maximum over the row, the same value in every lane (a fixed order).
__device__ __forceinline__ double row_sum(double x) {
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) x += __shfl_xor(x, o, 64);
    return x;
}
__device__ __forceinline__ double row_max(double x) {
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) x = fmax(x, __shfl_xor(x, o, 64));
    return x;
}
// Whether every lane of this lane's row holds c.
__device__ __forceinline__ bool row_all(bool c) {
    const unsigned long long b = __builtin_amdgcn_ballot_w64(!c);
    return ((b >> (threadIdx.x & 48)) & 0xffffull) == 0;
}

// Depths per lane: the fewest that cover D on sixteen lanes, at least two so
// that lane 0 holds both depths of the surface extrapolation.
static_assert(MAXD <= 80, "five depths per lane");
__host__ __device__ constexpr int row_np(int D) { return D <= 32 ? 2 : (D + 15) / 16; }

}  // namespace pz
