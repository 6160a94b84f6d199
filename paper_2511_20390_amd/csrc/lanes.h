// Exchanges between the lanes of a wavefront on the vector ALU.  __shfl_xor is a ds_bpermute: an LDS round trip of some 100 cycles
// per step, six of them in a row in a sum over the wavefront.  A permlane swap or a DPP move takes a few cycles, and the sums are the
// same, pair by pair.  us per launch at width 1152, __shfl_xor -> these: LayerNorm of 256 rows 4.45 -> 3.93, of 512 rows behind
// split sums 8.1 -> 7.7, of 1024 rows 5.47 -> 5.08 and 9.9 -> 9.3 behind split sums.  All 64 lanes take part.  Device code.
#pragma once

#include "free_internal.h"

namespace freemi {

namespace {

// the value of lane ^ X within 16 lanes: X = 1, 2 within four lanes; 4 by two mirrors, i -> 7 - i and i -> 3 - i; 8 by a rotation
template <int X>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
    static_assert(X == 1 || X == 2 || X == 4 || X == 8, "within a row of 16 lanes");
    const int i = static_cast<int>(v);
    if constexpr (X == 1) return __builtin_amdgcn_update_dpp(0, i, 0xB1, 0xf, 0xf, true);              // quad_perm 1, 0, 3, 2
    else if constexpr (X == 2) return __builtin_amdgcn_update_dpp(0, i, 0x4E, 0xf, 0xf, true);         // quad_perm 2, 3, 0, 1
    else if constexpr (X == 4)
        return __builtin_amdgcn_update_dpp(0, __builtin_amdgcn_update_dpp(0, i, 0x141, 0xf, 0xf, true), 0x1B, 0xf, 0xf, true);
    else return __builtin_amdgcn_update_dpp(0, i, 0x128, 0xf, 0xf, true);                              // row_ror 8
}

template <int X>
__device__ __forceinline__ float lane_xor(float v) {
    return __uint_as_float(lane_xor<X>(__float_as_uint(v)));
}

// v + the value of lane ^ X, X = 16 or 32 (a swap leaves the two values in its two results, in either order)
template <int X>
__device__ __forceinline__ float add_lane_xor(float v) {
    static_assert(X == 16 || X == 32, "between rows of 16 lanes");
    typedef uint32_t pair_t __attribute__((ext_vector_type(2)));
    const uint32_t b = __float_as_uint(v);
    pair_t r;
    if constexpr (X == 32) r = __builtin_amdgcn_permlane32_swap(b, b, false, false);
    else r = __builtin_amdgcn_permlane16_swap(b, b, false, false);
    const uint32_t r0 = r[0], r1 = r[1];
    return __uint_as_float(r0) + __uint_as_float(r1);
}

template <int X>
__device__ __forceinline__ double add_lane_xor(double v) {
    typedef uint32_t pair_t __attribute__((ext_vector_type(2)));
    const uint64_t b = static_cast<uint64_t>(__double_as_longlong(v));
    const uint32_t lo = static_cast<uint32_t>(b), hi = static_cast<uint32_t>(b >> 32);
    if constexpr (X >= 16) {
        pair_t l, h;
        if constexpr (X == 32) {
            l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
            h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
        } else {
            l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
            h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
        }
        const uint32_t l0 = l[0], l1 = l[1], h0 = h[0], h1 = h[1];
        return __longlong_as_double(static_cast<int64_t>(static_cast<uint64_t>(h0) << 32 | l0)) +
               __longlong_as_double(static_cast<int64_t>(static_cast<uint64_t>(h1) << 32 | l1));
    } else {
        return v + __longlong_as_double(static_cast<int64_t>(static_cast<uint64_t>(lane_xor<X>(hi)) << 32 | lane_xor<X>(lo)));
    }
}

// the larger of v and the value of lane ^ 32
__device__ __forceinline__ float max_lane_xor32(float v) {
    typedef uint32_t pair_t __attribute__((ext_vector_type(2)));
    const uint32_t b = __float_as_uint(v);
    const pair_t r = __builtin_amdgcn_permlane32_swap(b, b, false, false);
    const uint32_t r0 = r[0], r1 = r[1];
    return fmaxf(__uint_as_float(r0), __uint_as_float(r1));
}

// the sum over the 64 lanes, in every lane: halves added from the widest distance down
__device__ __forceinline__ float wave_sum(float v) {
    v = add_lane_xor<32>(v);
    v = add_lane_xor<16>(v);
    v += lane_xor<8>(v);
    v += lane_xor<4>(v);
    v += lane_xor<2>(v);
    return v + lane_xor<1>(v);
}

__device__ __forceinline__ double wave_sum(double v) {
    v = add_lane_xor<32>(v);
    v = add_lane_xor<16>(v);
    v = add_lane_xor<8>(v);
    v = add_lane_xor<4>(v);
    v = add_lane_xor<2>(v);
    return add_lane_xor<1>(v);
}

}  // namespace
}  // namespace freemi
