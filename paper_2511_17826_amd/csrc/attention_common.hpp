// What the attention kernels share: the constants that are part of the result, small helpers.
#pragma once

#include "tbik_device.hpp"
#include "tbik_internal.hpp"

namespace tbik {

constexpr int ATT_D = 128;    // head dimension
constexpr int ATT_BQ = 128;   // queries per workgroup
constexpr int ATT_KV = 64;    // keys per tile: part of the result, never tuned per call
constexpr int ATT_TILE_BYTES = ATT_KV * ATT_D * 2;
#ifndef TBIK_ATT_SPLIT
#define TBIK_ATT_SPLIT 64     // other values: timing experiments only (the bits change, the oracle's tests fail)
#endif
constexpr int ATT_SPLIT = TBIK_ATT_SPLIT;   // key tiles per split (4096 keys): part of the result as well

typedef short att_v4i16 __attribute__((ext_vector_type(4)));
typedef unsigned int att_u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int att_u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// A lane and its partner lane ^ 32 hold the two halves of one query's keys.  v_permlane32_swap exchanges the upper
// half of its first operand with the lower half of its second: from (v, v) it makes (lower half's values, upper
// half's values) in every lane, i.e. {mine, partner's} in some order -- enough for a maximum or a sum of the two.
__device__ __forceinline__ void both_halves(float v, float &a, float &b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    a = __uint_as_float(r[0]);
    b = __uint_as_float(r[1]);
}

}  // namespace tbik
