// The ragged last row tile of the tiled GEMM kernels of every operand format: a wavefront's accumulators to row-major memory.
#pragma once

#include "tree_walk.hpp"

namespace tbik {

// As the kernels store a full tile: the accumulators of a block row go through `patch` (32 x 32 NT floats of LDS, the
// wavefront's own), so that a lane holds consecutive columns of one row and stores 16 bytes.  `last` is the last row of the
// wavefront's tile that exists: lanes past it store that row once more, the same bytes to the same place, so a block row
// takes as many store instructions as a full one; block rows past it are skipped (uniformly).  Columns are whole and 16-byte
// aligned.  Stored value by value instead, two or four bytes a lane, the last row tile held a call up by 3 to 4 us:
// 1000 x 4096 x 4096 in 8 bits 25.0 us, 21.1 so; in bf16 42.1 and 39.3.
// (Full tiles keep code of their own: one copy of the two, with the rows clamped or with the choice inside, cost them 1 %.)
// A lane's offset inside a block row is 32 bits: with rows further apart than this (31 of them reach 2^31 bytes) a tile is
// stored value by value, with 64-bit addresses.
constexpr int64_t kMaxVectorRowBytes = (int64_t)1 << 26;

typedef unsigned int tile_u32x4 __attribute__((ext_vector_type(4)));

template <int MT, int NT>
__device__ __forceinline__ void fill_patch(const Acc<MT, NT> &acc, int a, float *patch, int lane) {
    const int li = lane & 31, lg = lane >> 5;
#pragma unroll
    for (int b = 0; b < NT; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) patch[(8 * (r >> 2) + 4 * lg + (r & 3)) * (32 * NT) + b * 32 + li] = acc.t[a][b][r];
}

// One 16-byte piece of 16-bit values, each rounded once from fp32.
template <bool F16>
__device__ __forceinline__ tile_u32x4 pack_8(const float *rd) {
    const f32x4 lo = *reinterpret_cast<const f32x4 *>(rd), hi = *reinterpret_cast<const f32x4 *>(rd + 4);
    tile_u32x4 o;
    o[0] = pack_16x2<F16>(lo[0], lo[1]);
    o[1] = pack_16x2<F16>(lo[2], lo[3]);
    o[2] = pack_16x2<F16>(hi[0], hi[1]);
    o[3] = pack_16x2<F16>(hi[2], hi[3]);
    return o;
}

// out: the first element of the wavefront's tile, ld in elements; to bf16 or binary16.
template <bool F16, int MT, int NT>
__device__ __forceinline__ void store_ragged_16bit(const Acc<MT, NT> &acc, float *patch, uint16_t *out, int64_t ld, int last, int lane) {
    constexpr int WCOLS = 32 * NT, CPR = WCOLS / 8, RPI = 64 / CPR, N_IT = 32 / RPI;      // 16-byte chunks per row, rows per store
    const int lrow = lane / CPR, lc = lane % CPR;
#pragma unroll
    for (int a = 0; a < MT; ++a) {
        if (last < 32 * a) continue;
        fill_patch(acc, a, patch, lane);
#pragma unroll
        for (int it = 0; it < N_IT; ++it) {
            const int row = min(lrow + it * RPI, last - 32 * a);
            *reinterpret_cast<tile_u32x4 *>(reinterpret_cast<char *>(out + a * 32 * ld) + (unsigned)(row * (int)ld + lc * 8) * 2u) =
                pack_8<F16>(patch + row * WCOLS + lc * 8);
        }
    }
}

// The same without a rounding; stream: the stores go around the caches.
template <int MT, int NT>
__device__ __forceinline__ void store_ragged_f32(const Acc<MT, NT> &acc, float *patch, float *out, int64_t ld, int last, int lane, bool stream) {
    constexpr int WCOLS = 32 * NT, CPR = WCOLS / 4, RPI = 64 / CPR, N_IT = 32 / RPI;
    const int lrow = lane / CPR, lc = lane % CPR;
#pragma unroll
    for (int a = 0; a < MT; ++a) {
        if (last < 32 * a) continue;
        fill_patch(acc, a, patch, lane);
#pragma unroll
        for (int it = 0; it < N_IT; ++it) {
            const int row = min(lrow + it * RPI, last - 32 * a);
            const f32x4 v = *reinterpret_cast<const f32x4 *>(patch + row * WCOLS + lc * 4);
            char *dst = reinterpret_cast<char *>(out + a * 32 * ld) + (unsigned)(row * (int)ld + lc * 4) * 4u;
            // (in assembly: written as two branches of ordinary code the compiler merges them and drops the hint)
            if (stream) asm volatile("global_store_dwordx4 %0, %1, off nt" ::"v"(dst), "v"(v) : "memory");
            else *reinterpret_cast<f32x4 *>(dst) = v;
        }
    }
}

}  // namespace tbik
