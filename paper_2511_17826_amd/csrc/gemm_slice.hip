// Tree-Based MatMul of up to 32 rows on 8-, 6- and 4-bit operands (decode batches) for gfx950, in one launch.
//
// The tiled kernels cut a small batch's K across workgroups to give every compute unit work, and a second launch combines
// the pieces.  A low-bit weight is stored transposed, one row of consecutive k per output channel, so here a workgroup takes
// a slice of 16 channels and all of K instead: its wavefronts take consecutive superleaves each (whole superleaves, in order:
// Sec. 4.2, App. D.1), the upper levels of the tree run over the wavefronts' sums in LDS (App. C), and the result is rounded
// and stored by the same launch.  Every wavefront streams its own part of the 16 weight rows and of the batch's rows through
// a ring of steps in LDS of its own (direct global->LDS loads of whole cache lines, no barrier until the sums are there).
// Eight wavefronts: with sixteen a wavefront's ring holds one or two steps, and 32 rows lose up to half (MXFP6).
// The matrix instruction, the lanes' bytes and the scales are those of the tiled kernels (v_mfma_scale_f32_32x32x64_f8f6f4;
// columns 16 .. 31 repeat 0 .. 15), so the bits are.
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "tbik_device.hpp"
#include "tbik_internal.hpp"

namespace tbik {

namespace {

template <int V>
using Int = std::integral_constant<int, V>;

typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x2 __attribute__((ext_vector_type(2)));

// Operand formats: FMT is the instruction's format code (0 E4M3, 1 E5M2, 2 E2M3, 3 E3M2, 4 E2M1).
template <int FMT, bool MX>
struct SliceFormat {
    static constexpr int bits = FMT < 2 ? 8 : FMT < 4 ? 6 : 4;
    static constexpr int step_k = FMT < 2 ? 128 : 256;                   // k of a step
    static constexpr int row_bytes = step_k * bits / 8;                  // of a row and step: 128, 192, 128
    static constexpr int chunks = row_bytes / 16;
    static constexpr int group_loads = 16 * chunks / 64;                 // 1 KiB loads of a group of 16 rows
    static constexpr int group_bytes = 16 * row_bytes;
    static constexpr int ksteps = step_k / 64;
    static constexpr int scale_bytes = MX ? step_k / 32 : 0;             // of a row and step
    // Where 16-byte chunk c of row r of a group lies in its row, so that the rows of a fragment read meet different banks.
    __device__ static constexpr int position(int c, int r) { return chunks == 8 ? c ^ ((r >> 1) & 7) : (c + (r >> 2)) % chunks; }
    __device__ static constexpr int chunk_at(int pos, int r) { return chunks == 8 ? pos ^ ((r >> 1) & 7) : (pos + chunks - (r >> 2)) % chunks; }
};

struct SliceParams {
    const uint8_t *X, *Wt, *Xs, *Ws;
    void *Y;
    int64_t ldx, ldw, ldxs, ldws, ldy;
    int M, N;
    int y_bf16;
    int steps_per_leaf;                 // superleaf / step_k
    int leaves_per_wave, active_waves;
};

template <int N>
__device__ __forceinline__ void slice_wait_loads() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// The last steps of a wavefront's stream: REST more are in flight behind the one that is waited for.
template <int REST, class Consume>
__device__ __forceinline__ void slice_tail(int steps, Consume &consume) {
    if (steps > REST) consume(Int<REST>{}, std::false_type{});
    if constexpr (REST > 0) slice_tail<REST - 1>(steps, consume);
}

// T over the wavefronts' sums of this thread's output element.
template <int WAVES>
__device__ __forceinline__ float slice_tree(const float *red, int active) {
    float v[WAVES];
#pragma unroll
    for (int w = 0; w < WAVES; ++w) v[w] = red[w < active ? w * 512 : 0];
#pragma unroll
    for (int s = 1; s < WAVES; s *= 2)
#pragma unroll
        for (int r = 0; r < WAVES; r += 2 * s)
            if (r + s < active) v[r] = v[r] + v[r + s];
    return v[0];
}

template <int FMT, bool MX, int GROUPS, int WAVES, int RING>
__global__ __launch_bounds__(64 * WAVES) void gemm_slice_kernel(const SliceParams p) {
    using F = SliceFormat<FMT, MX>;
    constexpr int DATA_BYTES = (1 + GROUPS) * F::group_bytes, STEP_BYTES = DATA_BYTES + (MX ? 512 : 0);
    constexpr int LOADS = (1 + GROUPS) * F::group_loads + (MX ? 2 : 0);
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int li = lane & 31, lg = lane >> 5;
    const int n0 = blockIdx.x * 16;
    float *const red = reinterpret_cast<float *>(smem);

    f32x16 acc;
    if (wave < p.active_waves) {
        const int steps = p.leaves_per_wave * p.steps_per_leaf;
        const int64_t k0 = (int64_t)wave * steps * F::step_k;
        // Load j of a group brings 64 chunks of its 16 rows in LDS order; rows past M or N re-read the last one (theirs are
        // never stored).  The instruction offset moves the LDS and the global address alike, hence the lane bias.
        const char *x_ptr = uniform_pointer(reinterpret_cast<const char *>(p.X + k0 * F::bits / 8));
        const char *w_ptr = uniform_pointer(reinterpret_cast<const char *>(p.Wt + n0 * p.ldw + k0 * F::bits / 8) - 4096);
        const char *xs_ptr = nullptr, *ws_ptr = nullptr;
        unsigned xoff[GROUPS][F::group_loads], woff[F::group_loads], xsoff = 0, wsoff = 0;
#pragma unroll
        for (int j = 0; j < F::group_loads; ++j) {
            const int at = j * 64 + lane, r = at / F::chunks, c = F::chunk_at(at % F::chunks, r);
            woff[j] = (unsigned)(min(r, p.N - 1 - n0) * (int)p.ldw + c * 16 + 4096 - j * 1024);
#pragma unroll
            for (int g = 0; g < GROUPS; ++g)
                xoff[g][j] = (unsigned)(min(16 * g + r, p.M - 1) * (int)p.ldx + c * 16 + ((GROUPS - g) * F::group_loads - j) * 1024);
        }
        if constexpr (MX) {                                            // a dword per lane: 8-bit, lane r a row; else lanes 2 r, 2 r + 1
            constexpr int per_row = F::scale_bytes / 4;
            const int r = lane / per_row % 32, d = lane % per_row;
            xs_ptr = uniform_pointer(reinterpret_cast<const char *>(p.Xs + k0 / 32));
            ws_ptr = uniform_pointer(reinterpret_cast<const char *>(p.Ws + n0 * p.ldws + k0 / 32) - 256);
            xsoff = (unsigned)(min(r, p.M - 1) * (int)p.ldxs + 4 * d);
            wsoff = (unsigned)(min(r & 15, p.N - 1 - n0) * (int)p.ldws + 4 * d);
        }
        // A step in LDS: X groups, then the W group (m0 points at it), then 256 bytes of X scales and 256 of W scales.
        const unsigned ring = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem + wave * RING * STEP_BYTES;
        auto issue = [&](int slot) __attribute__((always_inline)) {
            const unsigned m0v = ring + slot * STEP_BYTES + GROUPS * F::group_bytes;
            load_16B_per_lane_to_lds<0, true>(w_ptr, woff[0], m0v);
            load_16B_per_lane_to_lds<1024, false>(w_ptr, woff[1], m0v);
            if constexpr (F::group_loads > 2) load_16B_per_lane_to_lds<2048, false>(w_ptr, woff[F::group_loads - 1], m0v);
            constexpr int A = GROUPS * F::group_loads;
            static_assert(A <= 6 && F::group_loads >= 2 && F::group_loads <= 3, "loads of a step");
            const unsigned m0x = A > 4 ? m0v - 2048 : m0v;             // offsets reach -4 KiB
            constexpr int AO = A > 4 ? A - 2 : A;
            if constexpr (A > 4) {
                load_16B_per_lane_to_lds<(0 - AO) * 1024, true>(x_ptr - 2048, xoff[0][0], m0x);
                load_16B_per_lane_to_lds<(1 - AO) * 1024, false>(x_ptr - 2048, xoff[0][1], m0x);
                load_16B_per_lane_to_lds<(2 - AO) * 1024, false>(x_ptr - 2048, xoff[0][F::group_loads - 1], m0x);
                load_16B_per_lane_to_lds<(3 - AO) * 1024, false>(x_ptr - 2048, xoff[GROUPS - 1][0], m0x);
                load_16B_per_lane_to_lds<(4 - AO) * 1024, false>(x_ptr - 2048, xoff[GROUPS - 1][1], m0x);
                load_16B_per_lane_to_lds<(5 - AO) * 1024, false>(x_ptr - 2048, xoff[GROUPS - 1][F::group_loads - 1], m0x);
            } else {
                load_16B_per_lane_to_lds<(0 - A) * 1024, false>(x_ptr, xoff[0][0], m0v);
                load_16B_per_lane_to_lds<(1 - A) * 1024, false>(x_ptr, xoff[0][1], m0v);
                if constexpr (A == 3) load_16B_per_lane_to_lds<(2 - A) * 1024, false>(x_ptr, xoff[0][F::group_loads - 1], m0v);
                if constexpr (A == 4) {
                    load_16B_per_lane_to_lds<(2 - A) * 1024, false>(x_ptr, xoff[GROUPS - 1][0], m0v);
                    load_16B_per_lane_to_lds<(3 - A) * 1024, false>(x_ptr, xoff[GROUPS - 1][1], m0v);
                }
            }
            if constexpr (MX) {
                const unsigned m0s = ring + slot * STEP_BYTES + DATA_BYTES;
                load_4B_per_lane_to_lds<0, true>(xs_ptr, xsoff, m0s);
                load_4B_per_lane_to_lds<256, false>(ws_ptr, wsoff, m0s);
                xs_ptr += F::scale_bytes;
                ws_ptr += F::scale_bytes;
            }
            x_ptr += F::row_bytes;
            w_ptr += F::row_bytes;
        };
        // ---- a lane's fragments: row li of X (groups of 16), row li % 16 of the slice ----
        const int xr = GROUPS == 2 ? li : li & 15, r16 = li & 15;
        const int x_at = (xr >> 4) * F::group_bytes + r16 * F::row_bytes, w_at = GROUPS * F::group_bytes + r16 * F::row_bytes;
        constexpr int PIECES = FMT < 2 ? 2 : FMT < 4 ? 3 : 1;
        int piece[F::ksteps][PIECES];                                  // byte offset of a piece in the row's step
#pragma unroll
        for (int ks = 0; ks < F::ksteps; ++ks)
#pragma unroll
            for (int q = 0; q < PIECES; ++q) {
                if (FMT < 2) piece[ks][q] = F::position(4 * ks + 2 * q + lg, r16) << 4;         // as in the tiled kernel
                else if (FMT < 4) {
                    const int o = 24 * (2 * ks + lg) + 8 * q;
                    piece[ks][q] = (F::position(o >> 4, r16) << 4) + (o & 15);
                } else piece[ks][q] = F::position(2 * ks + lg, r16) << 4;
            }
        const unsigned char *const ring_rd = smem + wave * RING * STEP_BYTES;
        f32x16 stash[4];
        int left = p.steps_per_leaf, leaf = 0, slot = 0;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.0f;

        auto consume = [&](auto rest, auto again) __attribute__((always_inline)) {
            slice_wait_loads<decltype(rest)::value * LOADS>();
            const unsigned char *const s = ring_rd + slot * STEP_BYTES;
            union Fragment {
                i32x8 v;
                i32x4 h[2];
                i32x2 d[4];
            } a[F::ksteps], b[F::ksteps];
            unsigned sx[2] = {0, 0}, sw[2] = {0, 0};
#pragma unroll
            for (int ks = 0; ks < F::ksteps; ++ks) {
                a[ks].v = b[ks].v = i32x8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
                for (int q = 0; q < PIECES; ++q) {
                    if (FMT == 2 || FMT == 3) {
                        a[ks].d[q] = *reinterpret_cast<const i32x2 *>(s + x_at + piece[ks][q]);
                        b[ks].d[q] = *reinterpret_cast<const i32x2 *>(s + w_at + piece[ks][q]);
                    } else {
                        a[ks].h[q & 1] = *reinterpret_cast<const i32x4 *>(s + x_at + piece[ks][q]);
                        b[ks].h[q & 1] = *reinterpret_cast<const i32x4 *>(s + w_at + piece[ks][q]);
                    }
                }
            }
            if constexpr (MX) {
                const unsigned *xs = reinterpret_cast<const unsigned *>(s + DATA_BYTES + xr * F::scale_bytes);
                const unsigned *ws = reinterpret_cast<const unsigned *>(s + DATA_BYTES + 256 + r16 * F::scale_bytes);
#pragma unroll
                for (int d = 0; d < F::scale_bytes / 4; ++d) {
                    sx[d] = xs[d];
                    sw[d] = ws[d];
                }
            }
            if constexpr (decltype(again)::value) {                    // the step's bytes are in registers before its slot is filled again
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                issue(slot);
            }
#pragma unroll
            for (int ks = 0; ks < F::ksteps; ++ks) {
                if constexpr (MX) {                                    // the lane's block of the K-step: 2 ks + lg
                    const unsigned at = 16u * (ks & 1) + 8u * lg;
                    acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a[ks].v, b[ks].v, acc, FMT, FMT, 0, (int)__builtin_amdgcn_ubfe(sx[ks >> 1], at, 8u),
                                                                          0, (int)__builtin_amdgcn_ubfe(sw[ks >> 1], at, 8u));
                } else {
                    acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a[ks].v, b[ks].v, acc, FMT, FMT, 0, 0, 0, 0);
                }
            }
            slot = slot + 1 == RING ? 0 : slot + 1;
            if (--left == 0) {                                         // a superleaf ends: the carry-over step of the tree
                const int t = __builtin_ctz(~leaf);
#pragma unroll
                for (int l = 0; l < 4; ++l)
                    if (l < t) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) acc[r] = stash[l][r] + acc[r];
                    }
                left = p.steps_per_leaf;
                if (++leaf < p.leaves_per_wave) {
#pragma unroll
                    for (int l = 0; l < 4; ++l)
                        if (l == t) stash[l] = acc;
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
                }
            }
        };
#pragma unroll
        for (int i = 0; i < RING; ++i)
            if (i < steps) issue(i);
        for (int s = RING; s < steps; ++s) consume(Int<RING - 1>{}, std::true_type{});
        slice_tail<RING - 1>(steps, consume);
    }
    __syncthreads();                                                   // the rings have been read: the sums take their place
    if (wave < p.active_waves && li < 16) {
#pragma unroll
        for (int r = 0; r < 16; ++r) red[wave * 512 + (8 * (r >> 2) + 4 * lg + (r & 3)) * 16 + li] = acc[r];
    }
    __syncthreads();
    const int row = threadIdx.x >> 4, col = n0 + (threadIdx.x & 15);
    if (threadIdx.x >= 512 || row >= p.M || col >= p.N) return;
    const float v = slice_tree<WAVES>(red + threadIdx.x, p.active_waves);
    if (p.y_bf16) reinterpret_cast<uint16_t *>(p.Y)[(int64_t)row * p.ldy + col] = (uint16_t)f32_to_bf16_bits(v);
    else reinterpret_cast<float *>(p.Y)[(int64_t)row * p.ldy + col] = v;
}

constexpr int SLICE_WAVES = 8;
inline int64_t slices_of(int N) { return ((int64_t)N + 15) / 16; }

template <int FMT, bool MX, int GROUPS, int RING, int WAVES = SLICE_WAVES>
hipError_t launch_slice_of(const GemmArgs &a, const Mxfp4Scales &sc, hipStream_t s) {
    using F = SliceFormat<FMT, MX>;
    SliceParams p;
    p.X = reinterpret_cast<const uint8_t *>(a.X); p.Wt = reinterpret_cast<const uint8_t *>(a.W);
    p.Xs = sc.Xs; p.Ws = sc.Ws;
    p.Y = a.Y;
    p.ldx = a.ldx; p.ldw = a.ldw; p.ldxs = sc.ldxs; p.ldws = sc.ldws; p.ldy = a.ldy;
    p.M = a.M; p.N = a.N;
    p.y_bf16 = a.y_dtype != TBIK_F32;
    p.steps_per_leaf = a.superleaf / F::step_k;
    p.leaves_per_wave = a.ns > WAVES ? a.ns / WAVES : 1;
    p.active_waves = a.ns > WAVES ? WAVES : a.ns;
    constexpr int lds = WAVES * RING * ((1 + GROUPS) * F::group_bytes + (MX ? 512 : 0));
    static_assert(lds <= 160 * 1024 && lds >= WAVES * 2048, "LDS of a compute unit; room for the sums");
    auto k = gemm_slice_kernel<FMT, MX, GROUPS, WAVES, RING>;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 32) dev = 32;      // 32: not remembered, set every time
    static std::atomic<unsigned> lds_allowed{0};                                 // bit d: the attribute is set on device d
    if (dev >= 32 || !((lds_allowed.load(std::memory_order_relaxed) >> dev) & 1u)) {
        hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        if (dev < 32) lds_allowed.fetch_or(1u << dev, std::memory_order_relaxed);
    }
    hipLaunchKernelGGL(k, dim3((unsigned)slices_of(a.N)), dim3(64 * WAVES), lds, s, p);
    return hipGetLastError();
}

// Steps in flight: all that LDS holds while every workgroup has a compute unit to itself; with more of them than compute units
// two, which lets two workgroups share one (16 rows of 4096 x 6144 in 8 bits 10.4 -> 8.8 us; 17 .. 32 rows and 6-bit steps are
// too large for that).
template <int FMT, bool MX>
hipError_t launch_slice_rows(const GemmArgs &a, const Mxfp4Scales &sc, hipStream_t s) {
    constexpr bool six_bits = FMT == 2 || FMT == 3;
    if (a.M > 16) return launch_slice_of<FMT, MX, 2, six_bits ? 2 : 3>(a, sc, s);
    if (!six_bits && slices_of(a.N) > 256) return launch_slice_of<FMT, MX, 1, 2>(a, sc, s);
    return launch_slice_of<FMT, MX, 1, six_bits ? 3 : 4>(a, sc, s);
}

}  // namespace

// Where slices are the quicker way.  What bounds them is what a compute unit takes in: its 16 weight rows and the whole batch
// (and, for 8-bit elements, a cache line per row and 128 k for the scales); the tiled kernels read less of the batch per
// compute unit and spread K over up to 16 workgroups, but pay a second launch and the planes' round trip where they do.  So
// slices begin ahead by that launch and lose with K:
//   ahead = launch + K / 4096 (k + narrow min(N, 4096) / 4096 - (N > 4096 ? wide : 0) - rows M / 16)      us
// More channels up to 4096 are free for slices (a workgroup per compute unit) and cost the tiles; above, workgroups share compute
// units or wait for one.  The constants are those with which wrong choices cost least over 1868 timed pairs (1 .. 32 rows, K = 2048 ..
// 24576, 256 .. 12288 channels; the geometric mean of weights from HBM and from the memory-side cache): the route takes at most 1.11 of
// the quicker one's time, 1.001 in the mean (profiles/slices_or_tiles.csv).  Device time of a call in a HIP graph, tiled kernel
// (with its combine) / slices, weights from HBM and from the cache, us:
//   1 x 4096 x 4096       8-bit 9.4 / 6.0, 6.8 / 3.8      MXFP8 10.1 / 6.3, 7.4 / 4.7    MXFP6 10.2 / 5.8, 7.8 / 4.8     MXFP4 8.8 / 4.5, 6.9 / 3.5
//   16 rows, K = 12288    8-bit 15.4 / 12.6, 15.1 / 9.2   MXFP8 17.8 / 16.4, 14.1 / 10.9 MXFP6 17.6 / 13.5, 13.4 / 10.1  MXFP4 13.0 / 9.6, 9.6 / 6.6
//   32 rows, K = 12288    8-bit 16.1 / 16.4, 14.0 / 10.4                                 MXFP6 18.4 / 16.5, 14.3 / 11.7  MXFP4 14.7 / 11.9, 11.2 / 8.0
//   with N = 6144 (tiles) 8-bit 20.9 / 28.6, 17.2 / 18.1                                                                 MXFP4 18.6 / 20.6, 13.7 / 14.8
//   16 rows, K = 8192, N = 1024  8-bit 8.9 / 7.3, 7.3 / 4.7      MXFP8 10.7 / 9.0, 8.2 / 6.9       MXFP6 10.9 / 8.6, 8.5 / 6.8
//   K = 24576 there (tiles)      8-bit 12.8 / 17.6, 9.5 / 10.5   MXFP8 16.5 / 27.3, 11.9 / 17.1    MXFP6 16.9 / 21.6, 11.7 / 12.9
struct SliceGain {
    double launch, k, narrow, wide, rows;
};
constexpr SliceGain kSliceGains[4][2] = {                                         // [format][17 .. 32 rows]
    {{4.46, -0.87, 0.68, 0.44, 0.16}, {4.22, -1.01, 1.00, 2.14, 0.35}},           // 8-bit
    {{3.05, -0.75, 1.08, 0.64, 0.82}, {7.21, -3.14, 1.02, 0.0, 0.39}},            // MXFP8
    {{3.51, -0.55, 0.44, 0.34, 0.26}, {4.83, -0.88, 0.39, 1.09, 0.16}},           // MXFP4
    {{3.74, -0.78, 0.60, 0.34, 0.19}, {4.80, -1.13, 0.82, 0.44, 0.26}},           // MXFP6
};

static bool slices_are_quicker(const GemmArgs &a, bool eight_bits, bool scaled) {
    const bool second_group = a.M > 16, six_bits = a.x_dtype == TBIK_FP6_E2M3 || a.x_dtype == TBIK_FP6_E3M2;
    const int64_t slices = slices_of(a.N);
    // Not measured beyond these.
    if (slices > (!second_group || !eight_bits ? 768 : scaled ? 256 : 384)) return false;
    if (second_group && eight_bits && scaled && a.K > 8192) return false;
    if (a.ns < 8) {
        // Fewer superleaves than wavefronts: the other wavefronts idle, but the tiled kernels cannot spread K either.  One superleaf, 16
        // rows, K = 4096: N = 4096 8-bit 14.3 / 8.3, 8.8 / 6.8, MXFP8 24.1 / 8.9, MXFP4 14.4 / 5.9; N = 12288 8-bit 16.4 / 24.6, 10.5 / 16.5,
        // MXFP8 26.0 / 36.4, MXFP4 15.2 / 20.4.  Short K bears twice as many slices (N = 8192, K = 2048 in 8 bits 9.2 / 8.0, 6.3 / 4.7),
        // and so do 17 .. 32 rows of MXFP4 (16.2 / 12.0, 9.9 / 9.6 at K = 4096).  MXFP6's tiles have 128 rows only: 26.9 / 20.3, 18.3 / 18.4 at
        // N = 12288; at K = 512 6.4 / 7.2, 4.9 / 6.0.
        if (slices <= 256) return true;
        const bool four_bits = !eight_bits && !six_bits;
        const int short_k = second_group ? (four_bits ? 4096 : 0) : four_bits ? 2048 : scaled ? 512 : 8192;
        if (six_bits ? slices > 512 && a.K < 2048 && a.ns < 4
                     : slices > std::max((a.K <= short_k ? 512 : 256) * a.ns, four_bits && second_group ? 512 : 0)) return false;
        if (a.ns < 4) return true;
    }
    const SliceGain &g = kSliceGains[eight_bits ? (scaled ? 1 : 0) : six_bits ? 3 : 2][second_group];
    const double ahead = g.launch + a.K * (1.0 / 4096) * (g.k + g.narrow * std::min(a.N, 4096) * (1.0 / 4096) - (a.N > 4096 ? g.wide : 0.0) - g.rows * a.M * (1.0 / 16));
    return ahead > 0.0;
}

bool gemm_slice_takes(const GemmArgs &a, const Mxfp4Scales *sc) {
    const bool eight_bits = a.x_dtype == TBIK_FP8_E4M3 || a.x_dtype == TBIK_FP8_E5M2;
    if (a.M > 32 || a.P != 1 || !a.Y) return false;
    if (a.superleaf % (eight_bits ? 128 : 256) != 0 || a.ns > 16 * SLICE_WAVES) return false;      // whole steps; four levels per wavefront
    if (a.ldx >= (1 << 22) || a.ldw >= (1 << 22)) return false;                     // 32-bit lane offsets
    if (sc) {
        auto a4 = [](const void *q) { return (reinterpret_cast<uintptr_t>(q) & 3) == 0; };
        if (!a4(sc->Xs) || !a4(sc->Ws) || sc->ldxs % 4 != 0 || sc->ldws % 4 != 0 || sc->ldxs >= (1 << 24) || sc->ldws >= (1 << 24)) return false;
    }
    return slices_are_quicker(a, eight_bits, sc != nullptr);
}

hipError_t launch_gemm_slice(const GemmArgs &a, const Mxfp4Scales *sc, hipStream_t s) {
    if (a.M <= 0 || a.N <= 0) return hipSuccess;
    if (!gemm_slice_takes(a, sc)) return hipErrorInvalidValue;
    static const Mxfp4Scales none{};
    const Mxfp4Scales &scales = sc ? *sc : none;
    switch (a.x_dtype) {
        case TBIK_FP8_E4M3: return sc ? launch_slice_rows<0, true>(a, scales, s) : launch_slice_rows<0, false>(a, scales, s);
        case TBIK_FP8_E5M2: return sc ? launch_slice_rows<1, true>(a, scales, s) : launch_slice_rows<1, false>(a, scales, s);
        case TBIK_FP6_E2M3: return launch_slice_rows<2, true>(a, scales, s);
        case TBIK_FP6_E3M2: return launch_slice_rows<3, true>(a, scales, s);
        case TBIK_MXFP4: return launch_slice_rows<4, true>(a, scales, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace tbik
