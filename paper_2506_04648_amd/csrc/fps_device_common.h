// Device helpers shared by the data-movement kernels of libfps (not part of the ABI).
#pragma once
#include "fps_internal.h"

namespace fps {

// Where a block of BS packed slots sits: its tile, the real box of its SUB-TILE and its first slot
// within the sub-tile.  Computed once per workgroup (the divisions are by run-time values).
struct BlockOrigin {
    RealBox box;
    long long tile_lin;  // bh * M + u
    int slot_base;       // first tiled slot of the sub-tile within its tile
    long long raster0;   // raster token index of the sub-tile's first token
    int slot0;           // first in-sub-tile packed slot of the block
};
__device__ __forceinline__ BlockOrigin block_origin(const Geom& g, int blk) {
    BlockOrigin o;
    const int group = quotient(blk, g.KBS, g.rc_kbs);           // 32-bit: the block count fits a grid dimension
    o.slot0 = (blk - group * g.KBS) * g.BS;
    const int tile_lin = quotient(group, g.NS, g.rc_ns), s = group - tile_lin * g.NS;
    const int bh = quotient(tile_lin, g.M, g.rc_m);
    const int u = tile_lin - bh * g.M;
    const int ut = quotient(u, g.nW * g.nH, g.rc_layer), rem = u - ut * (g.nW * g.nH);
    const int uh = quotient(rem, g.nW, g.rc_row), uw = rem - uh * g.nW;
    o.box = real_box(g, ((ut == g.nT - 1) << 2) | ((uh == g.nH - 1) << 1) | (uw == g.nW - 1), s);
    o.tile_lin = tile_lin;
    o.slot_base = s * g.QSP;
    o.raster0 = (((long long)bh * g.T + ut * g.Tt + o.box.o.t0) * g.H + uh * g.Th + o.box.o.h0) * g.W +
                uw * g.Tw + o.box.o.w0;
    return o;
}

// The 16 uint4 (256 bytes) of the bf16 row of the token in packed slot r of the block with origin o,
// in a TILED or RASTER input; nullptr for padding.
template <bool RASTER>
__device__ __forceinline__ const uint4* token_row(const uint4* x, const Geom& g, const BlockOrigin& o, int r) {
    const int k = o.slot0 + r;
    if (k >= o.box.n) return nullptr;
    // rows and planes of a sub-tile that is whole along h and w follow each other in a tiled tensor
    if (!RASTER && o.box.plane == g.Qh * g.Qw) return x + (o.tile_lin * g.TSP + o.slot_base + k) * 16;
    const Offset d = real_token(o.box, k);
    const long long row = RASTER ? o.raster0 + ((long long)d.t * g.H + d.h) * g.W + d.w
                                 : o.tile_lin * g.TSP + o.slot_base + (d.t * g.Qh + d.h) * g.Qw + d.w;
    return x + row * 16;
}

// max of the 15-bit magnitude patterns of 8 bf16 values (|x| of bf16 orders like that integer),
// two patterns per instruction: the running maximum m2 holds one candidate in each 16-bit half
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t amax_pairs16(const uint4& v, uint32_t m2) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    u16x2 m = __builtin_bit_cast(u16x2, m2);
#pragma unroll
    for (int i = 0; i < 4; ++i) m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, w[i] & 0x7FFF7FFFu));
    return __builtin_bit_cast(uint32_t, m);
}
__device__ __forceinline__ uint32_t amax_of_pairs(uint32_t m2) {        // the larger half
    const uint32_t lo = m2 & 0xFFFFu, hi = m2 >> 16;
    return lo > hi ? lo : hi;
}
// the larger of a lane's m and that of lane ^ 16, lane ^ 32
__device__ __forceinline__ uint32_t max_with_lane_16(uint32_t m) {
    const auto r = __builtin_amdgcn_permlane16_swap(m, m, false, false);
    return r[0] > r[1] ? r[0] : r[1];
}
__device__ __forceinline__ uint32_t max_with_lane_32(uint32_t m) {
    const auto r = __builtin_amdgcn_permlane32_swap(m, m, false, false);
    return r[0] > r[1] ? r[0] : r[1];
}
// max of m over a wave, and over a workgroup of WAVES waves (red: WAVES words of LDS); every thread gets it, and behind
// workgroup_max what the workgroup has written to its LDS before.  Lanes exchange through the vector unit: six trips through the
// LDS, one after the other, are 0.3 us of a small launch.
__device__ __forceinline__ uint32_t wave_max(uint32_t m) {
    auto rotated = [&](auto n) {                            // that of the lane n further on, in its row of 16
        const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x120 + decltype(n)::value, 0xf, 0xf, false);
        m = o > m ? o : m;
    };
    rotated(Count<8>{}); rotated(Count<4>{}); rotated(Count<2>{}); rotated(Count<1>{});
    return max_with_lane_32(max_with_lane_16(m));
}
template <int WAVES>
__device__ __forceinline__ uint32_t workgroup_max(uint32_t m, uint32_t* red) {
    m = wave_max(m);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    m = red[0];
#pragma unroll
    for (int i = 1; i < WAVES; ++i) m = red[i] > m ? red[i] : m;
    return m;
}

__device__ __forceinline__ int pow2_exponent_for_fp16(float amax) {   // e with amax*2^-e in [2^14,2^15)
    const uint32_t bits = __float_as_uint(amax);
    int e = (int)((bits >> 23) & 0xFF) - 127 - 14;
    return bits == 0 ? 0 : (e < -100 ? -100 : (e > 113 ? 113 : e));
}

// small in-place helpers (static: each translation unit that launches them has its own copy)
static __global__ void clear_kernel(uint32_t* p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}
static __global__ void amax_to_scale_kernel(float* p, int n) {       // amax -> amax/448 (1 for 0)
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) { const float a = p[i]; p[i] = a == 0.0f ? 1.0f : a / 448.0f; }
}
static __global__ void amax_to_pow2_kernel(float* p, int n) {        // amax -> 2^e (see above)
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = __uint_as_float((uint32_t)(127 + pow2_exponent_for_fp16(p[i])) << 23);
}
// a load that, if NT, leaves nothing in the caches
template <bool NT>
__device__ __forceinline__ uint4 load_chunk(const uint4* p) {
    if (!NT) return *p;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p)));
}
// N of the 16-byte chunks of a block that THREADS threads hold, chunk c = 8 channels (c & 15) of slot c >> 4: v[i] of
// thread tid is chunk tid + THREADS (first + i), zero for padding.  All N loads are in flight at once.
template <bool RASTER, int THREADS, bool NT = false, int N>
__device__ __forceinline__ void load_chunks(const uint4* x, const Geom& g, const BlockOrigin& o, int tid, int first,
                                            uint4 (&v)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const uint4* row = token_row<RASTER>(x, g, o, (tid >> 4) + THREADS / 16 * (first + i));
        v[i] = make_uint4(0, 0, 0, 0);
        if (row) v[i] = load_chunk<NT>(row + (tid & 15));
    }
}

// amax over the KBS blocks of each quantisation group, merged with an atomic max on the float bit
// pattern (amax_bits must be cleared first).  A workgroup of 256 threads takes one block of 128 slots, or
// four of 32, one a wave: finding out where a block sits costs a wave more than reading its 8 KB.
template <int BS, bool RASTER>
__global__ __launch_bounds__(256) void block_amax_kernel(const uint4* __restrict__ x,
                                                         uint32_t* __restrict__ amax_bits, Geom g, int blocks) {
    constexpr int THREADS = BS == 128 ? 256 : 64;
    __shared__ uint32_t red[THREADS / 64];
    const int blk = BS == 128 ? blockIdx.x : blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (BS != 128 && blk >= blocks) return;
    const int tid = BS == 128 ? threadIdx.x : threadIdx.x & 63;
    uint4 v[BS * 16 / THREADS];
    load_chunks<RASTER, THREADS>(x, g, block_origin(g, blk), tid, 0, v);
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < BS * 16 / THREADS; ++i) m = amax_pairs16(v[i], m);
    m = amax_of_pairs(m);
    m = BS == 128 ? workgroup_max<4>(m, red) : wave_max(m);
    if (tid == 0) atomicMax(&amax_bits[blk / g.KBS], m << 16);
}
template <int BS>
static void launch_block_amax(const void* x, int raster, float* amax, const Geom& g, hipStream_t st) {
    const int blocks = g.BH * g.M * g.KB, grid = BS == 128 ? blocks : (blocks + 3) / 4;
    const uint4* xi = (const uint4*)x;
    if (raster) block_amax_kernel<BS, true><<<grid, 256, 0, st>>>(xi, (uint32_t*)amax, g, blocks);
    else        block_amax_kernel<BS, false><<<grid, 256, 0, st>>>(xi, (uint32_t*)amax, g, blocks);
}

}  // namespace fps
