// Layout kernels of libfps: raster <-> tile order (Sec. 3.2 step (1)), the BF16 operand packing,
// and the debug unpacking of packed E4M3 tensors.  All of them are pure data movement.
//
// Packed operand layouts, per sub-block of 32 packed slots (a block of BS = 128 or 32 slots is four of them
// or one, a tile one or several blocks; packed slots hold the real tokens of a scale group first, see
// real_box in fps_internal.h); lane = 32h + n.
// E4M3 -- operands of v_mfma_f32_32x32x64_f8f6f4, h the half of the 64 contraction slots of one step:
//   Q : row-major [token][128]                                              (4 KB)
//   K : 16-byte chunk ((ks*2 + e)*64 + lane) = K[n][64ks + 32h + 16e + 0..15]
//   V : 16-byte chunk (db*64 + lane), byte jj = V[key][32db + n] with key = 8(jj/4) + 4h + jj%4
//   The accumulator of S^T = K Q^T for a sub-block holds, in lane (n,h) and register r, query n and key
//   8(r/4) + 4h + r%4; the 32 weights of two sub-blocks of a lane are therefore, unchanged, its 32
//   contraction slots of one step of the PV product O^T = V^T P^T, and 8 of them those of a
//   32x32x16 step.
// BF16 -- operands of the 32x32x16 instructions:
//   Q : row-major [token][128]                                              (8 KB)
//   K : 16-byte chunk (ks*64 + lane) = K[n][16ks + 8h + 0..7]
//   V : 16-byte chunk ((kk*4 + db)*64 + lane), element el = V[key][32db + n] with
//       key = 16kk + 8(el/4) + 4h + el%4 (the key order of the accumulator), stored as fp16 after an
//       exact power-of-two scaling per scale group (see pack_bf16_kernel)
#include "fps_device_common.h"


namespace fps {

// ---- raster <-> tiled: 16-byte chunks, CPR of them a token -----------------------------------------
// Bound by HBM.  A wave's slots, 32 or a part of 32, lie in one sub-tile: where that is costs scalar instructions once, a
// slot's place in it two products by stored reciprocals.  With a chunk a thread and its place by 64-bit divisions, 12
// heads x 21x30x52 tokens in (1,8,16) tiles took 52 us to tile order and 47 back, now 36 and 35; 24 heads in (2,8,16)
// tiles with sub-tiles of 64 tokens 107 and 91 us, now 78 and 73 (6.1 and 5.5 TB/s).
// NT: the input is read past the caches, for tensors that do not fit them (launch_reorder).
// U: loads in flight of a wave.  8: all 32 slots, in fp32 16 and then 16; 4: two or four waves share the 32.
template <int CPR, int U> constexpr int kWavesOfSegment = U == 8 ? 1 : 32 * CPR / (64 * U);
template <int CPR, bool TO_TILES, bool NT, int U>
__global__ __launch_bounds__(256) void reorder_kernel(const uint4* __restrict__ in, uint4* __restrict__ out, Geom g,
                                                      int waves) {
    constexpr int SLOTS = 64 * U / CPR;                 // the slots that the loads cover
    constexpr int PARTS = kWavesOfSegment<CPR, U>;
    const int wave = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), seg = wave / PARTS;
    if (wave >= waves) return;
    const int lane = threadIdx.x & 63, c = lane & (CPR - 1), per_block = g.BS >> 5;      // 4 or 1
    const int blk = per_block == 1 ? seg : seg >> 2;
    const BlockOrigin org = block_origin(g, blk);
    const int slot0 = org.slot0 + 32 * (seg & (per_block - 1)) + SLOTS * (wave % PARTS);    // in the sub-tile
    const long long tiled0 = org.tile_lin * g.TSP + org.slot_base + slot0;
#pragma unroll
    for (int first = 0; first < 32 / PARTS; first += SLOTS) {
        uint4 v[U];
        long long row[U];                               // in the raster tensor; -1: padding
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int r = first + 64 / CPR * i + lane / CPR, k = slot0 + r;
            const int t = div_by_recip(k, g.inv_plane[0][0]), rem = k - t * (g.Qh * g.Qw);
            const int h = div_by_recip(rem, g.inv_w[0]), w = rem - h * g.Qw;
            const bool token = k < g.QS && t * org.box.plane < org.box.n && h < org.box.eh && w < org.box.ew;
            row[i] = token ? org.raster0 + ((long long)t * g.H + h) * g.W + w : -1;
            v[i] = make_uint4(0, 0, 0, 0);
            if (token) v[i] = load_chunk<NT>(in + (TO_TILES ? row[i] : tiled0 + r) * CPR + c);
        }
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int r = first + 64 / CPR * i + lane / CPR;
            if (TO_TILES)         out[(tiled0 + r) * CPR + c] = v[i];
            else if (row[i] >= 0) out[row[i] * CPR + c] = v[i];
        }
    }
}

// ---- BF16 operand packing -----------------------------------------------------------------------
// One workgroup of 256 threads per block of BS tokens; the block (BS*256 bytes) is staged in LDS.
// Q and K keep their bf16 values.  V is converted to fp16 so that the PV product can take P in
// fp16 (11 significant bits instead of bf16's 8): each TILE is first multiplied by 2^-e with
// amax * 2^-e in [2^14, 2^15), which keeps every bf16 value exact unless it is more than 2^28
// times smaller than the tile's largest one, and vscale[tile] = 2^e undoes it in the kernel.
// For tiles of several blocks the tile amax is computed beforehand (tile_amax != nullptr).
// RASTER: `in` is the raster tensor and the block's tokens are gathered from it (padding slots read
// as zero), which fuses the tile ordering into this pass.
// Bound by HBM, small calls by latency.  Loads in flight: all of a thread's for V, which has to have the block
// anyway; two for K and one for Q, between stores -- at 720p (40 heads) a Q of all loads, then all stores takes 284
// instead of 264 us, although it is the faster one at 480p (40.7 against 45.7 us).
template <int BS, bool RASTER>
__global__ __launch_bounds__(256) void pack_bf16_kernel(const uint4* __restrict__ in,
                                                        uint4* __restrict__ out,
                                                        float* __restrict__ vscale, int role, Geom g,
                                                        const float* __restrict__ tile_amax) {
    constexpr int THREADS = 256, U = BS * 16 / THREADS;    // U: 16-byte chunks per thread
    __shared__ __attribute__((aligned(16))) uint16_t tile[BS * 128];
    __shared__ uint32_t red[THREADS / 64];
    const long long blk = blockIdx.x;
    uint4* dst = out + blk * (BS * 16);
    const BlockOrigin org = block_origin(g, blockIdx.x);
    if (role != FPS_ROLE_V) {
        auto copy = [&](auto n_tag) __attribute__((always_inline)) {       // N chunks at a time
            constexpr int N = decltype(n_tag)::value;
#pragma unroll
            for (int first = 0; first < U; first += N) {
                uint4 v[N];
                load_chunks<RASTER, THREADS>(in, g, org, threadIdx.x, first, v);
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    int c = threadIdx.x + THREADS * (first + i);
                    if (role == FPS_ROLE_K) {              // 32x32x16 operand: lane 32h + n, step ks
                        const int j = c >> 4, c8 = c & 15; // row, 8-channel chunk
                        const int sb = j >> 5, n = j & 31, ks = c8 >> 1, h = c8 & 1;
                        c = (sb * 8 + ks) * 64 + 32 * h + n;
                    }
                    dst[c] = v[i];
                }
                __builtin_amdgcn_sched_barrier(0);         // the next loads follow these stores
            }
        };
        if (role == FPS_ROLE_Q) copy(Count<1>{});
        else                    copy(Count<2>{});
        return;
    }
    uint4 v[U];
    load_chunks<RASTER, THREADS>(in, g, org, threadIdx.x, 0, v);
    uint4* t4 = reinterpret_cast<uint4*>(tile);
    uint32_t mb = 0;
#pragma unroll
    for (int i = 0; i < U; ++i) {
        t4[threadIdx.x + THREADS * i] = v[i];
        mb = amax_pairs16(v[i], mb);
    }
    float amax;
    if (tile_amax) {
        amax = tile_amax[blk / g.KBS];
        __syncthreads();
    } else {
        mb = workgroup_max<THREADS / 64>(amax_of_pairs(mb), red);   // also orders the LDS writes above
        amax = __uint_as_float(mb << 16);
    }
    const int e = pow2_exponent_for_fp16(amax);
    const float down = __uint_as_float((uint32_t)(127 - e) << 23);     // 2^-e
    if (!tile_amax && threadIdx.x == 0) vscale[blk] = __uint_as_float((uint32_t)(127 + e) << 23);
#pragma unroll
    for (int i = 0; i < U; ++i) {
        const int c = threadIdx.x + THREADS * i, lane = c & 63;
        union { uint4 v; _Float16 h[8]; } o;
        const int kk = c >> 8, db = (c >> 6) & 3, hh = lane >> 5, n = lane & 31;
#pragma unroll
        for (int el = 0; el < 8; ++el) {
            const uint32_t bits = tile[(16 * kk + 8 * (el >> 2) + 4 * hh + (el & 3)) * 128 + 32 * db + n];
            o.h[el] = (_Float16)(__uint_as_float(bits << 16) * down);
        }
        dst[c] = o.v;
    }
}
// ---- debug unpack of E4M3 tensors ---------------------------------------------------------------
// one workgroup per block of BS slots of the tile-ordered output; padding slots become zero
template <int BS>
__global__ __launch_bounds__(256) void unpack_q8_kernel(const uint8_t* __restrict__ in,
                                                        uint8_t* __restrict__ out, int role, Geom g) {
    const int blk = blockIdx.x, group = blk / g.KBS;
    const int slot0 = (blk - group * g.KBS) * BS, s = group % g.NS, u = (group / g.NS) % g.M;
    const int uw = u % g.nW, uh = (u / g.nW) % g.nH, ut = u / (g.nW * g.nH);
    const int cls = ((ut == g.nT - 1) << 2) | ((uh == g.nH - 1) << 1) | (uw == g.nW - 1);
    const RealBox box = real_box(g, cls, s);
    const uint8_t* src = in + (long long)group * g.QSP * 128;      // the sub-tile's packed blocks
    uint8_t* dst = out + (long long)blk * (BS * 128);
    for (int i = threadIdx.x; i < BS * 128; i += 256) {
        const int c = i & 127;                             // channel
        int rt, rh, rw;
        if (!sub_slot_coords(g, box.o, slot0 + (i >> 7), &rt, &rh, &rw) || !coords_in_class(g, cls, rt, rh, rw)) {
            dst[i] = 0;
            continue;
        }
        const int k = packed_slot(box, rt, rh, rw), j = k & (BS - 1);   // packed slot, within its block
        int off;
        if (role == FPS_ROLE_Q) {
            off = j * 128 + c;
        } else if (role == FPS_ROLE_K) {
            const int sb = j >> 5, n = j & 31, ks = c >> 6, h = (c >> 5) & 1, e = (c >> 4) & 1;
            off = (((sb * 2 + ks) * 2 + e) * 64 + 32 * h + n) * 16 + (c & 15);
        } else {                                           // inverse of the accumulator's key order
            const int sb = j >> 5, rem = j & 31, h = (rem >> 2) & 1, jj = 4 * (rem >> 3) + (rem & 3);
            off = ((sb * 4 + (c >> 5)) * 64 + 32 * h + (c & 31)) * 16 + jj;
        }
        dst[i] = src[(long long)(k - j) * 128 + off];
    }
}

// ---- plain copy (calibration of HBM traffic counters against a kernel of known size) ------------
__global__ void copy_kernel(const uint4* __restrict__ in, uint4* __restrict__ out, long long n_chunks) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_chunks) out[i] = in[i];
}

static inline int grid_for(long long n, int block) { return (int)((n + block - 1) / block); }

// Input and output together beyond the Infinity Cache's 256 MB: the input, not read again soon, leaves the cache to the
// output.  478 MB 92 -> 78 us, 403 MB back 80 -> 73, in fp32 806 MB 162 -> 163; of 232 MB, which the cache holds, 36.0 -> 38.6
// and 35 -> 38.5.
template <int CPR, bool TO_TILES, bool NT, int U>
static void launch_reorder_as(const Geom& g, int segments, const void* in, void* out, hipStream_t st) {
    const int waves = segments * kWavesOfSegment<CPR, U>;
    reorder_kernel<CPR, TO_TILES, NT, U><<<grid_for(waves, 4), 256, 0, st>>>((const uint4*)in, (uint4*)out, g, waves);
}

// Fewer than 4096 segments of 32 slots, 16 a CU: half as many loads a wave and more waves.  From tile order in fp32, 8 loads
// a wave against 4: 384 segments 6.6 -> 4.4 us (a chunk a thread 4.5), 1536 8.4 -> 6.0 (6.8), 2688 13.5 -> 11.4 (17.7), of tile (4,16,16)
// or (1,8,16); 5040 of tile (1,7,15) 17.2 -> 18.1 and in bf16 8.7 -> 10.0.
template <int CPR, bool TO_TILES>
static void launch_reorder(const Geom& g, const void* in, void* out, hipStream_t st) {
    const int segments = g.BH * g.M * (g.TSP / 32);
    const long long bytes = ((long long)g.BH * g.T * g.H * g.W + 32LL * segments) * CPR * 16;
    if (segments < 4096)            launch_reorder_as<CPR, TO_TILES, false, 4>(g, segments, in, out, st);
    else if (bytes > (256LL << 20)) launch_reorder_as<CPR, TO_TILES, true, 8>(g, segments, in, out, st);
    else                            launch_reorder_as<CPR, TO_TILES, false, 8>(g, segments, in, out, st);
}

int launch_tile_order(const Geom& g, const void* in, void* out, hipStream_t st) {
    launch_reorder<16, true>(g, in, out, st);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? FPS_OK : hip_fail(e, "tile_order launch");
}

int launch_tile_unorder(const Geom& g, const void* in, int elem_bytes, void* out, hipStream_t st) {
    if (elem_bytes == 2) launch_reorder<16, false>(g, in, out, st);
    else                 launch_reorder<32, false>(g, in, out, st);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? FPS_OK : hip_fail(e, "tile_unorder launch");
}

int launch_copy(const void* in, void* out, long long bytes, hipStream_t st) {
    const long long n = bytes / 16;
    copy_kernel<<<grid_for(n, 256), 256, 0, st>>>((const uint4*)in, (uint4*)out, n);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? FPS_OK : hip_fail(e, "copy launch");
}

int launch_pack_bf16(const Geom& g, const void* x, int raster, int role, void* xp, float* vscale,
                     hipStream_t st) {
    const int blocks = g.BH * g.M * g.KB, ntiles = g.BH * g.M * g.NS;   // ntiles: quantisation groups
    const float* tile_amax = nullptr;
    if (role == FPS_ROLE_V && g.KBS > 1) {                  // `vscale` holds the tile amax meanwhile
        clear_kernel<<<(ntiles + 255) / 256, 256, 0, st>>>((uint32_t*)vscale, ntiles);
        if (g.BS == 128) launch_block_amax<128>(x, raster, vscale, g, st);
        else             launch_block_amax<32>(x, raster, vscale, g, st);
        tile_amax = vscale;
    }
    const uint4* xi = (const uint4*)x;
    uint4* xo = (uint4*)xp;
    if (g.BS == 128) {
        if (raster) pack_bf16_kernel<128, true><<<blocks, 256, 0, st>>>(xi, xo, vscale, role, g, tile_amax);
        else        pack_bf16_kernel<128, false><<<blocks, 256, 0, st>>>(xi, xo, vscale, role, g, tile_amax);
    } else {
        if (raster) pack_bf16_kernel<32, true><<<blocks, 256, 0, st>>>(xi, xo, vscale, role, g, tile_amax);
        else        pack_bf16_kernel<32, false><<<blocks, 256, 0, st>>>(xi, xo, vscale, role, g, tile_amax);
    }
    if (tile_amax) amax_to_pow2_kernel<<<(ntiles + 255) / 256, 256, 0, st>>>(vscale, ntiles);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? FPS_OK : hip_fail(e, "pack_bf16 launch");
}

int launch_unpack_q8(const Geom& g, const void* xq, int role, uint8_t* out, hipStream_t st) {
    const int blocks = g.BH * g.M * g.KB;
    if (g.BS == 128) unpack_q8_kernel<128><<<blocks, 256, 0, st>>>((const uint8_t*)xq, out, role, g);
    else             unpack_q8_kernel<32><<<blocks, 256, 0, st>>>((const uint8_t*)xq, out, role, g);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? FPS_OK : hip_fail(e, "unpack_q8 launch");
}

}  // namespace fps
