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

#include <type_traits>

namespace fps {

// ---- raster -> tiled (bf16, 16-byte chunks of 8 channels) -------------------------------------
__global__ void tile_order_kernel(const uint4* __restrict__ in, uint4* __restrict__ out, Geom g,
                                  long long n_chunks) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_chunks) return;
    const int c16 = (int)(i & 15);
    const long long pos = i >> 4;                       // bh * (M*TSP) + u*TSP + r
    const int r = (int)(pos % g.TSP);
    const long long bu = pos / g.TSP;
    const int u = (int)(bu % g.M);
    const long long bh = bu / g.M;
    const int uw = u % g.nW, uh = (u / g.nW) % g.nH, ut = u / (g.nW * g.nH);
    const int s = r / g.QSP;
    int rt = 0, rh = 0, rw = 0;
    const bool slot_used = sub_slot_coords(g, sub_tile_origin(g, s), r - s * g.QSP, &rt, &rh, &rw);
    const int t = ut * g.Tt + rt, h = uh * g.Th + rh, w = uw * g.Tw + rw;
    uint4 val = make_uint4(0, 0, 0, 0);
    if (slot_used && t < g.T && h < g.H && w < g.W) {
        const long long src = (((bh * g.T + t) * g.H + h) * (long long)g.W + w) * 16 + c16;
        val = in[src];
    }
    out[i] = val;
}

// ---- tiled -> raster (elem_bytes 2 or 4; 16-byte chunks) ---------------------------------------
__global__ void tile_unorder_kernel(const uint4* __restrict__ in, uint4* __restrict__ out, Geom g,
                                    int chunks_per_row, long long n_chunks) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_chunks) return;
    const int c = (int)(i % chunks_per_row);
    long long tok = i / chunks_per_row;                 // ((bh*T + t)*H + h)*W + w
    const int w = (int)(tok % g.W); tok /= g.W;
    const int h = (int)(tok % g.H); tok /= g.H;
    const int t = (int)(tok % g.T);
    const long long bh = tok / g.T;
    const int u = ((t / g.Tt) * g.nH + h / g.Th) * g.nW + w / g.Tw;
    const int rt = t % g.Tt, rh = h % g.Th, rw = w % g.Tw;
    const int s = ((rt / g.Qt) * g.nsH + rh / g.Qh) * g.nsW + rw / g.Qw;
    const int r = s * g.QSP + ((rt % g.Qt) * g.Qh + rh % g.Qh) * g.Qw + rw % g.Qw;
    const long long src = ((bh * g.M + u) * (long long)g.TSP + r) * chunks_per_row + c;
    out[i] = in[src];
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
        if (role == FPS_ROLE_Q) copy(std::integral_constant<int, 1>{});
        else                    copy(std::integral_constant<int, 2>{});
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

int launch_tile_order(const Geom& g, const void* in, void* out, hipStream_t st) {
    const long long n = (long long)g.BH * g.M * g.TSP * 16;
    tile_order_kernel<<<grid_for(n, 256), 256, 0, st>>>((const uint4*)in, (uint4*)out, g, n);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? FPS_OK : hip_fail(e, "tile_order launch");
}

int launch_tile_unorder(const Geom& g, const void* in, int elem_bytes, void* out, hipStream_t st) {
    const int cpr = kHeadDim * elem_bytes / 16;
    const long long n = (long long)g.BH * g.T * g.H * g.W * cpr;
    tile_unorder_kernel<<<grid_for(n, 256), 256, 0, st>>>((const uint4*)in, (uint4*)out, g, cpr, n);
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
