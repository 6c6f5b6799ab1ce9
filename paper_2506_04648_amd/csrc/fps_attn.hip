// Host side of the attention launch, and the debug kernels that use its operand layouts.
#include "fps_attn_device.h"

namespace fps {

// Debug: raw E4M3 score accumulators sum_c q_ic * k_jc of pairs of slot blocks, produced by the same
// MFMA instruction as the attention kernel; out[query slot][key slot] in the tile's slot order, zero for
// padding slots.  The rows are gathered one by one, since packed operands hold a tile's real tokens
// in another order (real_box).
// Byte offset of 16-byte chunk c16 (channels 16 c16 ..) of slot `slot` of tile class cls inside the
// tile's packed Q (K: is_k) tensor; -1 for a padding slot.
__device__ __forceinline__ int packed_row_chunk(const Geom& G, int cls, int slot, int c16, bool is_k) {
    const int sub = slot / G.QSP;
    const RealBox box = real_box(G, cls, sub);
    int rt, rh, rw;
    if (!sub_slot_coords(G, box.o, slot - sub * G.QSP, &rt, &rh, &rw) || !coords_in_class(G, cls, rt, rh, rw)) return -1;
    const int k = sub * G.QSP + packed_slot(box, rt, rh, rw);
    if (!is_k) return k * 128 + c16 * 16;
    const int ks = c16 >> 2, h = (c16 >> 1) & 1, e = c16 & 1;
    return (k & ~31) * 128 + ((ks * 2 + e) * 64 + 32 * h + (k & 31)) * 16;
}
__device__ __forceinline__ v8i gather_operand(const uint8_t* base, int off_lo, int off_hi) {
    const uint4 z = make_uint4(0, 0, 0, 0);
    return make_v8i(off_lo < 0 ? z : *reinterpret_cast<const uint4*>(base + off_lo),
                    off_hi < 0 ? z : *reinterpret_cast<const uint4*>(base + off_hi));
}

// one wave per 32 x 32 slots: workgroup (x, y) = (32-slot key group, 32-slot query group) of the pair
__global__ __launch_bounds__(64) void scores_fp8_kernel(const uint8_t* __restrict__ q_tile, int q_cls, int q_slot0,
                                                        const uint8_t* __restrict__ k_tile, int k_cls, int k_slot0,
                                                        float* __restrict__ out, int out_pitch, Geom G) {
    const int lane = threadIdx.x, h = lane >> 5, n = lane & 31;
    const int qs = q_slot0 + 32 * blockIdx.y, ks0 = k_slot0 + 32 * blockIdx.x;
    float* o = out + (size_t)(32 * blockIdx.y) * out_pitch + 32 * blockIdx.x;
    v16f s = zero16();
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        const int c16 = 4 * ks + 2 * h;                    // channels 64ks + 32h ..
        const v8i qop = gather_operand(q_tile, packed_row_chunk(G, q_cls, qs + n, c16, false),
                                       packed_row_chunk(G, q_cls, qs + n, c16 + 1, false));
        const v8i kop = gather_operand(k_tile, packed_row_chunk(G, k_cls, ks0 + n, c16, true),
                                       packed_row_chunk(G, k_cls, ks0 + n, c16 + 1, true));
        s = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(kop, qop, s, 0, 0, 0, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) o[(size_t)n * out_pitch + 8 * (r >> 2) + 4 * h + (r & 3)] = s[r];
}

// MFMA-only loop: 8 independent accumulator chains of 16x16x128 (the attention kernel's 32x32x64 has the same rate).
__global__ __launch_bounds__(256) void mfma_rate_kernel(float* __restrict__ sink, int iters, int x) {
    v8i a = {x, x, x, x, x, x, x, x};
    v8i b = a;
    v4f c[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) c[i] = v4f{0.f, 0.f, 0.f, 0.f};
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
            c[i] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(a, b, c[i], 0, 0, 0, 0, 0, 0);
    }
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) s += c[i][0] + c[i][1] + c[i][2] + c[i][3];
    sink[blockIdx.x * 256 + threadIdx.x] = s;
}

int launch_mfma_rate(int workgroups, int iters, float* sink, hipStream_t st) {
    mfma_rate_kernel<<<workgroups, 256, 0, st>>>(sink, iters, 0x38383838);   // E4M3 code of 1.0 in every byte
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? FPS_OK : hip_fail(e, "mfma rate launch");
}

// slots slot_q .. of tile u against slots slot_k .. of tile v, `slots` of each
static int launch_scores(const Geom& g, const void* q, const void* k, int bh, int u, int slot_q, int v, int slot_k,
                         int slots, float* out, hipStream_t st) {
    const size_t tile_bytes = (size_t)g.TSP * 128;
    const uint8_t* qp = (const uint8_t*)q + ((size_t)bh * g.M + u) * tile_bytes;
    const uint8_t* kp = (const uint8_t*)k + ((size_t)bh * g.M + v) * tile_bytes;
    auto cls = [&g](int t) {
        return ((t / (g.nW * g.nH) == g.nT - 1) << 2) | (((t / g.nW) % g.nH == g.nH - 1) << 1) | (t % g.nW == g.nW - 1);
    };
    const dim3 grid(slots / 32, slots / 32);
    scores_fp8_kernel<<<grid, 64, 0, st>>>(qp, cls(u), slot_q, kp, cls(v), slot_k, out, slots, g);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? FPS_OK : hip_fail(e, "debug scores launch");
}

int launch_scores_fp8(const Geom& g, const void* q, const void* k, int bh, int u, int v, float* out,
                      hipStream_t st) {
    return launch_scores(g, q, k, bh, u, 0, v, 0, g.TSP, out, st);
}

int launch_scores_block_fp8(const Geom& g, const void* q, const void* k, int bh, int u, int jq, int v,
                            int jk, float* out, hipStream_t st) {
    return launch_scores(g, q, k, bh, u, jq * g.BS, v, jk * g.BS, g.BS, out, st);
}

int launch_attn(const Geom& g, const fps_window& win, int prec, const void* q, const void* k,
                const void* v, const float* sq, const float* sk, const float* sv, int vscale,
                void* out, int out_f32, int out_raster, uint8_t* visited, hipStream_t st) {
    AttnArgs a;
    a.q = (const uint8_t*)q; a.k = (const uint8_t*)k; a.v = (const uint8_t*)v;
    a.sq = sq; a.sk = sk; a.sv = sv;
    a.out = out; a.visited = visited;
    a.g = g;
    a.rt = win.wt / 2; a.rh = win.wh / 2; a.rw = win.ww / 2;
    a.edge_shift = win.edge == FPS_EDGE_SHIFT;
    a.out_f32 = out_f32;
    a.out_raster = out_raster;
    const int grid = 8 * plan_launch(a, prec == FPS_PREC_FP8);
    if (prec == FPS_PREC_FP8) launch_attn_fp8(a, vscale == FPS_VSCALE_CHANNEL, grid, st);
    else                      launch_attn_bf16(a, grid, st);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? FPS_OK : hip_fail(e, "attention launch");
}

}  // namespace fps
