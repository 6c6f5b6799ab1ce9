// Internal declarations shared by the translation units of libfps (not part of the ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdarg.h>
#include <type_traits>
#include "fps.h"

namespace fps {

constexpr int kHeadDim = 128;
constexpr int kMaxTileTokens = 32768;                // largest supported tile
constexpr int kMaxScoreSlots = 4096;                 // largest tile the score debug call accepts

template <int N> using Count = std::integral_constant<int, N>;   // a number as an argument's type

// n / d for any 32-bit n, given m = reciprocal(d): four scalar instructions instead of the ~35 of a division by a
// run-time value.  m = floor((2^32 - 1) / d) is at least 2^32/d - 1, so n m / 2^32 falls short of n / d by less than
// n / 2^32 < 1 and its floor by at most 1.
inline uint32_t reciprocal(int d) { return 0xFFFFFFFFu / (uint32_t)d; }
__host__ __device__ inline int quotient(int n, int d, uint32_t m) {
    const uint32_t q = (uint32_t)(((uint64_t)(uint32_t)n * m) >> 32);
    return (int)(q + ((uint32_t)n - q * (uint32_t)d >= (uint32_t)d ? 1u : 0u));
}

// Everything the kernels derive from an fps_shape.
struct Geom {
    int BH;              // B * heads
    int T, H, W;
    int Tt, Th, Tw;
    int nT, nH, nW;
    int M;
    // Quantisation sub-tile (Qt,Qh,Qw) (= the tile when none is given): a tile is NS = nsT*nsH*nsW
    // sub-tiles of QS tokens, each with its own scale; sub-tile s = (st*nsH + sh)*nsW + sw.
    int Qt, Qh, Qw;
    int nsT, nsH, nsW, NS, QS;
    // 1/(rows*columns) and 1/columns of a sub-tile as correctly rounded floats, for div_by_recip: [1] along an
    // axis that the grid's edge cuts, [0] along one it does not
    float inv_plane[2][2], inv_w[2];
    // The kernels work on blocks of BS slots (128 or 32).  A sub-tile occupies KBS = ceil(QS/BS)
    // consecutive blocks (QSP = KBS*BS slots, slot rr < QS holding the token of in-sub-tile rank
    // rr, the rest padding), a tile KB = NS*KBS blocks (TSP = KB*BS slots).  Block index =
    // tile * KB + block in tile; scale (group) index = tile * NS + sub-tile = block index / KBS.
    int BS, KBS, QSP, KB, TSP;
    // Real planes / rows / columns of the LAST tile along each axis (all others are full).  A
    // tile's boundary class is c = 4*(last along T) + 2*(last along H) + (last along W).
    int lastT, lastH, lastW;
    // The grid in sub-tiles that hold a real token: counts per axis, and for the last one along an
    // axis its real extent, its tile and its place in the tile.
    int gT, gH, gW;
    int cutT, cutH, cutW;
    // Key blocks of the attention kernels: KBG 128-slot blocks per sub-tile if BS = 128, otherwise the
    // sub-tile itself (at most 96 slots).
    int KBG;
    // Bit c of nh_classes[nh - 1]: sub-tiles cut along the axes of c (4: T, 2: H, 1: W) have a key
    // block whose real tokens fill nh 16-key halves.
    uint8_t nh_classes[8];
    uint32_t rc_kbs, rc_ns, rc_m, rc_layer, rc_row;   // reciprocals of KBS, NS, M, nH*nW, nW,
    uint32_t rc_sub_layer, rc_sub_row, rc_sub_blocks; // nsH*nsW, nsW and QSP/32
};

// n / d for 0 <= n < 2^21, given inv_d = 1.0f / d correctly rounded.  Exact: (n + 1/2) / d is at
// least 1/(2d) away from every integer, and the float product errs by less than n 2^-22 / d.
// Four cheap instructions instead of the ~25 of an integer division by a run-time value.
__host__ __device__ inline int div_by_recip(int n, float inv_d) {
    return (int)(((float)n + 0.5f) * inv_d);
}
// n / d for 0 <= n < 2^20, exact for the same reason, where no reciprocal is at hand and there are few to divide.  (With
// one made on the spot, 61 attention calls of tiles of several scale groups took 0.97 to 1.01 of the time, on average the same.)
__host__ __device__ inline int divide_small(int n, int d) { return (int)(((float)n + 0.5f) / (float)d); }

__host__ __device__ inline int min_of(int a, int b) { return a < b ? a : b; }

// In-tile coordinates of the first token of sub-tile s (decoded once per block: s is the same
// for all slots of a block).
struct SubTile { int t0, h0, w0; };
__host__ __device__ inline SubTile sub_tile_origin(const Geom& g, int s) {
    const int layer = g.nsH * g.nsW;
    const int st = quotient(s, layer, g.rc_sub_layer), srem = s - st * layer;
    const int sh = quotient(srem, g.nsW, g.rc_sub_row), sw = srem - sh * g.nsW;
    return SubTile{st * g.Qt, sh * g.Qh, sw * g.Qw};
}

// In-tile coordinates (rt, rh, rw) of slot rr of the sub-tile with origin o; false if the slot is
// padding of the sub-tile (rr >= QS).
__host__ __device__ inline bool sub_slot_coords(const Geom& g, const SubTile& o, int rr, int* rt, int* rh, int* rw) {
    if (rr >= g.QS) return false;
    const int a = div_by_recip(rr, g.inv_plane[0][0]), rem = rr - a * (g.Qh * g.Qw);
    const int b = div_by_recip(rem, g.inv_w[0]), c = rem - b * g.Qw;
    *rt = o.t0 + a; *rh = o.h0 + b; *rw = o.w0 + c;
    return true;
}

// in-tile coordinates (rt, rh, rw) lie inside the real extent of a tile of boundary class c
__host__ __device__ inline bool coords_in_class(const Geom& g, int c, int rt, int rh, int rw) {
    return rt < ((c & 4) ? g.lastT : g.Tt) && rh < ((c & 2) ? g.lastH : g.Th) &&
           rw < ((c & 1) ? g.lastW : g.Tw);
}

// slot rr of the sub-tile with origin o, in a tile of boundary class c, holds a real token
__host__ __device__ inline bool sub_slot_is_token(const Geom& g, int c, const SubTile& o, int rr) {
    int rt, rh, rw;
    return sub_slot_coords(g, o, rr, &rt, &rh, &rw) && coords_in_class(g, c, rt, rh, rw);
}

// Packed operands hold the REAL tokens of a sub-tile first, in raster order of the sub-tile's real
// box (the sub-tile cut at the grid's edge), then padding: packed slot k < n of a sub-tile of real
// extent (et, eh, ew), n = et*eh*ew, is its token (k / (eh*ew), k / ew % eh, k % ew).  The padding
// of a cut tile is thus one run at the end, whole matrix-instruction blocks of which are never
// computed, instead of being spread over every block (a tile cut along W has padding in every row).
// Tiled tensors keep the order of fps.h; for a sub-tile that is not cut the two orders agree.
struct RealBox {
    SubTile o;               // in-tile origin of the sub-tile
    int eh, ew, plane, n;    // real rows and columns, eh*ew, real tokens (0 if none)
    float inv_plane, inv_w;  // for div_by_recip
};
__host__ __device__ inline int real_tokens(const Geom& g, int c, const SubTile& o) {
    const int et = ((c & 4) ? g.lastT : g.Tt) - o.t0, eh = ((c & 2) ? g.lastH : g.Th) - o.h0,
              ew = ((c & 1) ? g.lastW : g.Tw) - o.w0;
    if (et <= 0 || eh <= 0 || ew <= 0) return 0;
    return (et < g.Qt ? et : g.Qt) * (eh < g.Qh ? eh : g.Qh) * (ew < g.Qw ? ew : g.Qw);
}
__host__ __device__ inline RealBox real_box(const Geom& g, int c, int s) {
    RealBox b;
    b.o = sub_tile_origin(g, s);
    const int eh = ((c & 2) ? g.lastH : g.Th) - b.o.h0, ew = ((c & 1) ? g.lastW : g.Tw) - b.o.w0;
    b.n = real_tokens(g, c, b.o);
    b.eh = b.n ? (eh < g.Qh ? eh : g.Qh) : 1;
    b.ew = b.n ? (ew < g.Qw ? ew : g.Qw) : 1;
    b.plane = b.eh * b.ew;
    const bool ch = b.eh < g.Qh, cw = b.ew < g.Qw;        // then they are cutH, cutW
    b.inv_plane = ch ? (cw ? g.inv_plane[1][1] : g.inv_plane[1][0]) : (cw ? g.inv_plane[0][1] : g.inv_plane[0][0]);
    b.inv_w = cw ? g.inv_w[1] : g.inv_w[0];
    return b;
}
// offset of real token k of the box from the sub-tile's origin
struct Offset { int t, h, w; };
__host__ __device__ inline Offset real_token(const RealBox& b, int k) {
    const int t = div_by_recip(k, b.inv_plane), rem = k - t * b.plane;
    const int h = div_by_recip(rem, b.inv_w);
    return Offset{t, h, rem - h * b.ew};
}
// packed slot within the sub-tile of in-tile coordinates inside its box (inverse of real_token)
__host__ __device__ inline int packed_slot(const RealBox& b, int rt, int rh, int rw) {
    return (rt - b.o.t0) * b.plane + (rh - b.o.h0) * b.ew + (rw - b.o.w0);
}

// Brings the first LINES 64-byte lines of the kernel's arguments into the scalar cache, at once.  Read where they are
// first used they miss one after the other, each miss a trip to where the host wrote them.  Attention launches gain: 4032
// workgroups 314 -> 310 us, 400 32.9 -> 32.0, 64 16.9 -> 16.6.  The quantisation kernels have few arguments and do not.
template <int LINES>
__device__ __forceinline__ void load_arguments() {
    static_assert(LINES >= 2 && LINES <= 9, "as many loads as are written here");
    const auto* p = (const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr();
    uint32_t x;
    asm volatile("s_load_dword %0, %1, 0x0\n\t"
                 "s_load_dword %0, %1, 0x40\n\t"
                 "s_load_dword %0, %1, %2\n\t"
                 "s_load_dword %0, %1, %3\n\t"
                 "s_load_dword %0, %1, %4\n\t"
                 "s_load_dword %0, %1, %5\n\t"
                 "s_load_dword %0, %1, %6\n\t"
                 "s_load_dword %0, %1, %7\n\t"
                 "s_load_dword %0, %1, %8\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&s"(x)
                 : "s"(p), "n"(64 * (LINES > 2 ? 2 : 0)), "n"(64 * (LINES > 3 ? 3 : 0)), "n"(64 * (LINES > 4 ? 4 : 0)),
                   "n"(64 * (LINES > 5 ? 5 : 0)), "n"(64 * (LINES > 6 ? 6 : 0)), "n"(64 * (LINES > 7 ? 7 : 0)),
                   "n"(64 * (LINES > 8 ? 8 : 0)));
    asm volatile("" ::"s"(x));
}

void set_error(const char* fmt, ...);
int check_shape(const fps_shape* s, Geom* g);          // validates, fills g
int check_ptr(const void* p, const char* name);        // non-null and 16-byte aligned
int hip_fail(hipError_t e, const char* what);          // records and returns FPS_ERR_HIP

// kernel launchers (defined in the .hip files); all arguments already validated
int launch_tile_order(const Geom& g, const void* in, void* out, hipStream_t st);
int launch_tile_unorder(const Geom& g, const void* in, int elem_bytes, void* out, hipStream_t st);
int launch_quantize(const Geom& g, const void* x, int raster, int role, int vscale, void* xq,
                    float* scales, hipStream_t st);
int launch_pack_bf16(const Geom& g, const void* x, int raster, int role, void* xp, float* vscale,
                     hipStream_t st);
int launch_unpack_q8(const Geom& g, const void* xq, int role, uint8_t* out, hipStream_t st);
int launch_attn(const Geom& g, const fps_window& win, int prec, const void* q, const void* k,
                const void* v, const float* sq, const float* sk, const float* sv, int vscale,
                void* out, int out_f32, int out_raster, uint8_t* visited, hipStream_t st);

int launch_copy(const void* in, void* out, long long bytes, hipStream_t st);
int launch_mfma_rate(int workgroups, int iters, float* sink, hipStream_t st);
int launch_issue_mix(int kind, int nv, int op, int workgroups_per_cu, int workgroups, int iters,
                     float* sink, unsigned long long* cycles, hipStream_t st);
int launch_scores_fp8(const Geom& g, const void* q, const void* k, int bh, int u, int v, float* out,
                      hipStream_t st);
int launch_scores_block_fp8(const Geom& g, const void* q, const void* k, int bh, int u, int jq, int v,
                            int jk, float* out, hipStream_t st);

}  // namespace fps
