// Sliding-tile attention forward (Eq. 2-3, Sec. 3.2 aggregation; Algorithm 1 steps 4-5): what the FP8
// and the BF16 kernel share.
//
// A work item is one query block of a tile: W sub-blocks of 32 packed slots, one wave each.  The kernel
// walks the box of key tiles given by Eq. 2 -- tile pairs outside the box are never scheduled -- in key
// blocks of at most SB sub-blocks of 32 keys, staged through LDS.  A key block lies in one scale
// group (a tile, or a quantisation sub-tile):
//   SB = 4, W = 4        groups of more than 96 tokens; a group is one or several 128-slot blocks.  W = 2 or 1
//                        in launches of few items (narrow_waves)
//   SB = 1, 2, 3         groups of at most 32, 64, 96 tokens, one block each.  W = SB where the tile is
//                        one group, so that a workgroup is one tile and walks its window exactly; a tile
//                        of several groups gives its workgroups four of its sub-blocks, or SB where it
//                        has no multiple of four.  (On 16x16 instructions, one wave and 32 keys at a
//                        time, the whole path took 1552 instead of 957 us for tile (3,4,4), window 3x5x7 on
//                        21x30x52 x 12 heads, and 3949 instead of 2664 us for 64-token sub-tiles of (2,8,16)
//                        tiles, window 3x3x3, x 24 heads.)
// MB = true: a tile is several key blocks.
// KS = 2 or 4 (launches that would leave the chip half empty): KS times W waves; wave group kg takes the
// blocks kg, kg + KS, .. of every walk, with buffers of its own; at the end each group adds up, and stores, a share of
// the channels (SplitMerge).
//
// Scores are produced transposed, S^T = K Q^T, on the 32x32 matrix instructions, so that a lane's
// accumulator holds one query row and a fixed set of keys: lane (n, h) = lane & 31, lane >> 5 holds
// query n; of a 32-key sub-block the keys 8(r/4) + 4h + r%4, r = 0..15; of a 32-channel output block
// the channels of the same pattern.  The other lane of the row is lane n + 32.  After the softmax
// those registers are, unchanged, the second operand of the PV product O^T = V^T P^T (see the packed
// layouts in fps_layout.hip).
//
// Softmax is online in base 2 with an integer row reference m (ceil of the running row maximum):
// P = 2^(S' - m) <= 1, rescaling by 2^(m_old - m_new) is exact, and the E4M3 rounding of 448*P
// does not depend on the order in which key tiles arrive (apart from values in the subnormal
// range of the format).  The denominator accumulates the unrounded P.
#pragma once
#include "fps_attn_plan.h"

#include <stddef.h>

namespace fps {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));

typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

struct AttnArgs {
    const uint8_t* q;
    const uint8_t* k;
    const uint8_t* v;
    const float* sq;
    const float* sk;
    const float* sv;
    void* out;
    uint8_t* visited;
    Geom g;
    int rt, rh, rw;        // window radii in tiles
    int edge_shift;        // 1: clamp the window centre into the grid instead of truncating
    int out_f32;
    int out_raster;        // output in raster order (real tokens only) instead of tile order
    int waves;             // sub-blocks of 32 rows of a work item
    int qblocks;           // query blocks (work items) of a tile
    uint32_t rc_qblocks;
    int chunk;             // work items per XCD, a multiple of 4
    int rotate;            // deal each four consecutive work items in a turning order (see work_item)
    int total;             // BH * M * qblocks
    int tail;              // the items of an XCD are dealt in raster order up to this slot, the rest by `plan` (plan_tail);
                           // -1: all by `plan` (plan_items)
    ItemPlan plan;
};

// Every lambda of the kernels captures the accumulators by reference; left to the inliner's cost
// model a large one stays a call, which forces everything it captures into private memory.
#define FPS_INLINE __attribute__((always_inline))

constexpr float kLog2eOverSqrtD = 0.12751743f;   // log2(e) / sqrt(128)
constexpr float kLog2Of448 = 8.8073549f;          // log2(448)
constexpr float kFp16PScaleLog2 = 14.0f;          // BF16 mode holds 2^14 * P in fp16
constexpr float kMaxDrift = 64.0f;                // largest m - m_base before O and l are moved to a new reference

// Scales are read-only for the whole launch and indexed uniformly: reading them through the constant
// address space lets the compiler use scalar loads, which do not queue behind the vector-memory
// traffic that stages the K/V tiles.
typedef const __attribute__((address_space(4))) float* const_f32_ptr;
__device__ __forceinline__ float load_uniform(const float* p, size_t i) {
    return ((const_f32_ptr)(uintptr_t)p)[i];
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// two floats -> two bf16 (round to nearest even) in one dword; gfx950 converts in hardware
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v2f{lo, hi}, v2bf));
}

// Work item of this workgroup: query block jq of tile (ut, uh, uw) of head bh.  Workgroups are dealt round-robin to
// the 8 XCDs by the hardware; giving XCD x the contiguous range [x*chunk, (x+1)*chunk) of items (or that part of every
// section) keeps the key tiles of neighbouring query tiles of one head in that XCD's L2.  (It is the same part of every
// section: with the sections' odd items on other XCDs in turn, for an even load, an XCD met other heads' keys in every
// section, and of 10 000 random calls one in 12 was slower by 3 % or more, up to twice.)
//
// Within an XCD the hardware deals workgroups in order and round-robin to four shader engines, waiting
// for the one whose turn it is.  How long an item takes depends on its place in the row of tiles (cut
// tiles and the grid's edges are short), so with a row of 4, 8, .. items one engine gets all the short ones and
// stands idle: 21x30x52 tokens x 12 heads, tile (1,8,16), four tiles a row, had 355 of 512 workgroups
// resident.  There (deal_in_turns) each group of four items is dealt in an order that turns from group to group; with
// the group's index over 4 and 16 added, so that it also turns from row to row where a row is 8, 16 or 32 items.
// So too where the items are dealt by `plan`: idle and short items then still recur with the row (7x12x11 tokens x 36 heads,
// tile (4,8,8), window 1x3x2, 21.1 us in raster order, planned 30.6, in turns 21.5; 6x16x27 x 20 57.1, 71.4, 56.6).
__device__ __forceinline__ bool work_item(const AttnArgs& a, int* bh, int* ut, int* uh, int* uw, int* jq) {
    const Geom& G = a.g;
    const int xcd = blockIdx.x & 7;
    int slot = blockIdx.x >> 3;
    if (a.rotate) {
        const int group = slot >> 2;
        slot = 4 * group + ((slot + group + (group >> 2) + (group >> 4)) & 3);
    }
    // the plan is indexed by values known on the device only: read where it lies, in the kernel's argument segment
    // (AttnArgs is the kernels' only argument), since the compiler may copy an indexed argument to scratch memory
    typedef const __attribute__((address_space(4))) char* args_ptr;
    const auto& p = *(const __attribute__((address_space(4))) ItemPlan*)((args_ptr)__builtin_amdgcn_kernarg_segment_ptr() +
                                                                        offsetof(AttnArgs, plan));
    static_assert(kSectionLanes == 32, "half a wave");
    auto section = [&]() FPS_INLINE {
        return __popc((uint32_t)__ballot((int)(p.section[1 + (threadIdx.x & 31)] & kSectionStart) <= slot));
    };
    if (a.tail >= 0) {
        int wi = xcd * a.chunk + slot;
        if (slot >= a.tail) wi = tail_item(p, G, a.qblocks, a.rc_qblocks, xcd * a.chunk + a.tail, slot, section());
        if (wi >= a.total) return false;
        const int tile_lin = quotient(wi, a.qblocks, a.rc_qblocks);
        *jq = wi - tile_lin * a.qblocks;
        *bh = quotient(tile_lin, G.M, G.rc_m);
        const int u = tile_lin - *bh * G.M;
        *ut = quotient(u, G.nW * G.nH, G.rc_layer);
        const int rem = u - *ut * (G.nW * G.nH);
        *uh = quotient(rem, G.nW, G.rc_row);
        *uw = rem - *uh * G.nW;
        return true;
    }
    return planned_item(p, G, a.qblocks, a.rc_qblocks, xcd, slot, section(), bh, ut, uh, uw, jq);
}

template <typename G_>
__device__ __forceinline__ int tile_class(const G_& g, int t, int h, int w) {
    return ((t == g.nT - 1) << 2) | ((h == g.nH - 1) << 1) | (w == g.nW - 1);
}

__device__ __forceinline__ v16f zero16() {
    v16f z;
#pragma unroll
    for (int r = 0; r < 16; ++r) z[r] = 0.f;
    return z;
}
// Reductions over the two lanes n, n + 32 that hold one query row: gfx950 swaps halves of 32 lanes
// between two registers at VALU speed.
__device__ __forceinline__ float max_over_row_pair(float t) {          // lanes n and n + 32
    const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false);
    return __builtin_fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_over_row_pair(float t) {
    const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(t), __float_as_uint(t), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// x if bit `idx` of the lane's word `bits` is set, otherwise -inf: two vector instructions (a
// sign-extended one-bit field, a bitwise select) and no compare, so a run of them needs no scalar
// registers for compare results
__device__ __forceinline__ float keep_if_bit(float x, uint32_t bits, int idx) {
    const uint32_t m = (uint32_t)(-(int)((bits >> idx) & 1u));
    return __uint_as_float((__float_as_uint(x) & m) | (0xFF800000u & ~m));
}
// A key block whose last 16-key half is cut: of registers 8e .. 8e+7 of s, which hold the half, those of
// its keys from n on become -inf.
__device__ __forceinline__ void mask_cut_half(v16f& s, int e, int n, int h) {
    const uint32_t bits = ((1u << n) - 1u) >> (4 * h);
#pragma unroll
    for (int r = 0; r < 8; ++r) s[8 * e + r] = keep_if_bit(s[8 * e + r], bits, 8 * (r >> 2) + (r & 3));
}

// The 32 query rows of a wave: packed slots k0 .. k0 + 31 of one scale group, of which the first `rows`
// (at most 32; none if <= 0) are real tokens.
struct QueryRows {
    RealBox box;
    int k0, rows;
    int group;               // the scale group within the tile
    int slot_base;           // first tiled slot of the group within its tile
    size_t tile_lin;         // bh * M + u
    size_t raster0;          // raster token index of the group's first token
    // sub-block qs of the tile; sbg: sub-blocks per group, QSP / 32.  GROUPS: a tile may have several
    template <bool GROUPS>
    __device__ __forceinline__ void init(const Geom& G, int bh, int u, int cls, int ut, int uh, int uw, int qs, int sbg) {
        group = GROUPS ? quotient(qs, sbg, G.rc_sub_blocks) : 0;
        box = real_box(G, cls, group);
        k0 = 32 * (qs - group * sbg);
        rows = box.n - k0;
        slot_base = group * G.QSP;
        tile_lin = (size_t)bh * G.M + u;
        raster0 = (((size_t)bh * G.T + (ut * G.Tt + box.o.t0)) * G.H + (uh * G.Th + box.o.h0)) * G.W +
                  (uw * G.Tw + box.o.w0);
    }
    // output row of the group's first token, and that of row r (0 <= r < rows) from there: within a head, 32 bits do
    __device__ __forceinline__ size_t out_base(const AttnArgs& a) const {
        return a.out_raster ? raster0 : tile_lin * a.g.TSP + slot_base;
    }
    __device__ __forceinline__ int out_offset(const AttnArgs& a, int r) const {
        const Offset d = real_token(box, k0 + r);
        const int rows_of = a.out_raster ? a.g.H : a.g.Qh, columns = a.out_raster ? a.g.W : a.g.Qw;
        return (d.t * rows_of + d.h) * columns + d.w;
    }
};

// A tile-ordered output has rows for padding slots, and they are zero: each wave clears those among its
// 32 slots.
__device__ __forceinline__ void zero_padding_rows(const AttnArgs& a, const QueryRows& q, int cls, int lane) {
    if (a.out_raster || q.box.n == a.g.QSP) return;
    const int row_shift = a.out_f32 ? 5 : 4;                // log2 of the 16-byte chunks of a row
    uint4* dst = reinterpret_cast<uint4*>(a.out) + ((q.tile_lin * a.g.TSP + q.slot_base + q.k0) << row_shift);
    for (int i = lane; i < (32 << row_shift); i += 64)
        if (!sub_slot_is_token(a.g, cls, q.box.o, q.k0 + (i >> row_shift))) dst[i] = make_uint4(0, 0, 0, 0);
}

// Which sub-blocks of a tile of class `cls` hold real tokens: of its scale groups et x eh x ew do, the last ones along an axis
// with ct, ch, cw tokens.  sbg: sub-blocks per group.
struct RealSubBlocks {
    const Geom& g;
    int sbg, et, eh, ew, ct, ch, cw;
    __host__ __device__ RealSubBlocks(const Geom& g_, int cls, int sbg_) : g(g_), sbg(sbg_) {
        const int lt = cls & 4 ? g.lastT : g.Tt, lh = cls & 2 ? g.lastH : g.Th, lw = cls & 1 ? g.lastW : g.Tw;
        et = divide_small(lt + g.Qt - 1, g.Qt); eh = divide_small(lh + g.Qh - 1, g.Qh); ew = divide_small(lw + g.Qw - 1, g.Qw);
        ct = lt - (et - 1) * g.Qt; ch = lh - (eh - 1) * g.Qh; cw = lw - (ew - 1) * g.Qw;
    }
    // sub-blocks of a row of groups of `th` tokens a column, of a layer of groups of t planes
    __host__ __device__ int row(int th) const { return (ew - 1) * ((th * g.Qw + 31) >> 5) + ((th * cw + 31) >> 5); }
    __host__ __device__ int layer(int t) const { return (eh - 1) * row(t * g.Qh) + row(t * ch); }
    __host__ __device__ int total() const { return (et - 1) * layer(g.Qt) + layer(ct); }
    // the i-th of them, i < total()
    __host__ __device__ int sub_block(int i) const {
        const int full_layer = layer(g.Qt), st = et > 1 ? min_of(divide_small(i, full_layer), et - 1) : 0;
        i -= st * full_layer;
        const int t = st < et - 1 ? g.Qt : ct, full_row = row(t * g.Qh);
        const int sh = eh > 1 ? min_of(divide_small(i, full_row), eh - 1) : 0;
        i -= sh * full_row;
        const int th = t * (sh < eh - 1 ? g.Qh : ch), full = (th * g.Qw + 31) >> 5;
        const int sw = ew > 1 ? min_of(divide_small(i, full), ew - 1) : 0;
        return ((st * g.nsH + sh) * g.nsW + sw) * sbg + i - sw * full;
    }
};

// The sub-block of query rows that a wave takes, the `of_item`-th of work item jq; -1: the tile has no more, -2: for no wave of
// the item.  The items of a tile of several scale groups take its real sub-blocks one after the other where that saves an item:
// in the order of all sub-blocks, tiles whose groups are cut or missing had items of few waves with rows, each of them a walk
// (attention on 21x30x52 tokens x 24 heads, 64-token sub-tiles of (2,8,16) tiles, window 3x3x3, 1715 -> 1630 us, BF16 1870 ->
// 1817; x 8 heads, 15 planes, 128-token sub-tiles 252 -> 246; 96-token ones of (2,12,16) tiles x 12 815 -> 767).  Elsewhere it
// only costs the divisions (tiles that are one item, 16-token sub-tiles of (2,4,8) and 64-token ones of (2,8,8) tiles, 17
// calls, 0.5 %, up to 1.4; tiles of one group 281 -> 282), and as many sub-blocks as an item has are needed for an item without
// rows.
// uniform(x): x, the same in all lanes, as a scalar.
template <int SB, int W, typename F>
__host__ __device__ inline int item_sub_block(const Geom& G, int cls, int jq, int of_item, int sbg, F&& uniform) {
    const int i = jq * W + of_item;
    if (G.NS == 1) return i;                               // the rows of the one group lie together
    if (W == 1) return i;                                  // an item is a sub-block (36 of them 10.4 us, with the divisions 10.6)
    if (2 * SB <= W && G.NS * sbg <= W) return i;          // the tile is one item
    const bool cut = ((cls & 4) && G.lastT < G.Tt) || ((cls & 2) && G.lastH < G.Th) || ((cls & 1) && G.lastW < G.Tw);
    if (!cut && ((G.QS + 31) >> 5) == sbg) return i;       // all of them are real
    const RealSubBlocks real(G, cls, sbg);
    const int total = uniform(real.total());
    if (total > G.NS * sbg - W) return i;
    if (i >= total) return jq * W >= total ? -2 : -1;
    return uniform(real.sub_block(i));
}
template <int SB, int W, bool MB>
__device__ __forceinline__ int wave_sub_block(const Geom& G, int cls, int jq, int of_item, int sbg) {
    if (!MB) return jq * W + of_item;
    return item_sub_block<SB, W>(G, cls, jq, of_item, sbg, [](int x) FPS_INLINE { return __builtin_amdgcn_readfirstlane(x); });
}

// Epilogue: O = acc * inv (times the per-channel V scale if any), fp32 or bf16, tile or raster order; the ND blocks of 32
// channels from channel c0 on.  A lane holds 4 channels of one row per accumulator quarter, so direct stores would be 8- or
// 16-byte pieces of many rows; instead each wave transposes its rows through a private LDS region -- all 32 rows at
// once in bf16, 16 a pass in fp32 (rows n < 16 are held by lanes 0..15 and 32..47) -- and writes whole rows
// (of all channels 256 or 512 contiguous bytes).  The reads and stores of a pass are unrolled, so that one LDS round trip and
// one address calculation do not wait for the other: 720p attention 3.84 -> 3.81 ms, dense BF16 12x37x70 x 16 heads
// 8.27 -> 8.25 ms, one-wave workgroups of 32 tokens 12.4 -> 11.8 us.  Where a row goes is worked out by the lanes that hold it
// and fetched from them: worked out by every store for its rows, with two divisions and two branches each, it was half of
// the epilogue's 800 instructions (480p 299.6 -> 299, 225 items of two groups 30.7 -> 30.6 us).  The caller guarantees that no
// wave still reads the LDS buffers.
constexpr int store_region_bytes(int nd) { return 32 * (nd * 64 + 16); }   // a wave's; 16 rows of fp32: less
template <bool F32, int ND>
__device__ __forceinline__ void store_rows_as(const AttnArgs& a, const QueryRows& q, int lane, const v16f (&acc)[ND],
                                              float inv, uint8_t* wave_lds, const float* ch_scale, int c0) {
    constexpr int kElem = F32 ? 4 : 2, kRowBytes = ND * 32 * kElem, kRows = F32 ? 16 : 32;   // rows a pass
    constexpr int kPitch = kRowBytes + 16;                 // padding keeps the column writes off one bank
    constexpr int kLanes = kRowBytes / 16, kRowsPerStore = 64 / kLanes;
    static_assert(kRows * kPitch <= store_region_bytes(ND), "the wave's region holds a pass");
    const int h = lane >> 5, n = lane & 31, chunk = lane % kLanes;
    uint8_t* const out = reinterpret_cast<uint8_t*>(a.out) + q.out_base(a) * (128 * kElem) + c0 * kElem;
    const int offset = n < q.rows ? q.out_offset(a, n) : -1;       // of row n; the rows of a store ask for theirs
#pragma unroll
    for (int pass = 0; pass < 32 / kRows; ++pass) {
        if (!F32 || (n >> 4) == pass) {
            uint8_t* const row = wave_lds + (n & (kRows - 1)) * kPitch;
#pragma unroll
            for (int db = 0; db < ND; ++db)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    const int col = 32 * db + 8 * q4 + 4 * h;
                    v4f o = v4f{acc[db][4 * q4], acc[db][4 * q4 + 1], acc[db][4 * q4 + 2], acc[db][4 * q4 + 3]} * inv;
                    if (ch_scale) o *= *reinterpret_cast<const v4f*>(ch_scale + c0 + col);
                    if (F32) {
                        *reinterpret_cast<v4f*>(row + col * 4) = o;
                    } else {
                        uint2 pk;
                        pk.x = pack_bf16x2(o[0], o[1]);
                        pk.y = pack_bf16x2(o[2], o[3]);
                        *reinterpret_cast<uint2*>(row + col * 2) = pk;
                    }
                }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // not uint4: the compiler left an array of those in scratch memory in one kernel
        u32x4 val[kRows / kRowsPerStore];
        int at[kRows / kRowsPerStore];
#pragma unroll
        for (int i = 0; i < kRows / kRowsPerStore; ++i) {
            const int row = i * kRowsPerStore + lane / kLanes;
            at[i] = __builtin_amdgcn_ds_bpermute(4 * (pass * kRows + row), offset);
            val[i] = *reinterpret_cast<const u32x4*>(wave_lds + row * kPitch + chunk * 16);
        }
#pragma unroll
        for (int i = 0; i < kRows / kRowsPerStore; ++i)
            if (at[i] >= 0) reinterpret_cast<u32x4*>(out + (size_t)(uint32_t)at[i] * (128 * kElem))[chunk] = val[i];
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}
template <int ND>
__device__ __forceinline__ void store_rows(const AttnArgs& a, const QueryRows& q, int lane, const v16f (&acc)[ND],
                                           float inv, uint8_t* wave_lds, const float* ch_scale = nullptr, int c0 = 0) {
    if (a.out_f32) store_rows_as<true>(a, q, lane, acc, inv, wave_lds, ch_scale, c0);
    else           store_rows_as<false>(a, q, lane, acc, inv, wave_lds, ch_scale, c0);
}

__device__ __forceinline__ v8i make_v8i(const uint4& lo, const uint4& hi) {
    return v8i{(int)lo.x, (int)lo.y, (int)lo.z, (int)lo.w, (int)hi.x, (int)hi.y, (int)hi.z, (int)hi.w};
}

// Linear HBM -> LDS copies of the 16-byte chunks FIRST .. FIRST + N - 1 (at most 4) of each lane, done by the load unit itself:
// lane i of the wave deposits chunk c at lds_wave_base + 1024 c + 16 i.  Written as inline assembly so that the compiler's
// wait-count bookkeeping does not serialise them against LDS reads of OTHER buffers; the kernel waits for them explicitly
// (s_waitcnt vmcnt(0)) before the barrier that publishes the tile.  gsrc is a wave-uniform base (kept in scalar registers),
// lane_off the lane's byte offset from it.  The instruction's immediate offset is added by the hardware to the global address
// AND to the LDS address, so the pieces of a 4 KB share need one scalar base each side.
template <int FIRST, int N>
__device__ __forceinline__ void dma_chunks(const void* gsrc, uint32_t lane_off, uint32_t lds_wave_base) {
    static_assert(FIRST >= 0 && N >= 1 && FIRST + N <= 4, "immediate offsets of at most 3072");
    // both are wave-uniform by construction; say so where the compiler cannot prove it
    const uint64_t p = reinterpret_cast<uint64_t>(gsrc);
    gsrc = reinterpret_cast<const void*>(
        (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p) |
        ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32)) << 32));
    lds_wave_base = __builtin_amdgcn_readfirstlane(lds_wave_base);
#define FPS_DMA(more) asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:%3" more : \
                                   : "v"(lane_off), "s"(gsrc), "s"(lds_wave_base), "n"(1024 * FIRST), "n"(1024 * (FIRST + 1)), \
                                     "n"(1024 * (FIRST + 2)), "n"(1024 * (FIRST + 3)) : "memory", "m0")
#define FPS_DMA_AT(offset) "\n\tglobal_load_lds_dwordx4 %0, %1 offset:%" #offset
    if constexpr (N == 1)      FPS_DMA("");
    else if constexpr (N == 2) FPS_DMA(FPS_DMA_AT(4));
    else if constexpr (N == 3) FPS_DMA(FPS_DMA_AT(4) FPS_DMA_AT(5));
    else                       FPS_DMA(FPS_DMA_AT(4) FPS_DMA_AT(5) FPS_DMA_AT(6));
#undef FPS_DMA_AT
#undef FPS_DMA
}
// chunk c of a wave's contiguous share
__device__ __forceinline__ void dma_chunk(int c, const uint8_t* gsrc_wave, uint32_t lane_off, uint32_t lds_wave) {
    gsrc_wave += (c >> 2) * 4096;
    lds_wave += (c >> 2) * 4096;
    switch (c & 3) {
        case 0: dma_chunks<0, 1>(gsrc_wave, lane_off, lds_wave); break;
        case 1: dma_chunks<1, 1>(gsrc_wave, lane_off, lds_wave); break;
        case 2: dma_chunks<2, 1>(gsrc_wave, lane_off, lds_wave); break;
        default: dma_chunks<3, 1>(gsrc_wave, lane_off, lds_wave); break;
    }
}
// copy b of a wave's contiguous share of CHUNKS chunks: chunks 4b .. 4b + 3, or as many as there are
template <int CHUNKS>
__device__ __forceinline__ void dma_copy(int b, const uint8_t* gsrc_wave, uint32_t lane_off, uint32_t lds_wave) {
    gsrc_wave += b * 4096;
    lds_wave += b * 4096;
    if (b < CHUNKS / 4) dma_chunks<0, 4>(gsrc_wave, lane_off, lds_wave);
    else                dma_chunks<0, CHUNKS % 4 ? CHUNKS % 4 : 4>(gsrc_wave, lane_off, lds_wave);
}

// The kernels walk the key-tile box once per number NH = 2*SB .. 1 of 16-key halves: first every key
// block that fills its slots, then those of fewer halves, each with a main loop compiled for its NH
// (score and PV products by 32-key sub-blocks, row maxima and exponentials by halves), so that the
// padding of tiles cut by the grid's edge, or of tiles that do not fill their blocks, costs no more
// than the rest of its last half or sub-block.  Only O and the row sums live from one walk to the
// next; loops that hand over to each other in mid-pipeline need more registers than there are (250
// to 460 spilled in two such arrangements).  Whole path, walks by sub-blocks against blocks of 128
// slots with padding in tile order: 21x30x52 x 12 heads, tile (1,8,16), window 3x3x3: FP8 550 -> 514
// us, BF16 741 -> 664 us; tile (6,8,8) 614 -> 522 us; 21x45x80 x 40 heads, window 5x3x3: 4.59 -> 4.50
// ms, dense BF16 114.6 -> 110.1 ms.
//
// The box is walked in units of scale groups, which a window always takes whole.
struct KeyBox {
    int t0, t1, h0, h1, w0, w1;         // first and last key tile of the box, per axis
    uint32_t classes;                   // bit c: the box has sub-tiles of class c (cut along 4: T, 2: H, 1: W)
    __device__ __forceinline__ void init(const AttnArgs& a, int ut, int uh, int uw) {
        const Geom& G = a.g;
        if (a.edge_shift) {                 // clamp the centre into [r, n-1-r]; an axis not longer than
            // the window has no such centre and is kept whole by the truncation below with u = n/2
            ut = G.nT > 2 * a.rt + 1 ? min(max(ut, a.rt), G.nT - 1 - a.rt) : G.nT / 2;
            uh = G.nH > 2 * a.rh + 1 ? min(max(uh, a.rh), G.nH - 1 - a.rh) : G.nH / 2;
            uw = G.nW > 2 * a.rw + 1 ? min(max(uw, a.rw), G.nW - 1 - a.rw) : G.nW / 2;
        }
        t0 = max(0, ut - a.rt); h0 = max(0, uh - a.rh); w0 = max(0, uw - a.rw);
        t1 = min(G.nT - 1, ut + a.rt); h1 = min(G.nH - 1, uh + a.rh); w1 = min(G.nW - 1, uw + a.rw);
        const bool et = has_cut(t1, G.nT, G.cutT, G.Qt), eh = has_cut(h1, G.nH, G.cutH, G.Qh),
                   ew = has_cut(w1, G.nW, G.cutW, G.Qw);
        classes = ((has_full(t0, G.nsT, G.gT, et) ? 0x0Fu : 0u) | (et ? 0xF0u : 0u)) &
                  ((has_full(h0, G.nsH, G.gH, eh) ? 0x33u : 0u) | (eh ? 0xCCu : 0u)) &
                  ((has_full(w0, G.nsW, G.gW, ew) ? 0x55u : 0u) | (ew ? 0xAAu : 0u));
    }
    // the box ends with the axis' last sub-tile, and that one is cut
    static __device__ __forceinline__ bool has_cut(int last, int n, int cut, int q) { return last == n - 1 && cut < q; }
    static __device__ __forceinline__ bool has_full(int first, int ns, int g, bool cut) { return !cut || first * ns < g - 1; }
    // visited[v] = 1 for every tile of the box (threads of one workgroup)
    __device__ __forceinline__ void mark(const Geom& G, uint8_t* visited, int nthr) const {
        const int eh = h1 - h0 + 1, ew = w1 - w0 + 1, total = (t1 - t0 + 1) * eh * ew;
        for (int i = threadIdx.x; i < total; i += nthr) {
            const int t = i / (eh * ew), rem = i - t * (eh * ew), h = rem / ew, w = rem - h * ew;
            visited[((t0 + t) * G.nH + (h0 + h)) * G.nW + (w0 + w)] = 1;
        }
    }
};

// G.nh_classes as one word: a byte of it at an index known on the device only is a vector load of the arguments, which the
// waves that have rows wait for at the walk's first barrier (450 items of two groups 30.5 -> 30.2 us, 120 27.6 -> 27.0).  In the
// kernels of tiles of several blocks the word costs what it saves: 76 blocks of them 13.9 -> 14.1 us.
__device__ __forceinline__ uint64_t packed_classes(const Geom& G) {
    uint64_t w = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) w |= (uint64_t)G.nh_classes[i] << (8 * i);
    return w;
}

// n / d for n >= 0 of a lane and uniform d > 0, given rcp = 1.0f / d to an ulp or two: the estimate is exact
// below 2^20; beyond it (`large`, uniform) the loops settle it.  The walk waits for these divisions where a list begins:
// with the loops always there, and groups divided off tiles that are one, calls of few items were 3 to 11 % slower
// (18 items of (6,8,8) tiles, window 3x3x3, 26.2 us, now 23.2).
__device__ __forceinline__ int divide_lane(int n, int d, float rcp, bool large) {
    int q = (int)(((float)n + 0.5f) * rcp);
    if (large) {
        int r = n - q * d;
        while (r < 0) { --q; r += d; }
        while (r >= d) { ++q; r -= d; }
    }
    return q;
}

// One axis of a class of sub-tiles in the box: the sub-tiles first .. first + count - 1 along the axis.
struct AxisPart {
    int first, count;
    // the axis' full sub-tiles of the tiles lo .. hi, or (cut_part) only its last one, which is cut
    __device__ __forceinline__ AxisPart(int lo, int hi, int ns, int g, bool cut_part, bool has_cut) {
        first = cut_part ? g - 1 : lo * ns;
        count = cut_part ? 1 : min((hi + 1) * ns, g) - (has_cut ? 1 : 0) - first;
    }
};

// One key block: packed slots of one scale group, the first n of them real tokens.  Indices count from
// the head's first tile.
struct KeyBlock { int blk, group, n; };

// The key blocks of NH 16-key halves of the box, class by class, w fastest; of every KS of them the one with
// index kg (mod KS).  A lane works out the place of one block, so that a wave has the next 64 in two vector
// registers and a block costs its loop two v_readlane: stepping through the box axis by axis took 25 to 40 scalar
// instructions a block, and the FP8 kernel of tiles of several 128-slot blocks spilled 228 scalar registers to lanes
// of vector registers (now 20, with per-channel V 29; of several small groups a tile 0 to 59, with the keys split 10 to 36).
// Attention: 64-token sub-tiles of (2,8,16) tiles, 21x30x52 tokens x 24 heads, 1920 -> 1859 us, one-block tiles of that grid
// x 12 heads 315 -> 311.
template <bool MB, int KS>
struct BlockList {
    const Geom& G;
    const KeyBox& box;
    uint32_t classes;
    int NH, kg;
    int group, meta;                    // this lane's block: scale group; real tokens + 256 * (block within the group)
    __device__ __forceinline__ BlockList(const Geom& G_, const KeyBox& box_, int nh, uint32_t classes_, int kg_)
        : G(G_), box(box_), classes(classes_), NH(nh), kg(kg_), group(0), meta(0) {}
    // f(t, h, w parts, real tokens of a sub-tile, first block, blocks of NH halves) for every class
    template <typename F>
    __device__ __forceinline__ void for_classes(F&& f) const {
        const bool et = KeyBox::has_cut(box.t1, G.nT, G.cutT, G.Qt), eh = KeyBox::has_cut(box.h1, G.nH, G.cutH, G.Qh),
                   ew = KeyBox::has_cut(box.w1, G.nW, G.cutW, G.Qw);
        for (uint32_t left = classes; left; left &= left - 1) {
            const int c = __builtin_ctz(left);
            const AxisPart t(box.t0, box.t1, MB ? G.nsT : 1, G.gT, c & 4, et), h(box.h0, box.h1, MB ? G.nsH : 1, G.gH, c & 2, eh),
                w(box.w0, box.w1, MB ? G.nsW : 1, G.gW, c & 1, ew);
            const int n = ((c & 4) ? G.cutT : G.Qt) * ((c & 2) ? G.cutH : G.Qh) * ((c & 1) ? G.cutW : G.Qw);
            const int jb0 = NH == 8 || !MB ? 0 : n >> 7;       // 128-slot blocks; smaller groups have one
            f(t, h, w, n, jb0, MB && NH == 8 ? (n + 15) >> 7 : 1);
        }
    }
    __device__ __forceinline__ int total() const {
        int sum = 0;
        for_classes([&](const AxisPart& t, const AxisPart& h, const AxisPart& w, int, int, int blocks) FPS_INLINE {
            sum += t.count * h.count * w.count * blocks;
        });
        return sum;
    }
    // lane l gets the wave group's block first + l
    __device__ __forceinline__ void fill(int first) {
        int i = kg + KS * (first + (int)(threadIdx.x & 63));
        const bool large = G.M * (MB ? G.NS * G.KBG : 1) >= 1 << 20;    // a head's blocks, and so all that is divided here
        for_classes([&](const AxisPart& t, const AxisPart& h, const AxisPart& w, int n, int jb0, int blocks) FPS_INLINE {
            const int size = t.count * h.count * w.count * blocks;
            if (i >= 0 && i < size) {
                int rest = i, jb = jb0;
                if (MB && blocks > 1) {
                    const int q = divide_lane(rest, blocks, __builtin_amdgcn_rcpf((float)blocks), large);
                    jb += rest - q * blocks;
                    rest = q;
                }
                const int row = divide_lane(rest, w.count, __builtin_amdgcn_rcpf((float)w.count), large);
                const int layer = divide_lane(row, h.count, __builtin_amdgcn_rcpf((float)h.count), large);
                int it = t.first + layer, ih = h.first + row - layer * h.count, iw = w.first + rest - row * w.count;
                int sub = 0;                                   // scale group within its tile
                if (MB && G.NS > 1) {
                    const int ut = divide_lane(it, G.nsT, __builtin_amdgcn_rcpf((float)G.nsT), large),
                              uh = divide_lane(ih, G.nsH, __builtin_amdgcn_rcpf((float)G.nsH), large),
                              uw = divide_lane(iw, G.nsW, __builtin_amdgcn_rcpf((float)G.nsW), large);
                    sub = ((it - ut * G.nsT) * G.nsH + (ih - uh * G.nsH)) * G.nsW + (iw - uw * G.nsW);
                    it = ut; ih = uh; iw = uw;
                }
                const int tile = (it * G.nH + ih) * G.nW + iw;
                group = MB ? tile * G.NS + sub : tile;
                meta = (MB ? min(128, n - 128 * jb) : n) + 256 * jb;
            }
            i -= size;                                         // negative once found: sizes are below 2^31
        });
    }
    // block i of the wave group; fill() has covered it
    __device__ __forceinline__ KeyBlock block(int i) const {
        const int m = __builtin_amdgcn_readlane(meta, i & 63);
        KeyBlock b;
        b.group = __builtin_amdgcn_readlane(group, i & 63);
        b.n = m & 255;
        b.blk = MB ? b.group * G.KBG + (m >> 8) : b.group;
        return b;
    }
};

// Key split (KS > 1): the wave groups add up their O and row sums.  Each group takes 4 / KS of the channel blocks of 32, leaves
// what it has of the others in LDS with three numbers a lane, adds up its own after a barrier and stores it; the LDS holds the
// regions of the output transpose first.  (Group 0 adding up and storing everything, one group after the other: attention on
// 64 one-wave items of four groups, 4x16x16 tokens x 2 heads, 8.0 us, now 7.0, BF16 8.7, now 7.8; 225 items of two 36.6,
// now 35.6.)
template <int W, int KS>
struct SplitMerge {
    static constexpr int kOwn = 4 / KS;                    // channel blocks of a group
    static constexpr int kStoreBytes = store_region_bytes(kOwn);
    static constexpr int kWaveBytes = 64 * 16 * ((4 - kOwn) * 4 + 1);
    static constexpr int kBytes = KS * W * (kStoreBytes + kWaveBytes);
    uint8_t* lds;
    int row_block, kg, lane;            // the 32 query rows of the work item that the wave has; its group
    __device__ __forceinline__ uint8_t* store_region() const { return lds + (kg * W + row_block) * kStoreBytes; }
    __device__ __forceinline__ v4f* region(int from) const {
        return reinterpret_cast<v4f*>(lds + KS * W * kStoreBytes + (from * W + row_block) * kWaveBytes) + lane;
    }
    // where group `from` leaves its share of group `to`
    __device__ __forceinline__ v4f* share(int from, int to) const { return region(from) + (to - (to > from)) * kOwn * 4 * 64; }
    __device__ __forceinline__ void leave(const v16f (&acc)[4], float x, float y, float z = 0.f) const {
#pragma unroll
        for (int g = 0; g < KS; ++g) {
            if (g == kg) continue;
#pragma unroll
            for (int i = 0; i < 4 * kOwn; ++i) {
                const int db = g * kOwn + i / 4, r = 4 * (i & 3);
                share(kg, g)[i * 64] = v4f{acc[db][r], acc[db][r + 1], acc[db][r + 2], acc[db][r + 3]};
            }
        }
        region(kg)[(4 - kOwn) * 4 * 64] = v4f{x, y, z, 0.f};
    }
    __device__ __forceinline__ v4f numbers(int g) const { return region(g)[(4 - kOwn) * 4 * 64]; }
    // own = the sum over the groups of their accumulators, times factor[g]
    __device__ __forceinline__ void add(const v16f (&acc)[4], const float (&factor)[KS], v16f (&own)[kOwn]) const {
        float mine = factor[0];
#pragma unroll
        for (int g = 0; g < KS; ++g) {
            if (g != kg) continue;
            mine = factor[g];
#pragma unroll
            for (int j = 0; j < kOwn; ++j) own[j] = acc[g * kOwn + j];
        }
#pragma unroll
        for (int j = 0; j < kOwn; ++j) own[j] *= mine;
#pragma unroll
        for (int g = 0; g < KS; ++g) {
            if (g == kg) continue;
#pragma unroll
            for (int i = 0; i < 4 * kOwn; ++i) {
                const v4f v = share(g, kg)[i * 64];
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    own[i / 4][4 * (i & 3) + k] = __builtin_fmaf(v[k], factor[g], own[i / 4][4 * (i & 3) + k]);
            }
        }
    }
};

// Rows of two or of 4, 8, .. items are dealt in a turning order (see work_item): attention in order against turning, us:
//   2 items   20 tokens wide, 24 heads, tile (1,8,16)           213 -> 204
//   4         52 wide, 12 heads                                 366 -> 315    BF16 548 -> 503
//   8         120 wide, 6 heads; 52 wide, tile (2,8,16)         393 -> 384, 574 -> 548
//   16, 32    250 wide, tile (1,8,16); 52 wide, tile (4,16,16)  416 -> 412, 1456 -> 1408
//   12, 20    192 and 310 wide                                  419 -> 420, 400 -> 398
// Others spread by themselves, and turning costs them locality:
//   5, 7      80 and 112 wide                                   310 -> 313, 346 -> 345
//   6         96 wide, 8 heads; 720p of that width, 40 heads    386 -> 404, 4887 -> 5037    BF16 616 -> 644
//   10, 18    160 wide; 48 wide, tile (6,8,8)                   423 -> 426, 701 -> 705
inline bool deal_in_turns(int items_per_row) { return items_per_row % 4 == 0 || items_per_row == 2; }

// waves of a workgroup (= sub-blocks of a query block)
inline int query_waves(const Geom& g) {
    const int sb = g.BS == 128 ? 4 : g.KBS, tsb = g.TSP / 32;
    return sb == 4 || (g.NS > 1 && tsb % 4 == 0) ? 4 : sb;
}

// Key blocks of the largest walk box of a window, counting full tiles.
inline int window_blocks(const AttnArgs& a) {
    auto span = [](int n, int r) { return n < 2 * r + 1 ? n : 2 * r + 1; };
    const long long tiles = (long long)span(a.g.nT, a.rt) * span(a.g.nH, a.rh) * span(a.g.nW, a.rw);
    return (int)(tiles * a.g.NS * a.g.KBG > 1 << 20 ? 1 << 20 : tiles * a.g.NS * a.g.KBG);
}
// The keys of a work item are split over `ks` wave groups where all the launch's workgroups are resident at once
// with that, and the walk is long enough to pay for adding up.  Workgroups are placed whole: of 8 waves of these
// kernels' registers on each of 256 CUs, workgroups of three waves, split in two, fill six (300 items of 77 tokens:
// split 47.1 us FP8, 57.5 BF16, in a second and mostly empty round; not split 44.6 and 53.1), and the wave
// groups' LDS buffers (16 to 32 KB a wave) allow no more.  A wave alone on its SIMD takes 1.6 us a 128-key block, two that
// share one 2.3 us for two.  Attention, split against not, before SplitMerge's adding up was shared: 225 items of up to 27
// blocks 45.2 -> 37.9 us, of 6 blocks 15.5 -> 15.2, of 4 blocks 13.0 -> 13.6 (two groups); 64 one-wave items of up to 9 blocks
// 11.6 -> 10.3 (four groups).
inline bool split_keys(const AttnArgs& a, int ks) {
    const int resident = 256 * (8 / (query_waves(a.g) * ks)), blocks = window_blocks(a);
    return a.total <= resident && blocks >= 2 * ks && blocks >= 6;
}

// Narrow items: launches of few 128-row items are cut into items of 32 rows (FP8), whose keys four wave groups share, or of 64
// rows and two groups: four waves a workgroup either way (eight in narrow_in_four), and one buffer of K and V each (FP8 64 KB a
// workgroup of 64 rows, so two on a CU; 128 KB, one on a CU, of 32 rows and in BF16).  Twice or four times the workgroups reach
// more CUs, and where walks differ in length the longest, which the launch waits for, takes half a CU of its own.  Each
// workgroup stages K and V for itself, and a step has two barriers: where the CUs were loaded evenly, or the hardware puts two
// long items on one CU, that costs more.  79 000 random FP8 calls, time against 128 rows (keys in two groups up to 256
// items, else in one): cells' means, the slowest call and the share slower by 3 %, by items, blocks and the longest walk over
// the mean:
//   1-64       6 blocks or more                     0.55-0.72   0.95   none      (32 rows; 65 items and more 1.05 to 1.3)
//   65-128     6 or more                            0.64-0.83   0.99   none      (64 rows)
//   129-160    12 or more        1.3 or more        0.80-0.87   1.09   0.2 %
//   161-256    12 to 17          1.5 or more        0.88        1.06   0.9 %     (1.3 to 1.5 0.94, 1.13, 10 %: not taken)
//              18 to 59          1.4 or more        0.84-0.89   1.11   0.8 %     (1.3 to 1.4 0.89-0.91, 1.13, 3 %: not taken)
//              60 or more        1.3 or more        0.82-0.87   1.14   0.4 %
//   257-288    40 to 59          1.4 or more        0.79-0.85   1.07   0.3 %     (1.1 to 1.4 0.87-0.91, 1.30, 14 %: not taken)
//              60 or more        1.3 or more        0.74-0.86   1.09   0.3 %     (1.1 to 1.3 0.88, 1.13, 7 %: not taken)
//              40 or more        less than 1.1      0.82-0.85   1.12   2 %
//              30 to 39          1.4 or more        0.84-0.91   1.20   2 %       (less 0.85-0.93, 1.24, 15 %): not taken
//   289-320    30 or more        1.8 or more        0.74-0.83   0.98   none
//   321-400    40 or more        1.8 or more        0.81-0.85   1.07   0.3 %     (30 to 39 blocks 0.89, 1.10, 7 %: not taken)
// Where the slow calls are few no property of theirs was found that tells them apart.
// 225 items of up to 27 blocks, 5x23x37 tokens x 5 heads: 35.6 -> 30.9 us.
// BF16, 64 rows, up to 128 items, 18 000 calls: none slower; blocks 6-8 0.84, 9-29 0.81, more 0.79; 117 items of up to 21
// blocks 39.0 -> 31.0 us.  (2-3 blocks 0.94, 4-5 0.90, not taken; more than 128 items not measured.)
// Waves (of 32 rows) of an item; 128-slot blocks only, otherwise query_waves.
inline int narrow_waves(long long items, int blocks, double longest_over_mean) {
    if (blocks < 6 || items > 400) return 4;
    if (items <= 64) return 1;
    if (items <= 128) return 2;
    if (items <= 160) return blocks >= 12 && longest_over_mean >= 1.3 ? 2 : 4;
    const bool uneven = longest_over_mean >= (blocks >= 60 ? 1.3 : blocks >= 18 ? 1.4 : 1.5);
    if (items <= 256) return blocks >= 12 && uneven ? 2 : 4;
    if (items <= 288) return blocks >= 40 && (uneven || longest_over_mean < 1.1) ? 2 : 4;
    return blocks >= (items <= 320 ? 30 : 40) && longest_over_mean >= 1.8 ? 2 : 4;
}
inline int row_waves(const AttnArgs& a, int blocks, bool fp8) {
    const Geom& g = a.g;
    const long long items = (long long)g.BH * g.M * (g.TSP / 128);
    if (g.BS != 128 || items > 400) return query_waves(g);
    if (!fp8) return items <= 128 && blocks >= 6 ? 2 : 4;
    return narrow_waves(items, blocks, longest_over_mean(g, {a.rt, a.rh, a.rw}, a.edge_shift));
}

// FP8 items of 64 rows that leave CUs without a second workgroup (up to 128 items of 128 rows) and have long walks: four wave
// groups, 128 KB of buffers.  16 000 random calls of 65 to 128 items, time against two groups, by blocks: 6-8 1.06, 9-11 1.02,
// 12-29 0.97 (one in six slower by 5 % or more), 30-59 0.90, the slowest 1.10, more 0.86; 120 items of (4,8,8) tiles, window
// 3x9x9 of 60 blocks, 45.2 -> 41.7 us.  (Against 128 rows none of them is slower: see above.)
inline bool narrow_in_four(const AttnArgs& a) { return a.waves == 2 && a.total <= 256 && window_blocks(a) >= 30; }

// Cuts a launch into work items and plans the order in which they are dealt; returns the workgroups of an XCD.
//
// plan_items rounds every section up to the same number of slots on each XCD, so up to 256 items of 128 rows, cut in two, may
// need more than the 64 workgroups that an XCD holds at once, two on a CU; the last of them then wait for a long one to end.
// Those stay whole, one on a CU: cut in two, 240 random calls took 0.92 of that time, but one in eight was slower by 3 % or
// more, the slowest 1.34.
inline int plan_launch(AttnArgs& a, bool fp8) {
    const Geom& g = a.g;
    // narrow items in two groups are workgroups of four waves as well; the plans pass over launches of 256 workgroups or less,
    // which those in four groups are
    const int radius[3] = {a.rt, a.rh, a.rw}, row_bytes = fp8 ? 128 : 256, blocks = window_blocks(a), waves = query_waves(g);
    auto cut = [&](int of_rows) {
        a.waves = of_rows;
        a.qblocks = g.TSP / (32 * a.waves);
        a.rc_qblocks = reciprocal(a.qblocks);
        a.total = g.BH * g.M * a.qblocks;
        return plan_items(g, radius, a.edge_shift, a.qblocks, waves, row_bytes, blocks, a.plan);
    };
    int slots = cut(row_waves(a, blocks, fp8));
    if (a.waves < waves && a.total <= 512 && slots > 64) slots = cut(waves);
    a.rotate = deal_in_turns(g.nW * a.qblocks);
    a.chunk = ((a.total + 7) / 8 + 3) / 4 * 4;
    a.tail = -1;
    if (slots > 0) return slots;
    const int tail = plan_tail(g, radius, a.edge_shift, a.qblocks, waves, row_bytes, blocks, a.chunk, a.plan);
    a.tail = tail < 0 ? a.chunk : tail;
    return a.chunk;
}

// FP8, small scale groups: several key blocks go through a step together where the walk is long enough to pay for the part of
// the last step that may be empty and, in workgroups of fewer than four waves, for the one buffer of K and V that leaves
// room for.  There two blocks against one, 1.00 = as fast, 12x30x52 tokens in groups of 32 to 64, 3, 12 and 30 heads, both
// scale modes of V:
//   blocks of a window       7            9            15           21           25 to 28     35 to 45     60 and more
//   time                     0.99-1.08    0.99-1.07    0.98-1.04    0.95-1.02    0.94-1.03    0.95-1.00    0.93-1.02
// and of one block, on 21x30x52 tokens x 12 heads, 1.07 to 1.13.  Four waves have two buffers of either: of two blocks, groups
// of 64 tokens, 66.6 -> 67.6 us (216 tiles 8.1 -> 9.2), of four 81.9 -> 78.9, and of four groups of 16 tokens 121 -> 110.
inline bool blocks_together(const AttnArgs& a) { return window_blocks(a) >= (query_waves(a.g) == 4 ? 4 : 26); }

// Kernel launchers of the two precisions; grid: workgroups
void launch_attn_fp8(const AttnArgs& a, bool vch, int grid, hipStream_t st);
void launch_attn_bf16(const AttnArgs& a, int grid, hipStream_t st);
}  // namespace fps
