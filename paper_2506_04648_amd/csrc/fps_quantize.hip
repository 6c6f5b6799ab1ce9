// Per-group amax -> scale -> E4M3 encode (Sec. 3.2, Eq. 4-5; Algorithm 1 step 2), writing the
// packed operand layouts described in fps_layout.hip.  A scale group is a 3D tile, or a
// quantisation sub-tile of it.  The pass is HBM-bound (2 bytes read, 1 byte written per element) as long as
// the encoding takes few instructions and little code: a test for ties per element, with the exact
// quotient unrolled behind it, was 18 instructions per element and 29 to 85 KB of code to fetch, against
// now 7 and 5 to 11 KB.  Three tensors of 720p 629 -> 602 us (5.8 TB/s), of 480p (12 heads x 32760 tokens) 143 ->
// 101 us, in tiles of three blocks 221 -> 113 us, of 5 heads x 4255 tokens 54 -> 20 us.
#include "fps_device_common.h"

namespace fps {

// The key, within its 32-key sub-block, behind byte jj of the 16-byte chunk of lane half h -- where the
// accumulator of S^T = K Q^T left that key's weight
__device__ __forceinline__ int key_of_slot(int h, int jj) { return 8 * (jj >> 2) + 4 * h + (jj & 3); }

// Quotient x/s prepared for the hardware's round-to-nearest-even conversion so that the final code
// equals the rounding of the EXACT quotient: the correctly rounded float quotient can land exactly
// on an E4M3 rounding midpoint although the true quotient lies beside it; the sign of the exact
// residual x - q*s (one fma) tells on which side, and q is moved one float ulp that way.
__device__ __forceinline__ float quotient_for_rne(float x, float s) {
    if (s < 0x1p-60f) { x *= 0x1p64f; s *= 0x1p64f; }   // exactly; so that the residual does not underflow
    float q = x / s;
    uint32_t qb = __float_as_uint(q);
    const float a = __builtin_fabsf(q);
    bool mid;
    if (a >= 0.015625f) {
        mid = (qb & 0xFFFFFu) == 0x80000u;          // 3 mantissa bits kept, next bit set, rest zero
    } else {
        const float t = a * 1024.0f;                 // subnormal grid 2^-9: midpoints are odd * 2^-10
        mid = (t == __builtin_floorf(t)) && (((int)t) & 1);
    }
    if (mid) {
        const float r = __builtin_fmaf(-q, s, x);
        if (r != 0.0f) {
            const bool up = (r > 0.0f) == (q > 0.0f);
            qb = up ? qb + 1u : qb - 1u;             // magnitude one ulp up / down
            q = __uint_as_float(qb);
        }
    }
    return __builtin_fminf(__builtin_fmaxf(q, -448.0f), 448.0f);
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// How the elements of a scale s = RN(amax / 448) are divided by it: multiply by rs = 1/s, round the
// product to 17 significant bits, move it `nudge` float ulps away from (or towards) zero.
//
// Why that rounds to the code of the EXACT quotient x / s.  x and amax have 8 significant bits, X and A
// as integers, and the quotient is (1 + delta) times the ideal 448 x / amax = 7 X 2^j / A, delta the
// rounding error of s (|delta| <= 2^-24).  A rounding boundary of E4M3 is M 2^i with M < 32 odd (also in its
// subnormal range), and |7 X 2^j / A - M 2^i| is zero or at least 1/(A M) > 2^-13 of it.  So an
// ideal quotient off the boundaries stays on its side through all of these roundings and the nudge (below
// 2^-16 together: 2^-17 for the 17 bits, 2^-19 for 16 ulps, the rest single roundings);
// one ON a boundary comes out of the rounding to 17 bits as the boundary itself, and the exact
// quotient lies beside it in the direction of delta, which is the same for the whole scale group: exactly
// on it (a tie, for the conversion to settle) if 448 s = amax.  Ties of the ideal quotient are
// common: 6 % of the 16-channel units of normal data hold one.
//
// The product is formed as fma(x, rs, kTiny), so that a zero (padding, common) does not meet the nudge: it gives
// code 0, whatever its sign; per-channel scales keep the sign of a zero (SIGNED), as the quotient has it.  For
// other inputs the addend is far below an ulp of anything that does not round to zero.  No clamp is
// needed: |x| <= amax makes the product at most 448 (1 + 2^-18), far below the next boundary (464).
struct Divisor {
    float rs;
    int nudge;
};
__device__ __forceinline__ bool is_finite(float a) { return (__float_as_uint(a) & 0x7FFFFFFFu) < 0x7F800000u; }
constexpr float kTiny = 1.3e-30f;
__device__ __forceinline__ Divisor divisor_of(float s, float amax) {
    const float rest = __builtin_fmaf(-448.0f, s, amax);   // its sign is exact
    // NaN in a group: its scale is 1, exactly, and ties go to even
    return Divisor{1.0f / s, !is_finite(amax) ? 0 : rest > 0.0f ? 16 : rest < 0.0f ? -16 : 0};
}
// a scale below the normal range has lost bits of amax / 448, and its reciprocal may be infinite: the
// exact quotients are taken
__device__ __forceinline__ bool is_divisor(float s) { return __float_as_uint(s) >= 0x00800000u; }

template <bool SIGNED>
__device__ __forceinline__ float divide(float x, const Divisor& d) {
    const uint32_t q = __float_as_uint(__builtin_fmaf(x, d.rs, SIGNED ? __builtin_copysignf(kTiny, x) : kTiny));
    return __uint_as_float(((q + 0x40u) & ~0x7Fu) + (uint32_t)d.nudge);
}

// 16 bf16 (two uint4) -> 16 E4M3 codes (one uint4); scale(i), divisor(i): of element i.  One copy of the
// exact quotient in a loop: code that has to be fetched is what a launch of few workgroups waits for.
template <bool SIGNED, typename D, typename S>
__device__ __forceinline__ uint4 encode16(const uint4& lo, const uint4& hi, bool usable, D&& divisor, S&& scale) {
    const uint32_t w[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    uint32_t o[4];
    if (__builtin_expect(usable, 1)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int r = __builtin_amdgcn_cvt_pk_fp8_f32(divide<SIGNED>(bf16_lo(w[2 * i]), divisor(4 * i)),
                                                    divide<SIGNED>(bf16_hi(w[2 * i]), divisor(4 * i + 1)), 0, false);
            r = __builtin_amdgcn_cvt_pk_fp8_f32(divide<SIGNED>(bf16_lo(w[2 * i + 1]), divisor(4 * i + 2)),
                                                divide<SIGNED>(bf16_hi(w[2 * i + 1]), divisor(4 * i + 3)), r, true);
            o[i] = (uint32_t)r;
        }
    } else {
        uint4 a = lo, b = hi;
        o[0] = o[1] = o[2] = o[3] = 0u;
#pragma unroll 1
        for (int i = 0; i < 16; i += 2) {
            const int pair = __builtin_amdgcn_cvt_pk_fp8_f32(quotient_for_rne(bf16_lo(a.x), scale(i)),
                                                             quotient_for_rne(bf16_hi(a.x), scale(i + 1)), 0, false);
            a = make_uint4(a.y, a.z, a.w, b.x);
            b = make_uint4(b.y, b.z, b.w, 0u);
            // the codes move in from the top, two at a time
            o[0] = (o[0] >> 16) | (o[1] << 16);
            o[1] = (o[1] >> 16) | (o[2] << 16);
            o[2] = (o[2] >> 16) | (o[3] << 16);
            o[3] = (o[3] >> 16) | ((uint32_t)pair << 16);
        }
    }
    return make_uint4(o[0], o[1], o[2], o[3]);
}

// V block in LDS (row-major codes [token][128]) -> key-contiguous packed layout in HBM, by THREADS threads
template <int BS, int THREADS>
__device__ __forceinline__ void write_v_block(const uint8_t* stage, uint4* dst, int tid) {
#pragma unroll
    for (int c = tid; c < BS * 8; c += THREADS) {
        const int lane = c & 63, db = (c >> 6) & 3, kb = c >> 8;
        const int h = lane >> 5, n = lane & 31;
        union { uint4 v; uint8_t b[16]; } o;
#pragma unroll
        for (int jj = 0; jj < 16; ++jj)
            o.b[jj] = stage[(32 * kb + key_of_slot(h, jj)) * 128 + 32 * db + n];
        dst[c] = o.v;
    }
}

// THREADS threads per block of BS slots; a workgroup is one scale group of up to three blocks (NB), in a
// single pass over HBM: the whole group is held in registers while the amax is reduced, then encoded.
// Larger groups take their amax from block_amax_kernel (tile_amax != nullptr, NB = 1) and this kernel
// only encodes.
// RASTER: x is the raster tensor [BH,T,H,W,128] and the block's tokens are gathered from it (padded
// slots read as zero), which fuses the tile ordering of Sec. 3.2 step (1) into this pass.
template <int BS, int THREADS, bool RASTER, int NB>
__global__ __launch_bounds__(THREADS * NB) void quantize_tiles_kernel(const uint4* __restrict__ x,
                                                                      uint8_t* __restrict__ xq,
                                                                      float* __restrict__ scales, int role,
                                                                      Geom g, const float* __restrict__ tile_amax) {
    constexpr int U = BS * 8 / THREADS;             // 32-byte units (16 channels of one token) per thread
    constexpr int WAVES = THREADS * NB / 64;
    __shared__ uint32_t red[WAVES];
    __shared__ __attribute__((aligned(16))) uint8_t stage[NB * BS * 128];
    const int kb = NB > 1 ? (int)threadIdx.x / THREADS : 0, tid = threadIdx.x - kb * THREADS;
    const int blk = blockIdx.x * NB + kb;
    const BlockOrigin org = block_origin(g, blockIdx.x * NB);

    uint4 lo[U], hi[U];
    uint32_t mb = 0;
#pragma unroll
    for (int i = 0; i < U; ++i) {
        const int unit = tid + THREADS * i;          // token = unit >> 3, 16-channel group = unit & 7
        const uint4* row = token_row<RASTER>(x, g, org, kb * BS + (unit >> 3));
        lo[i] = make_uint4(0, 0, 0, 0);
        hi[i] = lo[i];
        if (row) { lo[i] = row[2 * (unit & 7)]; hi[i] = row[2 * (unit & 7) + 1]; }
    }
    float amax;
    if (tile_amax) {
        amax = tile_amax[blockIdx.x / g.KBS];
    } else {
#pragma unroll
        for (int i = 0; i < U; ++i) {
            mb = amax_pairs16(lo[i], mb);
            mb = amax_pairs16(hi[i], mb);
        }
        mb = workgroup_max<WAVES>(amax_of_pairs(mb), red);
        amax = __uint_as_float(mb << 16);
    }
    const float s = (amax == 0.0f) ? 1.0f : amax / 448.0f;   // Eq. 4 (correctly rounded division)
    if (!tile_amax && threadIdx.x == 0) scales[blockIdx.x] = s;   // the workgroup is the whole group

    const Divisor div = divisor_of(s, amax);
    const bool usable = is_divisor(s);
    uint4* dst = reinterpret_cast<uint4*>(xq + (long long)blk * (BS * 128));
    uint8_t* const staged = stage + kb * (BS * 128);
#pragma unroll
    for (int i = 0; i < U; ++i) {
        const int unit = tid + THREADS * i;
        const uint4 codes = encode16<false>(lo[i], hi[i], usable, [&](int) { return div; }, [&](int) { return s; });
        const int j = unit >> 3, c16 = unit & 7;
        if (role == FPS_ROLE_Q) {
            dst[unit] = codes;
        } else if (role == FPS_ROLE_K) {
            // 32x32x64 operand: lane 32h + n, k-step ks, 16-byte half e
            const int sb = j >> 5, n = j & 31, ks = c16 >> 2, h = (c16 >> 1) & 1, e = c16 & 1;
            dst[((sb * 2 + ks) * 2 + e) * 64 + 32 * h + n] = codes;
        } else {
            reinterpret_cast<uint4*>(staged)[unit] = codes;
        }
    }
    if (role == FPS_ROLE_V) {                        // uniform branch: role is a kernel argument
        __syncthreads();
        write_v_block<BS, THREADS>(staged, dst, tid);
    }
}

// ---- per-channel V (Sec. 3.2, Algorithm 1 step 3): s_c = max over ALL tokens of |V[:,c]| / 448 ----
// Stream-ordered kernels: clear the 128 per-head maxima; column maxima of every block merged with
// an atomic max on the bit pattern (|x| of a float orders like its unsigned pattern); encode every
// block with the per-channel scales; finally turn the stored maxima into scales in place.
// A workgroup of 256 threads takes `per` consecutive blocks of a head, thread = (token group tid/16, 8-channel
// chunk tid%16): the maxima stay in registers from block to block, and what costs as much as reading a block -- bringing
// those of 16 token groups together and 128 atomics in memory -- is done once.  The whole quantisation of V, a
// block a workgroup against up to eight, us: 10x30x52 tokens x 13 heads in 32-slot blocks, tile (3,4,4), 69.6 -> 45.3, x 25
// heads 105 -> 73.9; in 128-slot blocks x 13 and 25 heads 34.9 -> 34.0 and 52.8 -> 51.6, 40 heads of 720p 366 -> 345.
// NT: read past the caches (launch_quantize_channels).
template <int BS, bool RASTER, bool NT>
__global__ __launch_bounds__(256) void channel_amax_kernel(const uint4* __restrict__ x,
                                                           uint32_t* __restrict__ amax_bits, Geom g, int per,
                                                           int parts) {
    __shared__ uint4 red[4][16];
    const int tid = threadIdx.x, c8 = tid & 15;
    const int bh = blockIdx.x / parts, first = (blockIdx.x - bh * parts) * per, blocks = g.M * g.KB;
    const int last = first + per < blocks ? first + per : blocks;
    u16x2 m[4] = {};
#pragma unroll 1
    for (int b = first; b < last; ++b) {
        uint4 v[BS / 16];
        load_chunks<RASTER, 256, NT>(x, g, block_origin(g, bh * blocks + b), tid, 0, v);
#pragma unroll
        for (int i = 0; i < BS / 16; ++i) {
            const uint32_t w[4] = {v[i].x, v[i].y, v[i].z, v[i].w};
#pragma unroll
            for (int j = 0; j < 4; ++j)
                m[j] = __builtin_elementwise_max(m[j], __builtin_bit_cast(u16x2, w[j] & 0x7FFF7FFFu));
        }
    }
    // the four token groups of a wave, then the four waves
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            m[j] = __builtin_elementwise_max(
                m[j], __builtin_bit_cast(u16x2, __shfl_xor(__builtin_bit_cast(int, m[j]), off)));
    if ((tid & 63) < 16)
        red[tid >> 6][c8] = make_uint4(__builtin_bit_cast(uint32_t, m[0]), __builtin_bit_cast(uint32_t, m[1]),
                                       __builtin_bit_cast(uint32_t, m[2]), __builtin_bit_cast(uint32_t, m[3]));
    __syncthreads();
    if (tid < 128) {
        const uint16_t* const col = reinterpret_cast<const uint16_t*>(red) + tid;       // a row of 128 per wave
        uint32_t top = col[0];
#pragma unroll
        for (int i = 1; i < 4; ++i) top = col[128 * i] > top ? col[128 * i] : top;
        atomicMax(&amax_bits[bh * 128 + tid], top << 16);
    }
}

template <int BS, bool RASTER>
__global__ __launch_bounds__(256) void quantize_channels_kernel(const uint4* __restrict__ x,
                                                                uint8_t* __restrict__ xq,
                                                                const float* __restrict__ amax, Geom g) {
    __shared__ __attribute__((aligned(16))) uint8_t stage[BS * 128];
    __shared__ float sc[128];
    __shared__ Divisor div[128];
    __shared__ int exact;                                    // some channel's scale is no divisor
    const int tid = threadIdx.x, c16 = tid & 7;
    const int blk = blockIdx.x;
    const int bh = blk / (g.M * g.KB);
    const BlockOrigin org = block_origin(g, blk);
    if (tid == 0) exact = 0;
    constexpr int U = BS / 32;
    uint4 lo[U], hi[U];
#pragma unroll
    for (int i = 0; i < U; ++i) {                            // 16 channels of one token
        const uint4* row = token_row<RASTER>(x, g, org, (tid >> 3) + 32 * i);
        lo[i] = make_uint4(0, 0, 0, 0);
        hi[i] = lo[i];
        if (row) { lo[i] = row[2 * c16]; hi[i] = row[2 * c16 + 1]; }
    }
    __syncthreads();
    if (tid < 128) {
        const float a = amax[bh * 128 + tid];
        const float s = a == 0.0f ? 1.0f : a / 448.0f;
        sc[tid] = s;
        div[tid] = divisor_of(s, a);
        // beside a channel with an infinity or a NaN the exact quotients are taken too: their clamp makes those -448
        const bool bad = !is_divisor(s) || !is_finite(a);
        if (__ballot(bad) != 0 && (tid & 63) == 0) exact = 1;
    }
    __syncthreads();
    Divisor d[16];                                           // of the thread's 16 channels
#pragma unroll
    for (int i = 0; i < 16; ++i) d[i] = div[c16 * 16 + i];
    const bool usable = exact == 0;
#pragma unroll
    for (int i = 0; i < U; ++i)
        reinterpret_cast<uint4*>(stage)[tid + 256 * i] =
            encode16<true>(lo[i], hi[i], usable, [&](int k) { return d[k]; }, [&](int k) { return sc[c16 * 16 + k]; });
    __syncthreads();
    write_v_block<BS, 256>(stage, reinterpret_cast<uint4*>(xq + (long long)blk * (BS * 128)), tid);
}

template <int BS, bool RASTER>
static void launch_channel_amax_from(const Geom& g, const uint4* x, bool past_caches, uint32_t* amax, int per, int parts,
                                     int grid, hipStream_t st) {
    if (past_caches) channel_amax_kernel<BS, RASTER, true><<<grid, 256, 0, st>>>(x, amax, g, per, parts);
    else             channel_amax_kernel<BS, RASTER, false><<<grid, 256, 0, st>>>(x, amax, g, per, parts);
}
template <int BS>
static void launch_channel_amax(const Geom& g, const uint4* x, int raster, bool past_caches, uint32_t* amax, int per, int parts,
                                int grid, hipStream_t st) {
    if (raster) launch_channel_amax_from<BS, true>(g, x, past_caches, amax, per, parts, grid, st);
    else        launch_channel_amax_from<BS, false>(g, x, past_caches, amax, per, parts, grid, st);
}

static int launch_quantize_channels(const Geom& g, const void* x, int raster, void* xq, float* scales,
                                    hipStream_t st) {
    const int blocks = g.BH * g.M * g.KB, n = g.BH * 128;
    const uint4* xi = (const uint4*)x;
    uint8_t* xo = (uint8_t*)xq;
    clear_kernel<<<(n + 255) / 256, 256, 0, st>>>((uint32_t*)scales, n);
    // as many blocks a workgroup, up to 8, as leave 2048 workgroups, eight a CU
    const int head = g.M * g.KB, most = blocks / 2048, per = most < 1 ? 1 : most > 8 ? 8 : most;
    const int parts = (head + per - 1) / per, grid = g.BH * parts;
    uint32_t* const amax = (uint32_t*)scales;
    // V and its codes together beyond the Infinity Cache's 256 MB: nothing of V would be left when it is read again, so it
    // leaves the cache to what else is there.  The whole quantisation, cached against past the caches, us: V and codes of
    // 40 MB 20.9 -> 21.6, 185 MB 73.9 -> 77.6, 252 MB 72.9 -> 74.6, 281 MB 105 -> 109; 331 and 370 MB 93.6 -> 93.8 and 137 -> 138;
    // 417 MB 128 -> 121, 550 MB 183 -> 171, 40 heads of 720p, 1.2 GB, 374 -> 345.
    const long long slots = (long long)blocks * g.BS, tokens = raster ? (long long)g.BH * g.T * g.H * g.W : slots;
    const bool past_caches = 256 * tokens + 128 * slots > (320LL << 20);
    if (g.BS == 128) launch_channel_amax<128>(g, xi, raster, past_caches, amax, per, parts, grid, st);
    else             launch_channel_amax<32>(g, xi, raster, past_caches, amax, per, parts, grid, st);
    if (g.BS == 128) {
        if (raster) quantize_channels_kernel<128, true><<<blocks, 256, 0, st>>>(xi, xo, scales, g);
        else        quantize_channels_kernel<128, false><<<blocks, 256, 0, st>>>(xi, xo, scales, g);
    } else {
        if (raster) quantize_channels_kernel<32, true><<<blocks, 256, 0, st>>>(xi, xo, scales, g);
        else        quantize_channels_kernel<32, false><<<blocks, 256, 0, st>>>(xi, xo, scales, g);
    }
    amax_to_scale_kernel<<<(n + 255) / 256, 256, 0, st>>>(scales, n);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? FPS_OK : hip_fail(e, "quantize_channels launch");
}

// Threads per block of slots.  More loads in flight per thread keep the memory system busier at large sizes,
// more threads shorten a small launch: 3 tensors of 720p (40 heads x 75600 tokens, 25200 blocks) take 602
// us with 256 threads and 680 us with 512; of 5 heads x 4255 tokens, 20 and 19 us.  In 32-slot blocks
// (21x30x52 tokens x 12 heads in tiles of 48) 139, 109 and 106 us with 256, 128 and 64 threads, the
// smallest launches alike.
template <int BS> constexpr int kQuantThreads = BS == 128 ? 256 : 128;

template <int BS, int NB>
static void launch_quantize_nb(const Geom& g, const uint4* xi, int raster, int role, uint8_t* xo, float* scales,
                               const float* tile_amax, int grid, hipStream_t st) {
    constexpr int TH = kQuantThreads<BS>;
    if (raster) quantize_tiles_kernel<BS, TH, true, NB><<<grid, TH * NB, 0, st>>>(xi, xo, scales, role, g, tile_amax);
    else        quantize_tiles_kernel<BS, TH, false, NB><<<grid, TH * NB, 0, st>>>(xi, xo, scales, role, g, tile_amax);
}

int launch_quantize(const Geom& g, const void* x, int raster, int role, int vscale, void* xq,
                    float* scales, hipStream_t st) {
    if (vscale != FPS_VSCALE_TILE) return launch_quantize_channels(g, x, raster, xq, scales, st);
    const int blocks = g.BH * g.M * g.KB, groups = g.BH * g.M * g.NS;
    const uint4* xi = (const uint4*)x;
    uint8_t* xo = (uint8_t*)xq;
    if (g.KBS <= 3) {                   // one workgroup per scale group: a single pass over the input
        if (g.BS == 128) {
            switch (g.KBS) {
                case 1: launch_quantize_nb<128, 1>(g, xi, raster, role, xo, scales, nullptr, groups, st); break;
                case 2: launch_quantize_nb<128, 2>(g, xi, raster, role, xo, scales, nullptr, groups, st); break;
                default: launch_quantize_nb<128, 3>(g, xi, raster, role, xo, scales, nullptr, groups, st); break;
            }
        } else {                        // 32-slot blocks: groups of at most 96 tokens, three blocks
            switch (g.KBS) {
                case 1: launch_quantize_nb<32, 1>(g, xi, raster, role, xo, scales, nullptr, groups, st); break;
                case 2: launch_quantize_nb<32, 2>(g, xi, raster, role, xo, scales, nullptr, groups, st); break;
                default: launch_quantize_nb<32, 3>(g, xi, raster, role, xo, scales, nullptr, groups, st); break;
            }
        }
    } else {                            // group amax over many blocks first; `scales` holds it meanwhile
        clear_kernel<<<(groups + 255) / 256, 256, 0, st>>>((uint32_t*)scales, groups);
        launch_block_amax<128>(x, raster, scales, g, st);
        launch_quantize_nb<128, 1>(g, xi, raster, role, xo, scales, scales, blocks, st);
        amax_to_scale_kernel<<<(groups + 255) / 256, 256, 0, st>>>(scales, groups);
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? FPS_OK : hip_fail(e, "quantize_tiles launch");
}

}  // namespace fps
