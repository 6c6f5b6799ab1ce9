// BF16 attention kernel: no quantisation.  K Q^T on v_mfma_f32_32x32x16_bf16; P is rounded to fp16 and
// multiplied with the fp16 V tiles (exact per-tile power-of-two scaling, undone by s^V) on
// v_mfma_f32_32x32x16_f16.  The in-wave pipeline and lane layout of the FP8 kernel.  A 128-slot block
// pair is 64 KB here, so K and V are single-buffered: V(i) streams in while P(i) is taken (after every
// wave has finished PV(i-1)), K(i+2) during PV(i) (after every wave has finished QK(i+1)); two barriers
// per iteration.
// V's scale per group is a power of two, so the PV product accumulates straight into O: O is kept relative to
// 2^e_ref, and a block's weights are 2^(S' + log2(s^V) - e_ref) with 2^14 on top, rounded to fp16.  e_ref
// moves, and O with it (exactly: powers of two), where a block needs it:
//   up,   so that no weight of the block exceeds 2^14: e_ref >= log2(s^V) + the block's row maximum;
//   down, so that the block's weights keep their bits: e_ref <= log2(s^V) + m + kMaxFold, m the row reference.
// fp16 holds all 11 bits of weights down to 2^-28 of 2^e_ref, hence those of at least 2^-24 of the row's largest
// weight whatever the scales of the groups met before -- a group of zeros (scale 1) beside values of 1e-6, or a
// group of large values whose keys have no weight.  Following only the largest scale met, as in a
// running maximum, such groups cost the row one bit per binade: output errors of 0.3 RMS at V of 1e-6 beside zeros.
// Groups of like magnitude never move O down.
#include "fps_attn_device.h"

namespace fps {

union Bf16x8 { uint4 u; v8bf v; v8h h; };
constexpr int kMaxFold = 4;                // binades by which a block's weights may lie under 2^14

template <int SB, int W, bool MB, int KS>
__global__ __launch_bounds__(KS * W * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_bf16_kernel(AttnArgs a) {
    load_arguments<(sizeof(AttnArgs) + 63) / 64>();
    constexpr int NTHR = KS * W * 64;
    constexpr int CPT = SB * 8 / W;                        // 16-byte chunks per thread per operand block
    constexpr int BLOCK_BYTES = SB * 8192;
    static_assert(CPT >= 1 && CPT <= 16 && CPT * W == SB * 8, "every wave copies the same share of a block");
    constexpr int GROUP_BYTES = 2 * BLOCK_BYTES;           // K, V
    constexpr int END_BYTES = KS > 1 ? SplitMerge<W, KS>::kBytes : W * store_region_bytes(4);
    constexpr int LDS_BYTES = KS * GROUP_BYTES > END_BYTES ? KS * GROUP_BYTES : END_BYTES;
    // the groups' blocks; afterwards their sums and the output transpose
    __shared__ __attribute__((aligned(16))) uint8_t lds[LDS_BYTES];
    const Geom& G = a.g;
    const int NS = MB ? G.NS : 1;
    const int KBG = MB && SB == 4 ? G.KBG : 1;             // key blocks of a scale group
    const int TSB = MB ? NS * KBG * SB : SB;               // sub-blocks of a tile
    int bh, ut, uh, uw, jq;
    if (!work_item(a, &bh, &ut, &uh, &uw, &jq)) return;
    const int u = (ut * G.nH + uh) * G.nW + uw;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5, n = lane & 31;
    const int wave_s = __builtin_amdgcn_readfirstlane(wave) % W, kg = KS > 1 ? __builtin_amdgcn_readfirstlane(wave) / W : 0;
    const int ucls = tile_class(G, ut, uh, uw);
    // the wave's sub-block of query rows; rotated from tile to tile (and wave group to wave group) so that the idle
    // waves of cut tiles fall on different SIMDs
    const int row_block = W == 4 || (SB == 4 && W == 2) ? (wave_s + kg + u) & (W - 1) : wave_s;
    if (MB && !a.out_raster) {                             // all items of a tile clear the padding of its output
        QueryRows slots;
        slots.init<MB>(G, bh, u, ucls, ut, uh, uw, jq * W + row_block, KBG * SB);
        zero_padding_rows(a, slots, ucls, lane);
    }
    const int taken = wave_sub_block<SB, W, MB>(G, ucls, jq, row_block, KBG * SB), qs = taken < 0 ? 0 : taken;
    if (MB && taken == -2) return;
    QueryRows rows;
    rows.init<MB>(G, bh, u, ucls, ut, uh, uw, qs, KBG * SB);
    if (MB && taken < 0) rows.rows = 0;
    if (!MB) zero_padding_rows(a, rows, ucls, lane);
    // no wave of the item has a row
    if ((MB || W < SB) && (W == 1 ? rows.rows <= 0 : NS == 1 && rows.box.n <= 32 * W * jq)) return;
    const size_t tile0 = (size_t)bh * G.M;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(&lds[0]) + kg * GROUP_BYTES;
    KeyBox box;
    box.init(a, ut, uh, uw);
    if (a.visited && bh == 0 && jq == 0) box.mark(G, a.visited + (size_t)u * G.M, NTHR);

    const uint8_t* const k_head = a.k + tile0 * TSB * 8192;
    const uint8_t* const v_head = a.v + tile0 * TSB * 8192;
    const float* const sv_head = a.sv + tile0 * NS;
    auto k_blk = [&](const KeyBlock& b) FPS_INLINE { return k_head + (size_t)b.blk * BLOCK_BYTES; };
    auto v_blk = [&](const KeyBlock& b) FPS_INLINE { return v_head + (size_t)b.blk * BLOCK_BYTES; };
    auto stage_chunk = [&](int buf, const uint8_t* src, int c) FPS_INLINE {
        dma_chunk(c, src + wave_s * (CPT * 1024), lane * 16, lds_base + buf * BLOCK_BYTES + wave_s * (CPT * 1024));
    };
    auto stage = [&](int buf, const uint8_t* src) FPS_INLINE {
#pragma unroll
        for (int c = 0; c < (CPT + 3) / 4; ++c)
            dma_copy<CPT>(c, src + wave_s * (CPT * 1024), lane * 16, lds_base + buf * BLOCK_BYTES + wave_s * (CPT * 1024));
    };

    typedef BlockList<MB, KS> List;
    // Of a list of `total` blocks, those of this wave group.  Group 0 never has fewer than another; what a group
    // has fewer barriers than group 0 (two a block, three a list) it makes up for at the end, as every barrier
    // is one of the whole workgroup.  (Made up for within the list, they cost 110 spilled registers.)
    int owed = 0;
    auto blocks_of_group = [&](int total) FPS_INLINE {
        if (KS == 1) return total;
        const int nblk = (total - kg + KS - 1) / KS;
        owed += 2 * ((total + KS - 1) / KS - nblk) + (nblk == 0 ? 3 : 0);
        return nblk;
    };
    auto make_up = [&]() FPS_INLINE {
        if (KS > 1)
            for (; owed > 0; --owed) __syncthreads();
    };

    if (rows.rows <= 0) {
        // no real row: this wave only copies its share of the K and V blocks, barrier for barrier
        const uint64_t all_classes = MB ? 0 : packed_classes(G);
        for (int nh = 2 * SB; nh >= 1; --nh) {
            const uint32_t classes = (MB ? G.nh_classes[nh - 1] : (uint32_t)(all_classes >> (8 * (nh - 1)))) & box.classes;
            if (!classes) continue;
            List list(G, box, nh, classes, kg);
            const int nblk = blocks_of_group(list.total());
            if (nblk == 0) continue;
            list.fill(0);
            KeyBlock cur = list.block(0), nxt = cur;
            stage(0, k_blk(cur));
            if (nblk > 1) nxt = list.block(1);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();                               // K(0) visible
            __syncthreads();                               // QK(0) done
            if (nblk > 1) stage(0, k_blk(nxt));
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            for (int i = 0; i < nblk; ++i) {
                stage(1, v_blk(cur));
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();                           // QK(i+1) done; V(i) visible
                cur = nxt;
                if (i + 2 < nblk) {
                    if (((i + 2) & 63) == 0) list.fill(i + 2);
                    nxt = list.block(i + 2);
                    stage(0, k_blk(nxt));
                }
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();                           // PV(i) done; K(i+2) visible
            }
        }
        make_up();
        if (KS > 1) __syncthreads();
        return;
    }

    Bf16x8 qop[8];                                         // Q^T, contraction steps of 16 channels
    float m_run = -INFINITY, l_run = 0.f;                  // row reference; sum of 2^14 P relative to it
    float e_ref = 0.f;                                     // O is relative to 2^e_ref
    int e_v_max = -127;                                    // of the largest V scale met
    v16f acc[4];
    {
        const uint4* p = reinterpret_cast<const uint4*>(a.q + (((tile0 + u) * TSB + qs) * 32 + n) * 256);
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) qop[ks].u = p[2 * ks + h];
#pragma unroll
        for (int db = 0; db < 4; ++db) acc[db] = zero16();
    }
    const float sc = kLog2eOverSqrtD;
    const uint4* ldsK4 = reinterpret_cast<const uint4*>(lds + kg * GROUP_BYTES);
    const uint4* ldsV4 = reinterpret_cast<const uint4*>(lds + kg * GROUP_BYTES + BLOCK_BYTES);

    auto pipeline = [&](auto nh_tag) FPS_INLINE {
        constexpr int NH = decltype(nh_tag)::value;        // 16-key halves
        constexpr int NB = (NH + 1) / 2;                   // 32-key sub-blocks
        const uint32_t classes = G.nh_classes[NH - 1] & box.classes;
        if (!classes) return;
        List list(G, box, NH, classes, kg);
        const int nblk = blocks_of_group(list.total());
        if (nblk == 0) return;
        list.fill(0);

        v16f s[NB];                                        // S^T, blocks of 32 keys
        Bf16x8 pop[NH];                                // P^T in fp16: contraction steps of 16 keys
        Bf16x8 ring[4];                                    // MFMA operands on their way from LDS
        float alpha_acc = 1.f;                             // rescale owed to O before the block's PV
        float alpha_l = 1.f, cm = 0.f;
        float to_l = 0.f;                                  // log2 of what the weights' sum counts in the row sum

        // operand j of the K block: key block j/8, contraction step j%8
        auto k_operand = [&](int j) FPS_INLINE { return ldsK4[j * 64 + lane]; };
        auto qk_step = [&](int j) FPS_INLINE {
            const int kb = j >> 3, ks = j & 7;
            s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[j & 3].v, qop[ks].v, ks == 0 ? zero16() : s[kb], 0, 0, 0);
        };
        // PV instructions alternate between two channel blocks, so that consecutive ones do not depend
        // on each other: instruction j -> channel block 2(j / 2NH) + j%2, contraction step (j % 2NH)/2
        auto pv_db = [](int j) { return 2 * (j / (2 * NH)) + (j & 1); };
        auto pv_kk = [](int j) { return (j % (2 * NH)) >> 1; };
        auto v_operand = [&](int j) FPS_INLINE { return ldsV4[(pv_kk(j) * 4 + pv_db(j)) * 64 + lane]; };
        auto pv_step = [&](int j) FPS_INLINE {
            acc[pv_db(j)] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ring[j & 3].h, pop[pv_kk(j)].h, acc[pv_db(j)], 0, 0, 0);
        };
        // a pair of weights (registers 2i, 2i + 1 of score block kb) in fp16
        auto weights_pair = [&](int kb, int i, float& rs) FPS_INLINE {
            const float p0 = fast_exp2(__builtin_fmaf(s[kb][2 * i], sc, cm));
            const float p1 = fast_exp2(__builtin_fmaf(s[kb][2 * i + 1], sc, cm));
            rs += p0;
            rs += p1;
            uint32_t wd = __builtin_bit_cast(uint32_t, __builtin_convertvector(v2f{p0, p1}, v2h));
            asm volatile("" : "+v"(wd), "+v"(rs));         // keep the pass in place
            reinterpret_cast<uint32_t*>(&pop[2 * kb + (i >> 2)].u)[i & 3] = wd;
        };
        // the row reference and weight exponents of the block whose row maximum mx was taken; svv: its
        // V scale, 2^e exactly.  O holds every earlier block but for the rescale alpha_acc.
        auto new_reference = [&](float mx, float svv) FPS_INLINE {
            const int e_vi = (int)((__float_as_uint(svv) >> 23) & 0xFFu) - 127;
            const float e_v = (float)e_vi;
            const float top = __builtin_ceilf(max_over_row_pair(mx) * sc);
            const float m_new = __builtin_fmaxf(m_run, top);
            const float e_low = e_v + top;
            float e_new = m_run == -INFINITY ? e_low : __builtin_fmaxf(e_ref, e_low);
            const float e_high = e_v + m_new + (float)kMaxFold;
            // e_ref <= e_v_max + m_run, so groups of like magnitude need only a scalar comparison here
            if (e_vi + kMaxFold < e_v_max && __any(e_new > e_high)) {
                // O moves down, as far as its largest element allows: up to 2^100 (2^126 times at most)
                float o = 0.f;
#pragma unroll
                for (int db = 0; db < 4; ++db)
#pragma unroll
                    for (int r = 0; r < 16; ++r) o = __builtin_fmaxf(o, __builtin_fabsf(acc[db][r]));
                const int e_o = (int)(__float_as_uint(max_over_row_pair(o)) >> 23) - 127;
                e_new = __builtin_fmaxf(__builtin_fminf(e_new, e_high), e_new - (float)min(99 - e_o, 126));
            }
            e_v_max = max(e_v_max, e_vi);
            alpha_l = fast_exp2(m_run - m_new);            // 0 on the first block (m_run = -inf)
            alpha_acc = m_run == -INFINITY ? 1.0f : fast_exp2(e_ref - e_new);
            m_run = m_new;
            e_ref = e_new;
            // <= 0: the block's largest weight relative to 2^14; 64 binades down every fp16 weight is zero
            const float below = __builtin_fmaxf(e_low - e_new, -64.0f);
            // 2^14 * 2^(S' - top) * 2^below: the factor 2^14 keeps small weights in fp16's normal range
            // and cancels against the row sum, which is taken of the same values
            cm = kFp16PScaleLog2 - top + below;
            to_l = top - m_new - below;
        };

        // prologue: S(0) and its row reference, then K(1) on its way
        KeyBlock cur = list.block(0), nxt = cur;
        stage(0, k_blk(cur));
        float svv = load_uniform(sv_head, cur.group);
        if (nblk > 1) nxt = list.block(1);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 8 * NB; ++j) {
            ring[j & 3].u = k_operand(j);
            qk_step(j);
        }
        // every wave has finished QK(0), so the K buffer is free: K(1) is on its way while the row maximum is taken
        __syncthreads();
        if (nblk > 1) stage(0, k_blk(nxt));
        if (cur.n < 16 * NH) mask_cut_half(s[NB - 1], (NH - 1) & 1, cur.n - 16 * (NH - 1), h);
        {
            float mx = -INFINITY;
#pragma unroll
            for (int k = 0; k < 4 * NH; ++k)
                mx = __builtin_fmaxf(__builtin_fmaxf(mx, s[k >> 3][2 * (k & 7)]), s[k >> 3][2 * (k & 7) + 1]);
            new_reference(mx, svv);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();

        // iteration i: P(i) | S(i+1) = K(i+1) Q^T | V(i) streams in, then row maximum of S(i+1) |
        // O += V^T P^T (i) | K(i+2) streams in
        for (int i = 0; i + 1 < nblk; ++i) {
            const uint8_t* vsrc = v_blk(cur);
            const int n_next = nxt.n;
            const float svv_next = load_uniform(sv_head, nxt.group);
            cur = nxt;
            // past the walk's end the last K is copied once more and nobody reads it (with the copies under a condition, which
            // cuts the steps of PV into pieces, dense 720p took 108.0 ms, now 106.9)
            if (i + 2 < nblk) {
                if (((i + 2) & 63) == 0) list.fill(i + 2);
                nxt = list.block(i + 2);
            }
            const uint8_t* ksrc = k_blk(nxt);

            // step (kb, ks): a pair of weights of score block kb beside the MFMA (kb - 1, ks) that
            // refills the block whose weights were taken one block earlier
            float rs = 0.f;
#pragma unroll
            for (int j = 0; j < 3; ++j) ring[j].u = k_operand(j);
#pragma unroll
            for (int kb = 0; kb <= NB; ++kb) {
#pragma unroll
                for (int ks = 0; ks < 8; ++ks) {
                    const int j = (kb - 1) * 8 + ks;
                    if (kb >= 1) {
                        if (j + 3 < 8 * NB) ring[(j + 3) & 3].u = k_operand(j + 3);
                        qk_step(j);
                    }
                    if (8 * kb + ks < 4 * NH) weights_pair(kb, ks, rs);
                    if (kb * 8 + ks < CPT) stage_chunk(1, vsrc, kb * 8 + ks);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            l_run = __builtin_fmaf(rs, fast_exp2(to_l), l_run * alpha_l);
            if (n_next < 16 * NH) mask_cut_half(s[NB - 1], (NH - 1) & 1, n_next - 16 * (NH - 1), h);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // V(i): this thread's share landed
            __syncthreads();             // every wave has finished QK(i+1): the K buffer is free; V(i) visible

            if (__any(alpha_acc != 1.0f)) {
#pragma unroll
                for (int db = 0; db < 4; ++db) acc[db] *= alpha_acc;
            }
            float mx = __builtin_fmaxf(__builtin_fmaxf(s[0][0], s[0][1]), __builtin_fmaxf(s[0][2], s[0][3]));
#pragma unroll
            for (int j = 0; j < 3; ++j) ring[j].u = v_operand(j);
#pragma unroll
            for (int j = 0; j < 4 * NH; ++j) {             // one MFMA and one max3 per step
                if (j + 3 < 4 * NH) ring[(j + 3) & 3].u = v_operand(j + 3);
                pv_step(j);
                if (j >= 2) {
                    mx = __builtin_fmaxf(__builtin_fmaxf(mx, s[j >> 3][2 * (j & 7)]), s[j >> 3][2 * (j & 7) + 1]);
                    asm volatile("" : "+v"(mx));
                }
                // K's copies ride in the first half, so that they have landed when the phase ends: one every other step where a
                // block has as many halves as a wave has copies, otherwise one a step, or as many a step as it takes, up
                // to eight (32-token tiles, window 5x21x21: 354 -> 334 us, one a step against two)
                constexpr int every = NH >= CPT ? 2 : 1, per = (CPT + 2 * NH - 1) / (2 * NH);
                if (j % every == 0) {
#pragma unroll
                    for (int c = j / every * per; c < (j / every + 1) * per && c < CPT; ++c) stage_chunk(0, ksrc, c);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            svv = svv_next;
            new_reference(mx, svv);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // K(i+2): this thread's share landed
            __syncthreads();             // every wave has finished PV(i): the V buffer is free; K(i+2) visible
        }

        // the last block's P and PV
        stage(1, v_blk(cur));
        float rs = 0.f;
#pragma unroll
        for (int k = 0; k < 4 * NH; ++k) weights_pair(k >> 3, k & 7, rs);
        l_run = __builtin_fmaf(rs, fast_exp2(to_l), l_run * alpha_l);
        if (__any(alpha_acc != 1.0f)) {
#pragma unroll
            for (int db = 0; db < 4; ++db) acc[db] *= alpha_acc;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 4 * NH; ++j) {
            ring[j & 3].u = v_operand(j);
            pv_step(j);
        }
        __syncthreads();                                   // both buffers are free
    };
    if constexpr (SB > 3) { pipeline(Count<8>{}); pipeline(Count<7>{}); }
    if constexpr (SB > 2) { pipeline(Count<6>{}); pipeline(Count<5>{}); }
    if constexpr (SB > 1) { pipeline(Count<4>{}); pipeline(Count<3>{}); }
    pipeline(Count<2>{});
    pipeline(Count<1>{});

    make_up();
    if constexpr (KS > 1) {                                // every wave is done with the buffers
        // O of a group is relative to 2^e_ref, l to 2^m_run: moving both to the largest is exact
        typedef SplitMerge<W, KS> Merge;
        const Merge merge{lds, row_block, kg, lane};
        // without a block: O and l are zero and their references the lowest
        merge.leave(acc, m_run == -INFINITY ? -INFINITY : e_ref, l_run, m_run);
        __syncthreads();
        v4f o[KS];
        float top = -INFINITY, m_top = -INFINITY, l = 0.f, factor[KS];
#pragma unroll
        for (int g = 0; g < KS; ++g) {
            o[g] = merge.numbers(g);
            top = __builtin_fmaxf(top, o[g][0]);           // finite: group 0 has a block
            m_top = __builtin_fmaxf(m_top, o[g][2]);
        }
#pragma unroll
        for (int g = 0; g < KS; ++g) {
            factor[g] = fast_exp2(o[g][0] - top);
            l = __builtin_fmaf(o[g][1], fast_exp2(o[g][2] - m_top), l);
        }
        v16f own[Merge::kOwn];
        merge.add(acc, factor, own);
        l = sum_over_row_pair(l);
        store_rows(a, rows, lane, own, l > 0.f ? fast_exp2(top - m_top) / l : 0.f, merge.store_region(), nullptr,
                   32 * Merge::kOwn * kg);
    } else {
        const float l = sum_over_row_pair(l_run);
        const float inv = l > 0.f ? fast_exp2(e_ref - m_run) / l : 0.f;
        store_rows(a, rows, lane, acc, inv, lds + row_block * store_region_bytes(4));
    }
}

template <int SB, int W, bool MB, int KS = 1>
static void launch(const AttnArgs& a, int grid, hipStream_t st) {
    attn_bf16_kernel<SB, W, MB, KS><<<grid, KS * W * 64, 0, st>>>(a);
}

void launch_attn_bf16(const AttnArgs& a, int grid, hipStream_t st) {
    const Geom& g = a.g;
    const bool four = query_waves(g) == 4;
    switch (g.BS == 128 ? 4 : g.KBS) {
        case 4:
            if (g.KB > 1) {
                if (a.waves == 2)          launch<4, 2, true, 2>(a, grid, st);
                else if (split_keys(a, 2)) launch<4, 4, true, 2>(a, grid, st);
                else                  launch<4, 4, true>(a, grid, st);
            } else {
                if (a.waves == 2)          launch<4, 2, false, 2>(a, grid, st);
                else if (split_keys(a, 2)) launch<4, 4, false, 2>(a, grid, st);
                else                  launch<4, 4, false>(a, grid, st);
            }
            break;
        case 3:
            if (g.NS == 1) {
                if (split_keys(a, 2)) launch<3, 3, false, 2>(a, grid, st);
                else                  launch<3, 3, false>(a, grid, st);
            } else if (four) {
                launch<3, 4, true>(a, grid, st);
            } else {
                launch<3, 3, true>(a, grid, st);
            }
            break;
        case 2:
            if (g.NS == 1) {
                if (split_keys(a, 4)) launch<2, 2, false, 4>(a, grid, st);
                else                  launch<2, 2, false>(a, grid, st);
            } else if (four) {
                launch<2, 4, true>(a, grid, st);
            } else {
                launch<2, 2, true>(a, grid, st);
            }
            break;
        default:
            if (g.NS == 1) {
                if (split_keys(a, 4)) launch<1, 1, false, 4>(a, grid, st);
                else                  launch<1, 1, false>(a, grid, st);
            } else if (four) {
                launch<1, 4, true>(a, grid, st);
            } else {
                launch<1, 1, true>(a, grid, st);
            }
            break;
    }
}

}  // namespace fps
