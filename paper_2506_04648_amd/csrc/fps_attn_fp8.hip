// FP8 attention kernel: K Q^T and V^T P^T on v_mfma_f32_32x32x64_f8f6f4.
//
// Software-pipelined inside each wave, because a wave whose next instruction is an MFMA holds the vector
// issue port while the matrix pipe is busy: MFMA and VALU work overlap well only when they alternate
// within one instruction stream.  Per key block i:
//   P(i) = 2^(S'(i) - m), FP8 pack (VALU)  interleaved with  S(i+1) = K(i+1) Q^T              (MFMA)
//   row maxima of S(i+1) (VALU)            interleaved with  O += s^V 2^(m - m_base) V^T P^T (i) (MFMA)
// so the QK product of a block runs one iteration early; a score sub-block's registers are refilled as
// soon as its exponentials are taken.  K(i+2) and V(i+1) stream into LDS meanwhile; one barrier per
// iteration.  The 32x32x64 shape rather than 16x16x128: what an MFMA costs the vector instructions
// around it is largely per instruction (measured with fps_debug_issue_mix: beside 32 vector
// instructions one 32x32x64 adds 30 clocks, two 16x16x128 add 49).
//
// Per-tile V scales: O and l are kept relative to a FIXED reference m_base (that of the item's first
// block) and each block's contribution is weighted by 2^(m - m_base) >= 1 instead -- the weight rides in
// the multiplier of the fma that applies s^V anyway, so a moving row reference costs nothing
// (rescaling O costs 64 multiplications per wave whenever ANY of its 32 rows moves, which is two
// tiles in three).  Powers of two commute with fp32 rounding: same results.
// VCH: V carries one scale per channel (the paper's variant) instead of one per tile; the PV MFMA
// then accumulates straight into O and the scales are applied once in the epilogue.
// P: key blocks (small scale groups) that one step of the pipeline takes, each with scales and a row reference of its own:
// as many of SB sub-blocks as fill four, so that the barriers and the bookkeeping of a step serve two or four blocks.  K and
// V of a step are double-buffered where a workgroup has four waves of rows; with less LDS a wave than that, K(i+2) and V(i) each
// stream into the one buffer while the other product runs, two barriers a step.  Attention on 21x30x52 tokens, one block a
// step against P, us: 24 heads, 64-token sub-tiles of (2,8,16) tiles, window 3x3x3, 1278 -> 1220; 12 heads, 16-token
// sub-tiles of (2,4,8) tiles, that window, 872 -> 745; tile (3,4,4), window 3x5x7, 783 -> 763, tile (2,4,4) 508 -> 495 and
// (2,8,4), window 3x3x5, 326 -> 324.
#include "fps_attn_device.h"

namespace fps {

template <int SB, int W, bool VCH, bool MB, int KS, int P>
__global__ __launch_bounds__(KS * W * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_fp8_kernel(AttnArgs a) {
    load_arguments<(sizeof(AttnArgs) + 63) / 64>();
    constexpr int NTHR = KS * W * 64;
    constexpr int CPT = SB * 4 / W;                        // 16-byte chunks per thread per operand block
    constexpr int BLOCK_BYTES = SB * 4096, STEP_BYTES = P * BLOCK_BYTES;
    static_assert(CPT >= 1 && CPT * W == SB * 4, "every wave copies the same share of a block");
    static_assert(KS == 1 || P == 1, "wave groups take single blocks");
    static_assert(P * SB <= 4, "scores of a step: at most 4 sub-blocks");
    // two buffers each for K and V where that leaves room for 8 waves on a CU, otherwise one
    constexpr bool TWO = P * SB <= W;
    constexpr int VBUF = TWO ? 2 : 1;                      // V's (first) buffer
    constexpr int GROUP_BYTES = 2 * VBUF * STEP_BYTES;     // K even, K odd, V even, V odd; or K, V
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

    const uint8_t* const k_head = a.k + tile0 * TSB * 4096;
    const uint8_t* const v_head = a.v + tile0 * TSB * 4096;
    const float* const sk_head = a.sk + tile0 * NS;
    const float* const sv_head = a.sv + tile0 * NS;
    // the key blocks of a step: of a list of `count`, those from P * step on; past the end the last one again
    // (its weights are then made zero)
    struct Step { KeyBlock b[P]; };
    typedef BlockList<MB, KS> List;
    auto step_blocks = [&](const List& list, int count, int step) FPS_INLINE {
        Step st;
#pragma unroll
        for (int g = 0; g < P; ++g) st.b[g] = list.block(P == 1 ? step : min(P * step + g, count - 1));
        return st;
    };
    // copy c of the wave's share of the step's blocks, up to four chunks at once: one chunk a pipeline step takes 0.5 to 1 %
    // longer (narrow items in two groups, one workgroup a CU, 28.5 against 27.4 us)
    constexpr int COPIES = P * ((CPT + 3) / 4);
    auto stage_copy = [&](int buf, const uint8_t* head, const Step& st, int c) FPS_INLINE {
        const int g = c / (COPIES / P);
        const uint8_t* const src = head + (size_t)st.b[g].blk * BLOCK_BYTES + wave_s * (CPT * 1024);
        const uint32_t dst = lds_base + buf * STEP_BYTES + g * BLOCK_BYTES + wave_s * (CPT * 1024);
        dma_copy<CPT>(c % (COPIES / P), src, lane * 16, dst);
    };
    auto stage = [&](int buf, const uint8_t* head, const Step& st) FPS_INLINE {
#pragma unroll
        for (int c = 0; c < COPIES; ++c) stage_copy(buf, head, st, c);
    };
    auto lds_block = [&](int buf) FPS_INLINE { return lds + kg * GROUP_BYTES + buf * STEP_BYTES; };
    auto landed = []() FPS_INLINE { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
    int par = 0;                                           // TWO: parity of the current step's K and V buffers
    auto k_buf = [&](int ahead) FPS_INLINE { return TWO ? par ^ ahead : 0; };
    auto v_buf = [&](int ahead) FPS_INLINE { return VBUF + (TWO ? par ^ ahead : 0); };

    // Of a list of `total` blocks, those of this wave group.  Group 0 never has fewer than another; what a group
    // has fewer barriers than group 0 (one a block, one a list; with one buffer two and three) it makes up for at the end,
    // as every barrier is one of the whole workgroup.  (Made up for within the list, they cost 110 spilled registers.)
    int owed = 0;
    auto blocks_of_group = [&](int total) FPS_INLINE {
        if (KS == 1) return total;
        const int nblk = (total - kg + KS - 1) / KS;
        owed += (TWO ? 1 : 2) * ((total + KS - 1) / KS - nblk) + (nblk == 0 ? (TWO ? 1 : 3) : 0);
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
            const int count = blocks_of_group(list.total());
            if (count == 0) continue;
            const int steps = (count + P - 1) / P;
            list.fill(0);
            Step cur = step_blocks(list, count, 0), nxt = cur;
            if (steps > 1) nxt = step_blocks(list, count, 1);
            stage(k_buf(0), k_head, cur);
            if (TWO) {
                stage(v_buf(0), v_head, cur);
                if (steps > 1) stage(k_buf(1), k_head, nxt);
            } else {
                landed();
                __syncthreads();                           // K(0) visible
                __syncthreads();                           // QK(0) done
                if (steps > 1) stage(k_buf(0), k_head, nxt);
            }
            landed();
            __syncthreads();
            for (int i = 0; i + 1 < steps; ++i) {
                if (TWO) {
                    __syncthreads();
                } else {
                    stage(v_buf(0), v_head, cur);
                    landed();
                    __syncthreads();                       // QK(i+1) done; V(i) visible
                }
                cur = nxt;
                if (i + 2 < steps) {
                    if (((P * (i + 2)) & 63) == 0) list.fill(P * (i + 2));
                    nxt = step_blocks(list, count, i + 2);
                    stage(k_buf(0), k_head, nxt);
                }
                if (TWO) stage(v_buf(1), v_head, cur);
                landed();
                if (!TWO) __syncthreads();                 // PV(i) done; K(i+2) visible
                par ^= 1;
            }
            if (!TWO) {
                stage(v_buf(0), v_head, cur);
                landed();
                __syncthreads();
            }
            __syncthreads();
            par ^= 1;
        }
        make_up();
        if (TWO) __syncthreads();
        if (KS > 1) __syncthreads();
        return;
    }

    v8i qop[2];                                            // Q^T, contraction steps 0 and 1
    float m_run = -INFINITY;
    float l_run = 0.f;                                     // running sum of 448 * P (this lane's keys)
    float m_base = 0.f;                                    // fixed reference: see above
    float w_owed = 0.f;                                    // weight of the fma owed to O's last channel block
    v16f acc[4];
    {
        const uint4* p = reinterpret_cast<const uint4*>(a.q + (((tile0 + u) * TSB + qs) * 32 + n) * 128 + 32 * h);
        qop[0] = make_v8i(p[0], p[1]);
        qop[1] = make_v8i(p[4], p[5]);
#pragma unroll
        for (int db = 0; db < 4; ++db) acc[db] = zero16();
    }
    const float sqc = load_uniform(a.sq, (tile0 + u) * NS + rows.group) * kLog2eOverSqrtD;

    auto pipeline = [&](auto nh_tag) FPS_INLINE {
        constexpr int NH = decltype(nh_tag)::value;        // 16-key halves of a block
        constexpr int NB = (NH + 1) / 2;                   // 32-key sub-blocks of a block
        constexpr int NT = P * NB;                         // and of a step: block kb / NB, its sub-block kb % NB
        constexpr int J = (NB + 1) / 2;                    // contraction steps of a block's PV product: two sub-blocks each,
        constexpr bool TAIL = NB % 2 != 0;                 // the last one of an odd number by itself
        constexpr int R = 4 * P;                           // PV products of 32 channels
        auto db_of = [](int r) { return VCH ? r % 4 : r / P; };        // channel block of product r,
        auto kb_of = [](int r) { return VCH ? r / 4 : r % P; };        // and key block of the step
        const uint32_t classes = G.nh_classes[NH - 1] & box.classes;
        if (!classes) return;
        List list(G, box, NH, classes, kg);
        const int count = blocks_of_group(list.total());
        if (count == 0) return;
        const int steps = (count + P - 1) / P;
        const bool odd = P > 1 && count < P * steps;       // the last step is not full
        list.fill(0);

        v16f s[NT];                                        // S^T, blocks of 32 keys
        v8i pb[P * J];                                     // P^T as packed E4M3, per contraction step
        v16f tq[2];                                        // raw V^T P^T of a product, until its fma
#pragma unroll
        for (int i = 0; i < P * J; ++i) pb[i] = v8i{0, 0, 0, 0, 0, 0, 0, 0};
        auto has_half = [](int t) { return 2 * ((t >> 1) % NB) + (t & 1) < NH; };   // half t & 1 of sub-block t >> 1
        // operand `step` of the staged blocks -- K: 32-key sub-block * 2 + contraction step; V: product * J +
        // contraction step (keys of sub-blocks 2j and 2j + 1)
        auto load_k = [&](const uint8_t* buf, int step) FPS_INLINE {
            const int kb = step >> 1, at = ((kb / NB * SB + kb % NB) * 4 + (step & 1) * 2) * 64;
            const uint4* b4 = reinterpret_cast<const uint4*>(buf);
            return make_v8i(b4[at + lane], b4[at + 64 + lane]);
        };
        auto load_v = [&](const uint8_t* buf, int step) FPS_INLINE {
            const int r = step / J, j = step % J, db = db_of(r), g = kb_of(r);
            const uint4* b4 = reinterpret_cast<const uint4*>(buf) + g * (BLOCK_BYTES / 16);
            const uint4 lo = b4[((2 * j + 0) * 4 + db) * 64 + lane];
            if (TAIL && j == J - 1) return make_v8i(lo, lo);           // only the lower half is used
            return make_v8i(lo, b4[((2 * j + 1) * 4 + db) * 64 + lane]);
        };
        auto qk_mfma = [&](const v8i& kop, int step) FPS_INLINE {
            const int kb = step >> 1, ks = step & 1;
            s[kb] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(kop, qop[ks], ks == 0 ? zero16() : s[kb],
                                                                   0, 0, 0, 0, 0, 0);
        };
        auto pv_mfma = [&](const v8i& vop, int step) FPS_INLINE {
            const int r = step / J, j = step % J, db = db_of(r);
            const v8i& pj = pb[kb_of(r) * J + j];
            v16f x = VCH ? acc[db] : j == 0 ? zero16() : tq[r & 1];
            if (TAIL && j == J - 1) {
                // a single sub-block: 32x32x16 instructions, 16 keys each.  They take 32.5 clocks against 64.9 of a
                // 32x32x64, so two halves cost what half of one would and a single half less.  A lane's 8
                // contraction slots of half e are the keys of its registers 8e .. 8e + 7
#pragma unroll
                for (int e = 0; e < (NH % 2 ? 1 : 2); ++e) {
                    const long va = (long)((uint64_t)(uint32_t)vop[2 * e] | ((uint64_t)(uint32_t)vop[2 * e + 1] << 32));
                    const long pa = (long)((uint64_t)(uint32_t)pj[2 * e] | ((uint64_t)(uint32_t)pj[2 * e + 1] << 32));
                    x = __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(va, pa, x, 0, 0, 0);
                }
            } else {
                x = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(vop, pj, x, 0, 0, 0, 0, 0, 0);
            }
            if (VCH) acc[db] = x; else tq[r & 1] = x;
        };
        // half `half` of O^T += w * raw product r, w = s^V 2^(m - m_base), pinned where it is written
        auto pv_accumulate_half = [&](int r, int half, float w) FPS_INLINE {
            if (VCH) return;
            const int db = db_of(r);
#pragma unroll
            for (int i = 8 * half; i < 8 * half + 8; ++i) acc[db][i] = __builtin_fmaf(tq[r & 1][i], w, acc[db][i]);
            asm volatile("" : "+v"(acc[db]));
        };
        auto pv_accumulate = [&](int r, float w) FPS_INLINE { pv_accumulate_half(r, 0, w); pv_accumulate_half(r, 1, w); };
        // row maximum of half `e` of score block kb
        auto max_half = [&](float mx, int kb, int e) FPS_INLINE {
#pragma unroll
            for (int r = 8 * e; r < 8 * e + 8; r += 2)
                mx = __builtin_fmaxf(__builtin_fmaxf(mx, s[kb][r]), s[kb][r + 1]);
            asm volatile("" : "+v"(mx));
            return mx;
        };
        // the first half of a block's row maximum starts it
        auto max_of_half = [&](float (&mx)[P], int t) FPS_INLINE {
            if (has_half(t)) mx[t / (2 * NB)] = max_half(t % (2 * NB) == 0 ? -INFINITY : mx[t / (2 * NB)], t >> 1, t & 1);
        };
        // of the step's blocks: log2(448) less the reference; the reference's weight, relative to m_base, or (VCH) the
        // rescale that it owes to what is added up so far
        float cm[P], rel[P];
        // the weights of half `e` of score block kb and their FP8 codes
        auto weights_half = [&](int kb, int e, float sc, float c, float& rs) FPS_INLINE {
            v8i& pj = pb[kb / NB * J + kb % NB / 2];
            const int at = 4 * (kb % NB % 2) + 2 * e;
#pragma unroll
            for (int q2 = 0; q2 < 2; ++q2) {
                float p[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    p[r] = fast_exp2(__builtin_fmaf(s[kb][8 * e + 4 * q2 + r], sc, c));
                    rs += p[r];
                }
                int pw = pj[at + q2];
                pw = __builtin_amdgcn_cvt_pk_fp8_f32(p[0], p[1], pw, false);
                pw = __builtin_amdgcn_cvt_pk_fp8_f32(p[2], p[3], pw, true);
                asm volatile("" : "+v"(pw), "+v"(rs));     // keep the pass where it is written
                pj[at + q2] = pw;
            }
        };
        auto mask_blocks = [&](const int (&nn)[P]) FPS_INLINE {
#pragma unroll
            for (int g = 0; g < P; ++g)
                if (nn[g] < 16 * NH) mask_cut_half(s[g * NB + NB - 1], (NH - 1) & 1, nn[g] - 16 * (NH - 1), h);
        };
        // the row references of the step's blocks, whose row maxima mx (not scaled) were taken: each block has its own, since
        // one shared by the step would take bits of the weights, and V's scales may make up for small weights
        auto new_references = [&](const float (&mx)[P], const float (&sc)[P]) FPS_INLINE {
            const bool first = m_run == -INFINITY;         // the item's first step
            float m[P];
#pragma unroll
            for (int g = 0; g < P; ++g) {
                const float m_old = g == 0 ? m_run : m[g - 1];
                m[g] = __builtin_fmaxf(m_old, __builtin_ceilf(max_over_row_pair(mx[g]) * sc[g]));
                if (!VCH && g == 0) m_base = first ? m[0] : m_base;
                rel[g] = fast_exp2(VCH ? m_old - m[g] : m[g] - m_base);
                cm[g] = kLog2Of448 - m[g];                 // 448 * 2^(S' - m) = 2^(S' + (log2(448) - m))
            }
            m_run = m[P - 1];
            if (!VCH && __any(m_run - m_base > kMaxDrift)) {
                const float down = fast_exp2(m_base - m_run);
#pragma unroll
                for (int db = 0; db < 4; ++db) acc[db] *= down;
                l_run *= down;
                w_owed *= down;            // the last product's fma is still owed
                m_base = m_run;
#pragma unroll
                for (int g = 0; g < P; ++g) rel[g] = fast_exp2(m[g] - m_run);
            }
        };
        auto load_scales = [&](const Step& st, float (&sc)[P], float (&sv)[P]) FPS_INLINE {
#pragma unroll
            for (int g = 0; g < P; ++g) {
                sc[g] = sqc * load_uniform(sk_head, st.b[g].group);
                sv[g] = VCH ? 1.f : load_uniform(sv_head, st.b[g].group);
            }
        };
        // block g's share of the row sums, and the rescale that O owes it (VCH)
        auto add_row_sum = [&](int g, float rs) FPS_INLINE {
            if (VCH) l_run = l_run * rel[g] + rs;
            else     l_run = __builtin_fmaf(rs, rel[g], l_run);
        };
        auto rescale = [&](int g) FPS_INLINE {
            if (VCH && __any(rel[g] != 1.0f)) {
#pragma unroll
                for (int db = 0; db < 4; ++db) acc[db] *= rel[g];
            }
        };

        // prologue: K(0), V(0), K(1) staged; S(0) and its row reference
        Step cur = step_blocks(list, count, 0), nxt = cur;
        if (steps > 1) nxt = step_blocks(list, count, 1);
        float sc[P], svv[P], mx[P];
        int n_cut[P];
#pragma unroll
        for (int g = 0; g < P; ++g) n_cut[g] = cur.b[g].n;
        stage(k_buf(0), k_head, cur);
        if (TWO) stage(v_buf(0), v_head, cur);
        load_scales(cur, sc, svv);
        if (TWO && steps > 1) stage(k_buf(1), k_head, nxt);
        landed();
        __syncthreads();
#pragma unroll
        for (int step = 0; step < 2 * NT; ++step) qk_mfma(load_k(lds_block(k_buf(0)), step), step);
        if (!TWO) {
            __syncthreads();                               // every wave is past QK(0)
            if (steps > 1) stage(k_buf(0), k_head, nxt);
        }
        mask_blocks(n_cut);
#pragma unroll
        for (int t = 0; t < 2 * NT; ++t) max_of_half(mx, t);
        w_owed = 0.f;
        new_references(mx, sc);
        if (!VCH) tq[(R - 1) & 1] = zero16();
        if (!TWO) {
            landed();
            __syncthreads();                               // K(1) visible
        }

        // iteration i: P(i) | S(i+1) = K(i+1) Q^T, then row maximum of S(i+1) | O += s^V (V^T P^T)(i)
        for (int i = 0; i + 1 < steps; ++i) {
            const uint8_t* knxt = lds_block(k_buf(1));           // K(i+1)
            const uint8_t* vcur = lds_block(v_buf(0));           // V(i)
            if (TWO) __syncthreads();    // every wave is past QK(i) and PV(i-1); staged blocks are visible
            v8i op[3];                   // MFMA operands on their way from LDS, two steps ahead
            constexpr int PV0 = TWO ? 2 * NT : 0;                // place in the ring of PV's first
            op[0] = load_k(knxt, 0);
            op[1] = load_k(knxt, 1);
#pragma unroll
            for (int g = 0; g < P; ++g) n_cut[g] = nxt.b[g].n;
            const Step v_step = TWO ? nxt : cur;                 // V(i+1), or V(i)
            float sc_next[P], sv_next[P];
            load_scales(nxt, sc_next, sv_next);
            cur = nxt;
            // TWO: past the walk's end the last K is copied once more, into the buffer that nobody reads again, while V(i+1) is
            // on its way too.  With these copies under a condition, which cuts the steps below into pieces, 480p took 303, now
            // 299 us, and 720p 3.85, now 3.78 ms.
            if (i + 2 < steps) {
                // Once in 64 blocks.  Said so only where the compiler put this code in the middle of the loop otherwise: per-channel
                // V, tiles of several blocks; 2 heads of 9x20x34 tokens, tile (4,16,16), window 5x3x3, 79.7 -> 74.7 us, launches
                // of 400 items and more 0.992.  Told the same, per-tile V takes up to 1 % more on 480p and 720p, small groups 1 %.
                const bool refill = ((P * (i + 2)) & 63) == 0;
                if (SB == 4 && VCH && MB && KS == 1 ? __builtin_expect(refill, false) : refill) list.fill(P * (i + 2));
                nxt = step_blocks(list, count, i + 2);
            }

            // ---- P(i) and its FP8 codes  |  QK(i+1) ------------------------------------------
            // step t: the exponentials of half a score block (block t/2, registers 8(t%2)..+7); the
            // MFMAs that refill a block follow one block behind, so steps 0, 1 have none (they take
            // the fma still owed to the last product of PV(i-1)) and the last two nothing else
            float rs[P];
#pragma unroll
            for (int g = 0; g < P; ++g) rs[g] = 0.f;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 2 * NT + 2; ++t) {
                if (t >= 2) {
                    if (t < 2 * NT) op[t % 3] = load_k(knxt, t);       // operand of step t + 2
                    else if (TWO)   op[t % 3] = load_v(vcur, t - 2 * NT);        // V(i) is there already: PV's first two
                    qk_mfma(op[(t - 2) % 3], t - 2);
                }
                if (t < 2) pv_accumulate_half(R - 1, t, w_owed);       // PV(i-1)'s last product
                if (t < 2 * NT && has_half(t)) {
                    const int g = t / (2 * NB);
                    weights_half(t >> 1, t & 1, sc[g], cm[g], rs[g]);
                }
                // from the first step on, one a step.  (In items of 32 and 64 rows, whose waves have four and two of them, every other
                // step, two from step 2 on: 1.004 of the time over 123 calls, 0.97 to 1.05, by kernel 1.002 to 1.008; 225 items of
                // 128 rows 28.9 against 28.8 us, 120 the same.)
                constexpr int per = (COPIES + 2 * NT + 1) / (2 * NT + 2);
#pragma unroll
                for (int c = t * per; c < (t + 1) * per && c < COPIES; ++c) {
                    if (TWO) stage_copy(k_buf(0), k_head, nxt, c);         // K(i) was consumed last iteration
                    else     stage_copy(v_buf(0), v_head, v_step, c);      // V(i-1) was consumed
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            float wg[P];                                         // weights of the step's products
#pragma unroll
            for (int g = 0; g < P; ++g) {
                add_row_sum(g, rs[g]);
                wg[g] = svv[g] * rel[g];
                sc[g] = sc_next[g];
                svv[g] = sv_next[g];
            }
            w_owed = wg[P - 1];
            if (!TWO) {
                landed();
                __syncthreads();         // every wave is past QK(i+1); V(i) is visible
            }
            if (!TWO) {
                op[0] = load_v(vcur, 0);
                op[1] = load_v(vcur, 1);
            }
            mask_blocks(n_cut);
            rescale(0);

            // ---- row maximum of S(i+1)  |  PV(i) ---------------------------------------------
            // step k: the MFMA of product k/J, contraction step k%J, 16-key halves of the row
            // maximum, and the fma of a product whose last MFMA was issued two or three steps
            // earlier (a 16-pass result may be read 18 issue slots after its instruction)
            constexpr int STEPS = R * J, HPS = (2 * NT + STEPS - 1) / STEPS;
#pragma unroll
            for (int k = 0; k < STEPS; ++k) {
                if (k + 2 < STEPS) op[(PV0 + k + 2) % 3] = load_v(vcur, k + 2);
                if (J == 2) {                              // before tq[..] is refilled
                    if (k >= 3) pv_accumulate_half((k - 3) >> 1, (k - 3) & 1, wg[((k - 3) >> 1) % P]);
                } else if (k >= 2) {
                    pv_accumulate(k - 2, wg[(k - 2) % P]);
                }
                if (VCH && k > 0 && k % (4 * J) == 0) rescale(k / (4 * J));
                pv_mfma(op[(PV0 + k) % 3], k);
#pragma unroll
                for (int t = k * HPS; t < (k + 1) * HPS && t < 2 * NT; ++t) max_of_half(mx, t);
                constexpr int per = (COPIES + STEPS - 1) / STEPS;
#pragma unroll
                for (int c = k * per; c < (k + 1) * per && c < COPIES; ++c) {
                    if (TWO) stage_copy(v_buf(1), v_head, v_step, c);          // V(i-1) was consumed last iteration
                    // K(i+1) was consumed.  With one buffer each the condition stays: without it 30 calls of tiles of 32 and 48 tokens
                    // and of one-wave items took 1.005 of the time (0.98 to 1.04; tile (3,4,4), window 3x5x7, 760 -> 750 us, window
                    // 3x3x3 257 -> 260, 63 items of 128 rows 26.2 -> 27.3)
                    else if (i + 2 < steps) stage_copy(k_buf(0), k_head, nxt, c);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if (J == 1) pv_accumulate_half(R - 2, 0, wg[(R - 2) % P]);
            pv_accumulate_half(R - 2, 1, wg[(R - 2) % P]);
            new_references(mx, sc);
            landed();                    // this thread's share of the staged blocks
            if (!TWO) __syncthreads();   // every wave is past PV(i); K(i+2) is visible
            par ^= 1;
        }

        // the last step's P and PV
        if (TWO) __syncthreads();
        else     stage(v_buf(0), v_head, cur);
        if (!VCH) pv_accumulate(R - 1, w_owed);
        float rs = 0.f;
#pragma unroll
        for (int t = 0; t < 2 * NT; ++t) {
            const int g = t / (2 * NB);
            // a block past the end has no weights
            const float c = g > 0 && odd && count <= P * (steps - 1) + g ? -INFINITY : cm[g];
            if (has_half(t)) weights_half(t >> 1, t & 1, sc[g], c, rs);
            if (t % (2 * NB) == 2 * NB - 1) {
                add_row_sum(g, rs);
                rs = 0.f;
            }
        }
        rescale(0);
        if (!TWO) {
            landed();
            __syncthreads();
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
            for (int j = 0; j < J; ++j) {
                if (j == 0 && r > 0 && r % 4 == 0) rescale(r / 4);
                pv_mfma(load_v(lds_block(v_buf(0)), r * J + j), r * J + j);
            }
            if (r > 0) pv_accumulate(r - 1, svv[kb_of(r - 1)] * rel[kb_of(r - 1)]);
        }
        pv_accumulate(R - 1, svv[P - 1] * rel[P - 1]);
        if (!TWO) __syncthreads();                         // both buffers are free
        par ^= 1;
    };
    if constexpr (SB > 3) { pipeline(Count<8>{}); pipeline(Count<7>{}); }
    if constexpr (SB > 2) { pipeline(Count<6>{}); pipeline(Count<5>{}); }
    if constexpr (SB > 1) { pipeline(Count<4>{}); pipeline(Count<3>{}); }
    pipeline(Count<2>{});
    pipeline(Count<1>{});

    make_up();
    if (TWO) __syncthreads();                              // all waves are done with the staged tiles
    const float* const ch_scale = VCH ? a.sv + (size_t)bh * 128 : nullptr;
    // l carries the factor 448
    auto inverse = [](float l) FPS_INLINE { l = sum_over_row_pair(l); return l > 0.f ? 1.0f / l : 0.f; };
    if constexpr (KS > 1) {
        // O and l of a group are relative to its reference, a power of two: moving them to the largest is exact
        typedef SplitMerge<W, KS> Merge;
        const Merge merge{lds, row_block, kg, lane};
        // -inf: the group had no block, all zero
        merge.leave(acc, VCH || m_run == -INFINITY ? m_run : m_base, l_run);
        __syncthreads();
        v4f o[KS];
        float top = -INFINITY, l = 0.f, factor[KS];
#pragma unroll
        for (int g = 0; g < KS; ++g) {
            o[g] = merge.numbers(g);
            top = __builtin_fmaxf(top, o[g][0]);           // finite: group 0 has a block
        }
#pragma unroll
        for (int g = 0; g < KS; ++g) {
            factor[g] = fast_exp2(o[g][0] - top);
            l = __builtin_fmaf(o[g][1], factor[g], l);
        }
        v16f own[Merge::kOwn];
        merge.add(acc, factor, own);
        store_rows(a, rows, lane, own, inverse(l), merge.store_region(), ch_scale, 32 * Merge::kOwn * kg);
    } else {
        store_rows(a, rows, lane, acc, inverse(l_run), lds + row_block * store_region_bytes(4), ch_scale);
    }
}

template <int SB, int W, bool MB, int KS = 1, int P = 1>
static void launch(const AttnArgs& a, bool vch, int grid, hipStream_t st) {
    if (vch) attn_fp8_kernel<SB, W, true, MB, KS, P><<<grid, KS * W * 64, 0, st>>>(a);
    else     attn_fp8_kernel<SB, W, false, MB, KS, P><<<grid, KS * W * 64, 0, st>>>(a);
}

void launch_attn_fp8(const AttnArgs& a, bool vch, int grid, hipStream_t st) {
    const Geom& g = a.g;
    const bool four = query_waves(g) == 4, together = blocks_together(a);
    switch (g.BS == 128 ? 4 : g.KBS) {
        case 4:
            if (g.KB > 1) {
                if (a.waves == 1)          launch<4, 1, true, 4>(a, vch, grid, st);
                else if (narrow_in_four(a)) launch<4, 2, true, 4>(a, vch, grid, st);
                else if (a.waves == 2)     launch<4, 2, true, 2>(a, vch, grid, st);
                else if (split_keys(a, 2)) launch<4, 4, true, 2>(a, vch, grid, st);
                else                  launch<4, 4, true>(a, vch, grid, st);
            } else {
                if (a.waves == 1)          launch<4, 1, false, 4>(a, vch, grid, st);
                else if (narrow_in_four(a)) launch<4, 2, false, 4>(a, vch, grid, st);
                else if (a.waves == 2)     launch<4, 2, false, 2>(a, vch, grid, st);
                else if (split_keys(a, 2)) launch<4, 4, false, 2>(a, vch, grid, st);
                else                  launch<4, 4, false>(a, vch, grid, st);
            }
            break;
        case 3:
            if (g.NS == 1) {
                if (split_keys(a, 2)) launch<3, 3, false, 2>(a, vch, grid, st);
                else                  launch<3, 3, false>(a, vch, grid, st);
            } else if (four) {
                launch<3, 4, true>(a, vch, grid, st);
            } else {
                launch<3, 3, true>(a, vch, grid, st);
            }
            break;
        case 2:
            if (g.NS == 1) {
                if (split_keys(a, 4)) launch<2, 2, false, 4>(a, vch, grid, st);
                else if (together)    launch<2, 2, false, 1, 2>(a, vch, grid, st);
                else                  launch<2, 2, false>(a, vch, grid, st);
            } else if (four) {
                if (together) launch<2, 4, true, 1, 2>(a, vch, grid, st);
                else          launch<2, 4, true>(a, vch, grid, st);
            } else if (together) {
                launch<2, 2, true, 1, 2>(a, vch, grid, st);
            } else {
                launch<2, 2, true>(a, vch, grid, st);
            }
            break;
        default:
            if (g.NS == 1) {
                if (split_keys(a, 4)) launch<1, 1, false, 4>(a, vch, grid, st);
                else if (together)    launch<1, 1, false, 1, 2>(a, vch, grid, st);
                else                  launch<1, 1, false>(a, vch, grid, st);
            } else if (four) {
                launch<1, 4, true, 1, 4>(a, vch, grid, st);
            } else if (together) {
                launch<1, 1, true, 1, 2>(a, vch, grid, st);
            } else {
                launch<1, 1, true>(a, vch, grid, st);
            }
            break;
    }
}

}  // namespace fps
