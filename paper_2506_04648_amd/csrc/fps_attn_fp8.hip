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
#include "fps_attn_device.h"

namespace fps {

template <int SB, int W, bool VCH, bool MB, int KS>
__global__ __launch_bounds__(KS * W * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
void attn_fp8_kernel(AttnArgs a) {
    constexpr int NTHR = KS * W * 64;
    constexpr int CPT = SB * 4 / W;                        // 16-byte chunks per thread per operand block
    constexpr int BLOCK_BYTES = SB * 4096;
    static_assert(CPT >= 1 && CPT <= 4 && CPT * W == SB * 4, "every wave copies the same share of a block");
    constexpr int GROUP_BYTES = 4 * BLOCK_BYTES;           // K even, K odd, V even, V odd
    constexpr int LDS_BYTES = KS * GROUP_BYTES > SplitMerge<W, KS>::kBytes ? KS * GROUP_BYTES : SplitMerge<W, KS>::kBytes;
    // the groups' blocks; afterwards their sums and the output transpose
    __shared__ __attribute__((aligned(16))) uint8_t lds[LDS_BYTES];
    const Geom& G = a.g;
    const int NS = MB ? G.NS : 1;
    const int KBG = MB && SB == 4 ? G.KBG : 1;             // key blocks of a scale group
    const int TSB = MB ? NS * KBG * SB : SB;               // sub-blocks of a tile
    int bh, u, jq;
    if (!work_item(a, &bh, &u, &jq)) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5, n = lane & 31;
    const int wave_s = __builtin_amdgcn_readfirstlane(wave) % W, kg = KS > 1 ? __builtin_amdgcn_readfirstlane(wave) / W : 0;
    const int ut = quotient(u, G.nW * G.nH, G.rc_layer), urem = u - ut * (G.nW * G.nH);
    const int uh = quotient(urem, G.nW, G.rc_row), uw = urem - uh * G.nW;
    const int ucls = tile_class(G, ut, uh, uw);
    // the wave's sub-block of query rows; rotated from tile to tile (and wave group to wave group) so that the idle
    // waves of cut tiles fall on different SIMDs
    const int row_block = W == 4 ? (wave_s + kg + u) & 3 : wave_s;
    const int qs = jq * W + row_block;
    QueryRows rows;
    rows.init(G, bh, u, ucls, ut, uh, uw, qs, KBG * SB);
    zero_padding_rows(a, rows, ucls, lane);
    if (!any_real_row<SB, W, MB>(G, ucls, jq, KBG * SB)) return;
    const size_t tile0 = (size_t)bh * G.M;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(&lds[0]) + kg * GROUP_BYTES;
    KeyBox box;
    box.init(a, ut, uh, uw);
    if (a.visited && bh == 0 && jq == 0) box.mark(G, a.visited + (size_t)u * G.M, NTHR);

    const uint8_t* const k_head = a.k + tile0 * TSB * 4096;
    const uint8_t* const v_head = a.v + tile0 * TSB * 4096;
    const float* const sk_head = a.sk + tile0 * NS;
    const float* const sv_head = a.sv + tile0 * NS;
    auto k_blk = [&](const KeyBlock& b) FPS_INLINE { return k_head + (size_t)b.blk * BLOCK_BYTES; };
    auto v_blk = [&](const KeyBlock& b) FPS_INLINE { return v_head + (size_t)b.blk * BLOCK_BYTES; };
    auto stage_chunk = [&](int buf, const uint8_t* src, int c) FPS_INLINE {
        dma_chunk_of(c, src + wave_s * (CPT * 1024), lane * 16, lds_base + buf * BLOCK_BYTES + wave_s * (CPT * 1024));
    };
    auto stage = [&](int buf, const uint8_t* src) FPS_INLINE {
#pragma unroll
        for (int c = 0; c < CPT; ++c) stage_chunk(buf, src, c);
    };
    auto lds_block = [&](int buf) FPS_INLINE { return lds + kg * GROUP_BYTES + buf * BLOCK_BYTES; };
    int par = 0;                                           // parity of the current block's K and V buffers

    // Of a walk of `total` blocks, those of this wave group.  Group 0 never has fewer than another; what a group
    // has fewer barriers than group 0 (one a block, one a walk) it makes up for at the end, as every barrier
    // is one of the whole workgroup.  (Made up for within the walk, they cost 110 spilled registers.)
    int owed = 0;
    auto blocks_of_group = [&](int total) FPS_INLINE {
        if (KS == 1) return total;
        const int nblk = (total - kg + KS - 1) / KS;
        owed += 1 * ((total + KS - 1) / KS - nblk) + (nblk == 0 ? 1 : 0);
        return nblk;
    };
    auto make_up = [&]() FPS_INLINE {
        if (KS > 1)
            for (; owed > 0; --owed) __syncthreads();
    };

    if (rows.rows <= 0) {
        // no real row: this wave only copies its share of the K and V blocks, barrier for barrier
        for (int nh = 2 * SB; nh >= 1; --nh) {
            const uint32_t classes = G.nh_classes[nh - 1] & box.classes;
            if (!classes) continue;
            BlockWalk<MB> walk(G, box, nh);
            const int total = walk.begin(classes);
            const int nblk = blocks_of_group(total);
            if (nblk == 0) continue;
            walk.skip(kg);
            KeyBlock nxt = walk.block();
            stage(par, k_blk(nxt));
            stage(2 + par, v_blk(nxt));
            if (nblk > 1) {
                walk.skip(KS);
                nxt = walk.block();
                stage(par ^ 1, k_blk(nxt));
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            for (int i = 0; i + 1 < nblk; ++i) {
                __syncthreads();
                const KeyBlock v_next = nxt;
                if (i + 2 < nblk) {
                    walk.skip(KS);
                    nxt = walk.block();
                    stage(par, k_blk(nxt));
                }
                stage(2 + (par ^ 1), v_blk(v_next));
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                par ^= 1;
            }
            __syncthreads();
            par ^= 1;
        }
        make_up();
        __syncthreads();
        if (KS > 1) __syncthreads();
        return;
    }

    v8i qop[2];                                            // Q^T, contraction steps 0 and 1
    float m_run = -INFINITY;
    float l_run = 0.f;                                     // running sum of 448 * P (this lane's keys)
    float alpha = 1.f;                                     // VCH: rescale owed to O before the delayed PV
    float m_base = 0.f, w_cur = 1.f, w_prev = 0.f;         // fixed reference and weights: see above
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
        constexpr int NH = decltype(nh_tag)::value;        // 16-key halves
        constexpr int NB = (NH + 1) / 2;                   // 32-key sub-blocks
        constexpr int J = (NB + 1) / 2;                    // contraction steps of the PV product: two sub-blocks each,
        constexpr bool TAIL = NB % 2 != 0;                 // the last one of an odd number by itself
        const uint32_t classes = G.nh_classes[NH - 1] & box.classes;
        if (!classes) return;
        BlockWalk<MB> walk(G, box, NH);
        const int total = walk.begin(classes);
        const int nblk = blocks_of_group(total);
        if (nblk == 0) return;
        walk.skip(kg);

        v16f s[NB];                                        // S^T, blocks of 32 keys
        v8i pb[2];                                         // P^T as packed E4M3: contraction steps 0 and 1
        v16f tq[2];                                        // raw V^T P^T of a channel block, until its fma
        pb[0] = v8i{0, 0, 0, 0, 0, 0, 0, 0};
        pb[1] = pb[0];
        // operand `step` of a staged block -- K: 32-key sub-block * 2 + contraction step; V: 32-channel
        // block * J + contraction step (keys of sub-blocks 2j and 2j + 1)
        auto load_k = [&](const uint8_t* buf, int step) FPS_INLINE {
            const uint4* b4 = reinterpret_cast<const uint4*>(buf);
            return make_v8i(b4[(step * 2 + 0) * 64 + lane], b4[(step * 2 + 1) * 64 + lane]);
        };
        auto load_v = [&](const uint8_t* buf, int step) FPS_INLINE {
            const int db = step / J, j = step % J;
            const uint4* b4 = reinterpret_cast<const uint4*>(buf);
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
            const int db = step / J, j = step % J;
            v16f r = VCH ? acc[db] : j == 0 ? zero16() : tq[db & 1];
            if (TAIL && j == J - 1) {
                // a single sub-block: 32x32x16 instructions, 16 keys each.  They take 32.5 clocks against 64.9 of a
                // 32x32x64, so two halves cost what half of one would and a single half less.  A lane's 8
                // contraction slots of half e are the keys of its registers 8e .. 8e + 7
#pragma unroll
                for (int e = 0; e < (NH % 2 ? 1 : 2); ++e) {
                    const long va = (long)((uint64_t)(uint32_t)vop[2 * e] | ((uint64_t)(uint32_t)vop[2 * e + 1] << 32));
                    const long pa = (long)((uint64_t)(uint32_t)pb[j][2 * e] | ((uint64_t)(uint32_t)pb[j][2 * e + 1] << 32));
                    r = __builtin_amdgcn_mfma_f32_32x32x16_fp8_fp8(va, pa, r, 0, 0, 0);
                }
            } else {
                r = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(vop, pb[j], r, 0, 0, 0, 0, 0, 0);
            }
            if (VCH) acc[db] = r; else tq[db & 1] = r;
        };
        // half `half` of O^T(db) += s^V 2^(m - m_base) * raw, pinned where it is written
        auto pv_accumulate_half = [&](int db, int half) FPS_INLINE {
            if (VCH) return;
#pragma unroll
            for (int r = 8 * half; r < 8 * half + 8; ++r) acc[db][r] = __builtin_fmaf(tq[db & 1][r], w_prev, acc[db][r]);
            asm volatile("" : "+v"(acc[db]));
        };
        // row maximum of half `e` of score block kb
        auto max_half = [&](float mx, int kb, int e) FPS_INLINE {
#pragma unroll
            for (int r = 8 * e; r < 8 * e + 8; r += 2)
                mx = __builtin_fmaxf(__builtin_fmaxf(mx, s[kb][r]), s[kb][r + 1]);
            asm volatile("" : "+v"(mx));
            return mx;
        };
        float cm = 0.f;
        // the weights of half `e` of score block kb and their FP8 codes
        auto weights_half = [&](int kb, int e, float sc, float& rs) FPS_INLINE {
#pragma unroll
            for (int q2 = 0; q2 < 2; ++q2) {
                float p[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    p[r] = fast_exp2(__builtin_fmaf(s[kb][8 * e + 4 * q2 + r], sc, cm));
                    rs += p[r];
                }
                int pw = pb[kb >> 1][4 * (kb & 1) + 2 * e + q2];
                pw = __builtin_amdgcn_cvt_pk_fp8_f32(p[0], p[1], pw, false);
                pw = __builtin_amdgcn_cvt_pk_fp8_f32(p[2], p[3], pw, true);
                asm volatile("" : "+v"(pw), "+v"(rs));     // keep the pass where it is written
                pb[kb >> 1][4 * (kb & 1) + 2 * e + q2] = pw;
            }
        };
        // the row reference of the block whose row maximum mx was taken
        auto new_reference = [&](float mx, float sc) FPS_INLINE {
            mx = max_over_row_pair(mx);
            const float m_new = __builtin_fmaxf(m_run, __builtin_ceilf(mx * sc));
            if (VCH) {
                alpha = fast_exp2(m_run - m_new);
            } else {
                m_base = m_run == -INFINITY ? m_new : m_base;          // the item's first block
                w_cur = fast_exp2(m_new - m_base);
            }
            m_run = m_new;
            cm = kLog2Of448 - m_new;       // 448 * 2^(S' - m) = 2^(S' + (log2(448) - m))
            if (!VCH && __any(m_run - m_base > kMaxDrift)) {
                const float down = fast_exp2(m_base - m_run);
#pragma unroll
                for (int db = 0; db < 4; ++db) acc[db] *= down;
                l_run *= down;
                w_prev *= down;            // the last channel block's fma is still owed
                m_base = m_run;
                w_cur = 1.0f;
            }
        };

        // prologue: K(0), V(0), K(1) staged; S(0) and its row reference
        KeyBlock nxt = walk.block();
        const int n0 = nxt.n;
        stage(par, k_blk(nxt));
        stage(2 + par, v_blk(nxt));
        float sc = sqc * load_uniform(sk_head, nxt.group);
        float svv = VCH ? 1.f : load_uniform(sv_head, nxt.group);
        if (nblk > 1) {
            walk.skip(KS);
            nxt = walk.block();
            stage(par ^ 1, k_blk(nxt));
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
#pragma unroll
        for (int step = 0; step < 2 * NB; ++step) qk_mfma(load_k(lds_block(par), step), step);
        if (n0 < 16 * NH) mask_cut_half(s[NB - 1], (NH - 1) & 1, n0 - 16 * (NH - 1), h);
        {
            float mx = -INFINITY;
#pragma unroll
            for (int k = 0; k < NH; ++k) mx = max_half(mx, k >> 1, k & 1);
            w_prev = 0.f;
            new_reference(mx, sc);
        }
        if (!VCH) tq[1] = zero16();

        // iteration i: P(i) | S(i+1) = K(i+1) Q^T, then row maximum of S(i+1) | O += s^V (V^T P^T)(i)
        for (int i = 0; i + 1 < nblk; ++i) {
            const uint8_t* knxt = lds_block(par ^ 1);            // K(i+1)
            const uint8_t* vcur = lds_block(2 + par);            // V(i)
            __syncthreads();             // every wave is past QK(i) and PV(i-1); staged blocks are visible
            v8i op[3];                   // MFMA operands on their way from LDS, two steps ahead
            op[0] = load_k(knxt, 0);
            op[1] = load_k(knxt, 1);
            const int n_next = nxt.n;
            const uint8_t* vsrc = v_blk(nxt);
            const float sc_next = sqc * load_uniform(sk_head, nxt.group);
            const float sv_next = VCH ? 1.f : load_uniform(sv_head, nxt.group);
            const bool fetch_k = i + 2 < nblk;
            const uint8_t* ksrc = nullptr;
            if (fetch_k) {
                walk.skip(KS);
                nxt = walk.block();
                ksrc = k_blk(nxt);
            }

            // ---- P(i) and its FP8 codes  |  QK(i+1) ------------------------------------------
            // step t: the exponentials of half a score block (block t/2, registers 8(t%2)..+7); the
            // MFMAs that refill a block follow one block behind, so steps 0, 1 have none (they take
            // the fma still owed to the last channel block of PV(i-1)) and the last two nothing else
            float rs = 0.f;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 2 * NB + 2; ++t) {
                if (t >= 2) {
                    if (t < 2 * NB) op[t % 3] = load_k(knxt, t);       // operand of step t + 2
                    qk_mfma(op[(t - 2) % 3], t - 2);
                }
                if (t < 2) pv_accumulate_half(3, t);                   // PV(i-1)'s last block
                if (t < NH) weights_half(t >> 1, t & 1, sc, rs);
                if (t < CPT && fetch_k) stage_chunk(par, ksrc, t);     // K(i) was consumed last iteration
                __builtin_amdgcn_sched_barrier(0);
            }
            if (VCH) l_run = l_run * alpha + rs;
            else     l_run = __builtin_fmaf(rs, w_cur, l_run);
            w_prev = svv * w_cur;
            sc = sc_next;
            svv = sv_next;
            op[0] = load_v(vcur, 0);
            op[1] = load_v(vcur, 1);
            if (n_next < 16 * NH) mask_cut_half(s[NB - 1], (NH - 1) & 1, n_next - 16 * (NH - 1), h);
            if (VCH && __any(alpha != 1.0f)) {
#pragma unroll
                for (int db = 0; db < 4; ++db) acc[db] *= alpha;
            }

            // ---- row maximum of S(i+1)  |  PV(i) ---------------------------------------------
            // step k: the MFMA of channel block k/J, contraction step k%J, a 16-key half of the row
            // maximum, and the fma of a channel block whose last MFMA was issued two or three steps
            // earlier (a 16-pass result may be read 18 issue slots after its instruction)
            float mx = __builtin_fmaxf(__builtin_fmaxf(s[0][0], s[0][1]), __builtin_fmaxf(s[0][2], s[0][3]));
#pragma unroll
            for (int k = 0; k < 4 * J; ++k) {
                if (k + 2 < 4 * J) op[(k + 2) % 3] = load_v(vcur, k + 2);
                if (J == 2) {                              // before tq[..] is refilled
                    if (k >= 3) pv_accumulate_half((k - 3) >> 1, (k - 3) & 1);
                } else if (k >= 2) {
                    pv_accumulate_half(k - 2, 0);
                    pv_accumulate_half(k - 2, 1);
                }
                pv_mfma(op[k % 3], k);
                if (k < NH) {
                    if (k == 0) {
                        mx = __builtin_fmaxf(__builtin_fmaxf(mx, s[0][4]), s[0][5]);
                        mx = __builtin_fmaxf(__builtin_fmaxf(mx, s[0][6]), s[0][7]);
                        asm volatile("" : "+v"(mx));
                    } else {
                        mx = max_half(mx, k >> 1, k & 1);
                    }
                }
                if (k < CPT) stage_chunk(2 + (par ^ 1), vsrc, k);      // V(i-1) was consumed last iteration
                __builtin_amdgcn_sched_barrier(0);
            }
            if (J == 1) pv_accumulate_half(2, 0);
            pv_accumulate_half(2, 1);
            new_reference(mx, sc);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this thread's share of the staged blocks landed
            par ^= 1;
        }

        // the last block's P and PV
        __syncthreads();
        pv_accumulate_half(3, 0);
        pv_accumulate_half(3, 1);
        float rs = 0.f;
#pragma unroll
        for (int t = 0; t < NH; ++t) weights_half(t >> 1, t & 1, sc, rs);
        if (VCH) l_run = l_run * alpha + rs;
        else     l_run = __builtin_fmaf(rs, w_cur, l_run);
        w_prev = svv * w_cur;
        if (VCH && __any(alpha != 1.0f)) {
#pragma unroll
            for (int db = 0; db < 4; ++db) acc[db] *= alpha;
        }
#pragma unroll
        for (int db = 0; db < 4; ++db) {
#pragma unroll
            for (int j = 0; j < J; ++j) pv_mfma(load_v(lds_block(2 + par), db * J + j), db * J + j);
            if (db > 0) { pv_accumulate_half(db - 1, 0); pv_accumulate_half(db - 1, 1); }
        }
        pv_accumulate_half(3, 0);
        pv_accumulate_half(3, 1);
        par ^= 1;
    };
    if constexpr (SB > 3) { pipeline(Count<8>{}); pipeline(Count<7>{}); }
    if constexpr (SB > 2) { pipeline(Count<6>{}); pipeline(Count<5>{}); }
    if constexpr (SB > 1) { pipeline(Count<4>{}); pipeline(Count<3>{}); }
    pipeline(Count<2>{});
    pipeline(Count<1>{});

    make_up();
    __syncthreads();                                       // all waves are done with the staged tiles
    if constexpr (KS > 1) {
        // O and l of a group are relative to its reference, a power of two: moving them to the largest is exact
        const SplitMerge<W, KS> merge{lds, row_block, lane};
        float ref = VCH || m_run == -INFINITY ? m_run : m_base;        // -inf: the group had no block, all zero
        if (kg > 0) merge.leave(kg, acc, ref, l_run);
        __syncthreads();
        if (kg > 0) return;
#pragma unroll 1
        for (int g = 1; g < KS; ++g) {
            const v4f o = merge.numbers(g);
            const float top = __builtin_fmaxf(ref, o[0]);   // finite: group 0 has a block
            const float mine = fast_exp2(ref - top), theirs = fast_exp2(o[0] - top);
            merge.add(g, acc, mine, theirs);
            l_run = __builtin_fmaf(o[1], theirs, l_run * mine);
            ref = top;
        }
    }
    const float l = sum_over_row_pair(l_run);
    const float inv = l > 0.f ? 1.0f / l : 0.f;            // l already carries the factor 448
    store_rows(a, rows, lane, acc, inv, lds + row_block * kStoreRegionBytes,
               VCH ? a.sv + (size_t)bh * 128 : nullptr);
}

template <int SB, int W, bool MB, int KS = 1>
static void launch(const AttnArgs& a, bool vch, int grid, hipStream_t st) {
    if (vch) attn_fp8_kernel<SB, W, true, MB, KS><<<grid, KS * W * 64, 0, st>>>(a);
    else     attn_fp8_kernel<SB, W, false, MB, KS><<<grid, KS * W * 64, 0, st>>>(a);
}

void launch_attn_fp8(const AttnArgs& a, bool vch, int grid, hipStream_t st) {
    const Geom& g = a.g;
    const bool four = query_waves(g) == 4;
    switch (g.BS == 128 ? 4 : g.KBS) {
        case 4:
            if (g.KB > 1) {
                if (split_keys(a, 2)) launch<4, 4, true, 2>(a, vch, grid, st);
                else                  launch<4, 4, true>(a, vch, grid, st);
            } else {
                if (split_keys(a, 2)) launch<4, 4, false, 2>(a, vch, grid, st);
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
                else                  launch<2, 2, false>(a, vch, grid, st);
            } else if (four) {
                launch<2, 4, true>(a, vch, grid, st);
            } else {
                launch<2, 2, true>(a, vch, grid, st);
            }
            break;
        default:
            if (g.NS == 1) {
                if (split_keys(a, 4)) launch<1, 1, false, 4>(a, vch, grid, st);
                else                  launch<1, 1, false>(a, vch, grid, st);
            } else if (four) {
                launch<1, 4, true>(a, vch, grid, st);
            } else {
                launch<1, 1, true>(a, vch, grid, st);
            }
            break;
    }
}

}  // namespace fps
