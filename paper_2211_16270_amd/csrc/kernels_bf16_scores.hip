// bf16 score kernels (gfx950): joint rows in registers, W_out^T streamed through LDS, one pass over the vocabulary.
//   z = tanh(enc_t + pred_u)                       (Eq. 4)
//   h = z W_out + b_out on MFMA, fp32 accumulation   (Eq. 6)
// and, per mode,
//   MODE 0  running log-softmax statistics                                        (f^W_1)
//   MODE 1  dh = gamma softmax - posteriors as bf16, and z, into the chunk buffers (f^W_4, backward)
//   MODE 2  MODE 0, and z and the scores themselves kept for the backward pass, as fp16 differences t = h - m to a running
//           maximum m (t <= 0, so an entry's error exp(t) |t| 2^-11 in the softmax is at most 2^-11 / e whatever the size of
//           the scores; m is the row's largest score so far in its segment of the vocabulary, one float per row and 64 entries)
//
// A workgroup is 4 waves (8: eight_waves_pay); a wave owns 32 RB rows (RB = 1: half a lattice tile, 2: a whole one) and keeps their joint
// activations in registers for the whole pass (H/16 fragments of 4 registers per 32 rows: 128 registers at H = 512).
// The scores are computed transposed (A = 32 vocabulary entries of W_out^T, B = 32 rows), so a lane owns one row (with its
// partner lane in the other half) and the softmax reductions over the vocabulary stay in registers.
//
// What bounds it: the power limit in the forward pass.  On random bf16 values a loop of MFMAs alone runs at 1.8 PFLOP/s, with one 1 KiB
// fragment read from LDS per MFMA at 1.6, with two vector and one exponential instruction per MFMA besides at 1.45; at H = 512, V = 1024,
// 106 M nodes the forward kernel runs at 1.55 GHz with the matrix pipes busy 64 % of the time (1.1 PFLOP/s).  The backward form (MODE 1) keeps
// 2.0 GHz with the pipes busy 45 % (0.9 PFLOP/s) and waits more (41 % of the wave cycles against 32): it stores 2 bytes per score beside.
// A design in which every compute unit pulls a fragment from the L2 for every two MFMAs (64-row tiles, joint tile in LDS) reached
// 1.0-1.1; here the 128 or 256 rows of a workgroup share every fragment: W_out^T goes L2 -> LDS once per workgroup (asynchronous
// copies, a ring of stages).  The row statistics of the previous block are computed in the shadow of the current
// block's MFMAs (an MFMA holds the matrix pipe for 32 clocks and the issue port for 4; up to about 4 vector or 2
// transcendental instructions behind each one cost nothing), so one wave per SIMD is enough where the joint rows leave
// no registers for a second one.  Measured (forward kernel): H = 512, V = 8192, 4 M nodes 53.6 ms (61.4 before), H = 640, V = 4096 7.8 ms
// (9.5), H = 512, V = 1024, 106 M nodes 98.7 ms (111.8).
#include "device_common.h"
#include "plan.h"

namespace rnnt {

namespace {

struct ScoreArgs {
    Problem pr;
    SampleTable st;
    LatticeState ls;
    const bf16_t* Wp;
    int tile0, tile1;
    unsigned char* dH;     // MODE 1, 2: chunk buffers (device_common.h)
    unsigned char* Z;
    float* kept_max;       // MODE 2: [tiles][V/64][64 rows]
    ActiveTiles at;        // MODE 1
    f32x4* part;           // vocabulary split over gridDim.y > 1 (MODE 0, 2): [segments][rows of the launch] {max, sum, blank, label score}
};

constexpr int SC_VB = 32;          // vocabulary entries per block
constexpr int SC_RING = 8;         // W_out fragments a wave holds ahead of its MFMAs
// Smallest running maximum, finite: entries that are masked out (bias -inf, or finite and below anything a network gives) then have the
// exponential 0, and blocks or segments of nothing else the sum 0, instead of -inf - -inf or the rounding error of -1e30 log2 e in the
// exponent.  At this size that error is at most 2^6, and 2^64 times as many entries as there may be is still finite in fp32: maxima
// just above the floor lose to any other segment's without an infinity.
constexpr float SC_MAX_FLOOR = -1073741824.0f;
constexpr int SC_SPLIT_MAX_WG = 512;  // launches of more workgroups fill the chip without sharing the vocabulary (forward)
constexpr int SC_AGPR_FRAGS = 64;  // joint fragments kept in the 256 accumulation registers; the rest in vector registers

// LDS ring: stages of SF fragments (1 KiB each), a whole or half block of W_out^T, so many of them that a stage's copies are sent
// at least one whole stage ahead of their use, inside the 160 KiB of a compute unit (half of it where two workgroups share one).
constexpr int stage_frags(int KK, int WPS, int WAVES) { return KK <= 16 || (4 * WPS == WAVES && KK <= 32) ? KK : KK / 2; }
constexpr int score_stages(int KK, int WPS, int WAVES) {
    const int room = (4 * WPS == WAVES ? 152 : 76) / stage_frags(KK, WPS, WAVES);
    return room < 6 ? room : 6;
}
constexpr size_t score_smem_bytes(int KK, int WPS, int WAVES) {
    return (size_t)score_stages(KK, WPS, WAVES) * (stage_frags(KK, WPS, WAVES) * 1024 + 256) + 256;
}

template <int MODE, int KK, int RB, int WPS, int WAVES>
__global__ __launch_bounds__(64 * WAVES, WPS) void k_scores(ScoreArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int NST = score_stages(KK, WPS, WAVES), SF = stage_frags(KK, WPS, WAVES), SPB = KK / SF;
    constexpr unsigned SB = SF * 1024;
    constexpr int PER = SF / WAVES;                       // fragments a wave copies per stage
    constexpr int RG = SC_RING;
    constexpr int TW = WAVES / 2 * RB;                // lattice tiles per workgroup
    constexpr int NACC = MODE == 2 ? 4 : 2;           // score blocks alive: running, previous (MODE 2: two more until their pair is stored)
    static_assert(KK % RG == 0 && KK % SF == 0 && SF % WAVES == 0 && SF >= RG && NST >= 4, "ring geometry");
    static_assert(6 * ((PER + 1) / 2 - 1) < SF, "a stage's copies go out before the next hand-over");
    static_assert((NST - 1) * SB >= WAVES * JR_SCRATCH, "the build scratch lies in the later stages");
    const int H = KK * 16, V = a.pr.V;
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hb = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the workgroup's tiles (uniform)
    int n_tiles = a.tile1 - a.tile0;
    if (MODE == 1 && a.at.active) {
        const int left = *a.at.n_active - a.at.cbase;
        n_tiles = left < n_tiles ? left : n_tiles;
    }
    if ((int)blockIdx.x * TW >= n_tiles) return;
    const unsigned smem_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;
    float* bias_lds = reinterpret_cast<float*>(smem + NST * SB);          // [NST][64], 32 values and their repetition
    float* esum_lds = bias_lds + NST * 64;                               // [WAVES], and the arrival order [1]
    // this workgroup's part of the vocabulary: blocks [vb0, vb0 + nvb)
    const int vb0 = score_part_begin((int)blockIdx.y, (int)gridDim.y, V, MODE != 1);
    const int nvb = score_part_begin((int)blockIdx.y + 1, (int)gridDim.y, V, MODE != 1) - vb0;
    const char* wpb = reinterpret_cast<const char*>(a.Wp) + (size_t)vb0 * (KK * 1024) + wave * (PER * 1024);
    const float* bias_g = a.pr.b_out + vb0 * SC_VB;
    const unsigned lane_b = (unsigned)lane * 16u;
    // stage content q (fragments [q SF, q SF + SF) of W_out^T) -> ring slot: PER copies of 1 KiB by this wave, and the
    // 32 biases of its block (by every wave, the same values).  Four copies share one base pair (their immediate offset
    // moves both addresses).  They go out in pairs: next to the MFMAs of one wave per SIMD every issue slot counts, and a pair pays for
    // M0 and its wait state once (against single copies in this kernel and the two GEMMs: kept scores at H = 1024, V = 4096 11.47 -> 11.39 ms a call, H = 512, V = 8192
    // 22.27 -> 22.11).
    const int nq = nvb * SPB;
    constexpr int NI = (PER + 1) / 2;                 // pairs (or a last single one) per stage; issue NI: the biases
    auto issue_one = [&](int q, int slot, auto i_tag) {
        constexpr int i = decltype(i_tag)::value;
        q = q < nq ? q : nq - 1;                      // (past the end: a slot nobody reads any more)
        if constexpr (i < NI) {
            constexpr int c = 2 * i;
            const void* src = wpb + (size_t)q * SB + (c >> 2) * 4096;
            const unsigned dst = smem_base + (unsigned)slot * SB + (unsigned)(wave * PER * 1024 + (c >> 2) * 4096);
            if constexpr (c + 1 < PER) lds_dma16_pair<(c & 3) * 1024>(src, lane_b, dst);
            else lds_dma16_imm<(c & 3) * 1024>(src, lane_b, dst);
        } else
            lds_dma4_s(bias_g + (q / SPB) * SC_VB, (unsigned)l32 * 4u, smem_base + NST * SB + (unsigned)slot * 256u);
    };
    auto issue = [&](int q, int slot) { static_for<0, NI + 1>([&](auto i) { issue_one(q, slot, i); }); };
    issue(0, 0);

    const int ti = (int)blockIdx.x * TW + (RB == 2 ? wave : wave >> 1);
    const bool present = ti < n_tiles;
    const int tslot = __builtin_amdgcn_readfirstlane(present ? ti : n_tiles - 1);     // the tile's 64-row slot in the chunk buffers
    const int tile = __builtin_amdgcn_readfirstlane(
        (MODE == 1 && a.at.active) ? a.at.active[a.at.group_tile0 + a.at.cbase + tslot] : a.tile0 + tslot);
    const TilePos tp = locate_tile(a.st, tile);
    const int b = tp.s;
    // rows of this wave in its tile: 32 (half0 + rb) + l32
    const int half0 = RB == 2 ? 0 : wave & 1;
    const bf16_t* enc = reinterpret_cast<const bf16_t*>(a.pr.enc) + (size_t)b * a.pr.T_max * H;
    const bf16_t* prd = reinterpret_cast<const bf16_t*>(a.pr.pred) + (size_t)b * (a.pr.U_max + 1) * H;
    JointInputs<KK> in[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) in[rb].load(enc, prd, H, tp, half0 + rb, lane);
    int lab[RB];
    float gexp[RB], vB[RB], vY[RB];                   // MODE 1: exponent offset of the row, its final values at blank and label
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int r = 32 * (half0 + rb) + l32, t = tp.t0 + (r >> tp.us), u = tp.u0 + (r & (tp.uw - 1));
        lab[rb] = (t < tp.T && u < tp.U) ? a.pr.labels[(size_t)b * a.pr.U_max + u] : -1;
        if (MODE == 1) {
            gexp[rb] = RNNT_NEG_INF;
            vB[rb] = vY[rb] = 0.0f;
            if (t < tp.T && u <= tp.U) {
                const long long idx = (a.st.row_off[b] - a.ls.row_base) + lattice_index(tp.T, tp.U + 1, t, u);
                const RowDh rd = row_score_gradient(a.ls, idx, t, u, tp.T, tp.U, b, lab[rb], a.pr.blank);
                gexp[rb] = rd.g;
                vB[rb] = rd.at_blank;
                vY[rb] = rd.at_label;
            }
        }
    }
    u32x4 z[RB][KK];
    unsigned char* dh_out[RB];
    static_for<0, RB>([&](auto rb_tag) {
        constexpr int rb = decltype(rb_tag)::value;
        const size_t block = (size_t)tslot * 2 + half0 + rb;
        unsigned char* zout = nullptr;
        if (MODE != 0 && present && blockIdx.y == 0) zout = a.Z + block * chunk_block_bytes(H);
        if (MODE != 0) dh_out[rb] = a.dH + block * chunk_block_bytes(V) + (size_t)vb0 * 2048;
        build_joint_rows<KK, rb * KK, SC_AGPR_FRAGS>(z[rb], in[rb], reinterpret_cast<float*>(smem + SB) + wave * (JR_SCRATCH / 4), enc,
                                                     prd, H, tp, half0 + rb, lane, zout);
    });

    // every wave has left the build scratch: the remaining stages may be filled
    __syncthreads();
#pragma unroll
    for (int q = 1; q < NST; ++q) issue(q, q);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 1) * (PER + 1)) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    float m_run[RB], s_run[RB], m_tot[RB], s_tot[RB], cap_b[RB], cap_y[RB], m_pair[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        m_run[rb] = m_tot[rb] = SC_MAX_FLOOR;
        cap_b[rb] = cap_y[rb] = RNNT_NEG_INF;
        s_run[rb] = s_tot[rb] = m_pair[rb] = 0.0f;
    }
    const u32x4* frag0 = reinterpret_cast<const u32x4*>(smem) + lane;
    const float* bias0 = bias_lds + 4 * hb;
    u32x4 wf[RG];
#pragma unroll
    for (int i = 0; i < RG; ++i) wf[i] = frag0[i * 64];
    f32x4 bn[4];                                      // bias of the next block
#pragma unroll
    for (int j = 0; j < 4; ++j) bn[j] = *reinterpret_cast<const f32x4*>(bias0 + 8 * j);

    // Work on a finished block, cut into KK - 1 pieces (one behind each MFMA step of the next block).
    // MODE 0, 2: first the block's maximum, then the rescaled running sum.
    float tmax[RB] = {}, mn2[RB] = {}, sum0[RB] = {}, sum1[RB] = {};
    auto stats = [&](const f32x16& p, int rb, int k) {
        constexpr int NM = KK >= 32 ? 8 : 2;          // pieces that take the maximum, 16 / NM values each
        constexpr int NE = KK >= 32 ? 16 : KK - NM - 2;  // pieces that take the exponentials
        constexpr int PE = (16 + NE - 1) / NE;
        if (k < NM) {
            if (k == 0) tmax[rb] = p[0];
#pragma unroll
            for (int i = 0; i < 16 / NM; i += 2)
                tmax[rb] = fmaxf(fmaxf(tmax[rb], p[k * (16 / NM) + i]), p[k * (16 / NM) + i + 1]);
        } else if (k == NM) {
            const float mn = fmaxf(m_run[rb], both_halves_max(tmax[rb]));
            mn2[rb] = mn * LOG2E_F;
            s_run[rb] *= __builtin_amdgcn_exp2f((m_run[rb] - mn) * LOG2E_F);
            m_run[rb] = mn;
            sum0[rb] = sum1[rb] = 0.0f;
        } else if (k - NM - 1 < NE) {
#pragma unroll
            for (int q = 0; q < PE; ++q) {
                const int i = (k - NM - 1) * PE + q;
                if (i < 16) {
                    const float e = __builtin_amdgcn_exp2f(fmaf(p[i], LOG2E_F, -mn2[rb]));
                    if (i & 1) sum1[rb] += e; else sum0[rb] += e;
                }
            }
        }
        // (finishes each piece where it stands: the compiler would sink the arithmetic to the end of the block)
        asm volatile("" : "+v"(tmax[rb]), "+v"(sum0[rb]), "+v"(sum1[rb]));
    };
    auto rare = [&](int rb, int vb, auto&& at_hit) {
        const int vbase = (vb0 + vb) * SC_VB;
        int relb = a.pr.blank - vbase, rely = lab[rb] - vbase;
        if (__any((unsigned)rely < 32u) || (unsigned)relb < 32u) {
            // rarely taken: keep it a branch, and its comparisons inside
            relb -= 4 * hb;
            rely -= 4 * hb;
            asm volatile("" : "+v"(relb), "+v"(rely)::"memory");
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int vloc = 8 * (i >> 2) + (i & 3);
                at_hit(i, vloc == relb, vloc == rely);
            }
        }
    };
    auto capture = [&](const f32x16 (&p)[RB], int vb) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
            rare(rb, vb, [&](int i, bool blank, bool label) {
                if (blank) cap_b[rb] = p[rb][i];
                if (label) cap_y[rb] = p[rb][i];
            });
    };
    // a segment of the vocabulary is complete: fold it in, or leave it to the workgroup that arrives last
    auto fold = [&](int rb, float M, float S) {
        const float mn = fmaxf(m_tot[rb], M);
        s_tot[rb] = s_tot[rb] * __builtin_amdgcn_exp2f((m_tot[rb] - mn) * LOG2E_F) + S * __builtin_amdgcn_exp2f((M - mn) * LOG2E_F);
        m_tot[rb] = mn;
    };
    const int seg_blocks = V / SC_VB / score_segments(V);
    int seg = vb0 / seg_blocks, seg_next = seg_blocks;       // (MODE 0, 2) the segment, and the part's block behind its end
    const size_t part_rows = (size_t)gridDim.x * TW * 64, part_row = (size_t)ti * 64 + 32 * half0 + l32;
    auto segment_end = [&](int segment) {
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const float S = both_halves_sum(s_run[rb]);
            if (gridDim.y == 1) {
                fold(rb, m_run[rb], S);
            } else {
                const float cb = both_halves_max(cap_b[rb]), cy = both_halves_max(cap_y[rb]);
                if (hb == 0) {
                    float* q = reinterpret_cast<float*>(a.part + (size_t)segment * part_rows + part_row + 32 * rb);
                    __hip_atomic_store(q, m_run[rb], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(q + 1, S, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(q + 2, cb, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(q + 3, cy, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            m_run[rb] = SC_MAX_FLOOR;
            s_run[rb] = 0.0f;
        }
    };
    // MODE 1: the block's scores become its score gradients, in place, then two bf16 fragments per 32 rows
    auto dh_piece = [&](f32x16& p, int rb, int vb, auto k_tag) {
        constexpr int k = decltype(k_tag)::value;     // 1 .. KK - 1
        constexpr int PE = KK >= 24 ? 1 : (16 + KK - 5) / (KK - 4), NE = (16 + PE - 1) / PE;
        if constexpr (k <= NE) {
#pragma unroll
            for (int q = 0; q < PE; ++q) {
                const int i = (k - 1) * PE + q;
                if (i < 16) {
                    float d = __builtin_amdgcn_exp2f(fmaf(p[i], LOG2E_F, gexp[rb]));
                    asm volatile("" : "+v"(d));
                    p[i] = d;
                }
            }
        } else if constexpr (k == NE + 1) {
            rare(rb, vb, [&](int i, bool blank, bool label) {
                if (blank) p[i] = vB[rb];
                if (label) p[i] = vY[rb];
            });
        } else if constexpr (k == NE + 2 || k == NE + 3) {
            constexpr int h = k - NE - 2;
            const u32x4 f = fragment_from_scores(p, h);
            if (present)
                __builtin_nontemporal_store(f, reinterpret_cast<u32x4*>(dh_out[rb] + (size_t)vb * 2048 + h * 1024 +
                                                                        frag_granule(lane, h)));
        }
    };
    // MODE 2: a pair of blocks (64 entries) leaves as fp16 differences to the running maximum after the pair
    typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
    auto keep_piece = [&](const f32x16& p, int rb, int vb, int h) {
        f16x8 t;
#pragma unroll
        for (int i = 0; i < 8; ++i) t[i] = (_Float16)(p[8 * h + i] - m_pair[rb]);
        if (present)
            __builtin_nontemporal_store(__builtin_bit_cast(u32x4, t),
                                        reinterpret_cast<u32x4*>(dh_out[rb] + (size_t)vb * 2048 + h * 1024 + lane_b));
    };
    auto keep_max = [&](int rb, int vb) {
        if (present && hb == 0)
            a.kept_max[((size_t)tslot * (V / 64) + ((vb0 + vb) >> 1)) * 64 + 32 * (half0 + rb) + l32] = m_pair[rb];
    };

    // One block: KK steps of RB MFMAs; behind them the LDS read of the fragment RG steps ahead, a piece of work on the
    // previous block and, every sixth step, a pair of copies into a slot that has been left.  RG steps before the end of a stage
    // its last fragment read is on its way; there the next stage is waited for (own copies, then everyone's; the stores of MODE 1 and 2
    // count in the same order, so the wait may cover a few of them).  Every wave has then consumed its fragments of the stage before,
    // whose slot may be refilled (refilling the slot just read would need a wait for the reads just sent).
    int q = 0, slot = 0;                              // stage being read (content, ring slot)
    const u32x4* fs = frag0;                          // its fragments
    f32x16 acc[NACC][RB];
    // CUR: accumulator set of block vb; the previous block's is (CUR + NACC - 1) % NACC
    auto block = [&](auto cur_tag, int vb, bool with_prev, bool with_pair) {
        constexpr int CUR = decltype(cur_tag)::value, PREV = (CUR + NACC - 1) % NACC;
        f32x16 (&cur)[RB] = acc[CUR];
        f32x16 (&prev)[RB] = acc[PREV];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) cur[rb][4 * j + i] = bn[j][i];
        static_for<0, KK>([&](auto k_tag) {
            constexpr int k = decltype(k_tag)::value, kk = k % SF;
            if constexpr (kk == SF - RG) {
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 3) * (PER + 1)) : "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                ++q;
                slot = slot + 1 == NST ? 0 : slot + 1;
                fs = frag0 + slot * (SB / 16);
            }
            if constexpr (k == 0) mfma_after_valu(cur);
            static_for<0, RB>([&](auto rb_tag) {
                constexpr int rb = decltype(rb_tag)::value;
                mfma_zb<(rb * KK + k < SC_AGPR_FRAGS)>(cur[rb], wf[k % RG], z[rb][k]);
            });
            wf[k % RG] = fs[((kk + RG) % SF) * 64];
            if constexpr (k >= KK - 4)
                bn[k - (KK - 4)] = *reinterpret_cast<const f32x4*>(bias0 + slot * 64 + 8 * (k - (KK - 4)));
            // refill of the slot before the one left last (q counts the stage being read): content q - 2 + NST, spread over the SF
            // steps up to the next hand-over
            constexpr int p = (kk + RG) % SF;
            if constexpr ((p % 6 == 0 && p / 6 < NI) || p == 3) {
                if (with_prev || k >= 2 * SF - RG)
                    issue_one(q - 2 + NST, slot < 2 ? slot + NST - 2 : slot - 2, std::integral_constant<int, p == 3 ? NI : p / 6>{});
            }
            __builtin_amdgcn_sched_barrier(0);
            if (with_prev) {
                if constexpr (MODE != 1) {
                    if constexpr (k == 1) capture(prev, vb - 1);
                    if constexpr (k >= 1) {
#pragma unroll
                        for (int rb = 0; rb < RB; ++rb) stats(prev[rb], rb, k - 1);
                    }
                    if constexpr (k == KK - 1) {
#pragma unroll
                        for (int rb = 0; rb < RB; ++rb) {
                            s_run[rb] += sum0[rb] + sum1[rb];
                            if (MODE == 2) m_pair[rb] = m_run[rb];
                        }
                        if (vb == seg_next) {
                            segment_end(seg++);
                            seg_next += seg_blocks;
                        }
                    }
                    if constexpr (MODE == 2 && CUR % 2 == 1) {
                        // the pair (vb - 3, vb - 2): its running maximum was complete when block vb - 1 ended
                        constexpr int S0 = KK >= 32 ? KK / 8 : 1;
                        if constexpr (k >= 1 && (k - 1) % S0 == 0 && (k - 1) / S0 < 4) {
                            constexpr int e = (k - 1) / S0;
                            if (with_pair) {
#pragma unroll
                                for (int rb = 0; rb < RB; ++rb) {
                                    keep_piece(acc[(CUR + 1 + e / 2) % NACC][rb], rb, vb - 3 + e / 2, e % 2);
                                    if (e == 0) keep_max(rb, vb - 3);
                                }
                            }
                        }
                    }
                } else if constexpr (k >= 1) {
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) dh_piece(prev[rb], rb, vb - 1, k_tag);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    typedef std::integral_constant<int, 0> I0;
    typedef std::integral_constant<int, 1> I1;
    typedef std::integral_constant<int, 2> I2;
    typedef std::integral_constant<int, 3> I3;
    block(I0{}, 0, false, false);
    if constexpr (MODE != 2) {
        for (int vb = 1; vb + 1 < nvb; vb += 2) {
            block(I1{}, vb, true, false);
            block(I0{}, vb + 1, true, false);
        }
        block(I1{}, nvb - 1, true, false);            // nvb is a multiple of 2 (MODE 2: of 4)
    } else {
        block(I1{}, 1, true, false);
        for (int vb = 2; vb + 2 < nvb; vb += 4) {
            block(I2{}, vb, true, false);
            block(I3{}, vb + 1, true, true);
            block(I0{}, vb + 2, true, false);
            block(I1{}, vb + 3, true, true);
        }
        block(I2{}, nvb - 2, true, false);
        block(I3{}, nvb - 1, true, true);
    }
    auto tail = [&](auto set_tag) {
        constexpr int S = decltype(set_tag)::value;
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) mfma_result_ready(acc[S][rb]);
        if constexpr (MODE == 1) {
            static_for<1, KK>([&](auto k_tag) {
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) dh_piece(acc[S][rb], rb, nvb - 1, k_tag);
            });
        } else {
            capture(acc[S], nvb - 1);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
                for (int k = 0; k < KK - 1; ++k) stats(acc[S][rb], rb, k);
                s_run[rb] += sum0[rb] + sum1[rb];
                if (MODE == 2) {
                    m_pair[rb] = m_run[rb];
#pragma unroll
                    for (int e = 0; e < 4; ++e) keep_piece(acc[S - 1 + e / 2][rb], rb, nvb - 2 + e / 2, e % 2);
                    keep_max(rb, nvb - 2);
                }
            }
            segment_end(seg);
        }
    };
    tail(std::integral_constant<int, NACC - 1>{});
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no copy may land after the workgroup has ended
    if constexpr (MODE == 1) return;

    if (gridDim.y > 1) {
        // the workgroup of this column that arrives last folds the segments of all of them, in order
        int* order = reinterpret_cast<int*>(esum_lds + WAVES);
        // (the segments leave as agent-scope stores, complete at the vmcnt(0) above, and are read by agent-scope loads: no cache
        // has to be written back or invalidated between them)
        __syncthreads();
        if (tid == 0) {
            // (the counter: the emission sum of the column's first tile, zero until the last one stores it below)
            int* arrived = reinterpret_cast<int*>(a.ls.tile_esum) + a.tile0 + blockIdx.x * TW;
            *order = __hip_atomic_fetch_add(arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (*order != (int)gridDim.y - 1) return;
        auto fold_all = [&](auto n_tag) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
                for (int seg = 0; seg < decltype(n_tag)::value; ++seg) {
                    const float* p = reinterpret_cast<const float*>(a.part + (size_t)seg * part_rows + part_row + 32 * rb);
                    const float M = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    const float S = __hip_atomic_load(p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    cap_b[rb] = fmaxf(cap_b[rb], __hip_atomic_load(p + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                    cap_y[rb] = fmaxf(cap_y[rb], __hip_atomic_load(p + 3, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                    fold(rb, M, S);
                }
            }
        };
        if (score_segments(V) == 8) fold_all(std::integral_constant<int, 8>{});
        else fold_all(std::integral_constant<int, 4>{});
    }
    float esum = 0.0f;
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int r = 32 * (half0 + rb) + l32, t = tp.t0 + (r >> tp.us), u = tp.u0 + (r & (tp.uw - 1));
        const float cb = both_halves_max(cap_b[rb]), cy = both_halves_max(cap_y[rb]);
        const float lse = m_tot[rb] + __logf(s_tot[rb]);
        if (present && t < tp.T && u <= tp.U && hb == 0) {
            const long long idx = (a.st.row_off[b] - a.ls.row_base) + lattice_index(tp.T, tp.U + 1, t, u);
            a.ls.lse[idx] = lse;
            a.ls.em[idx] = emissions(cb - lse, lab[rb] >= 0 ? cy - lse : EMISSION_FLOOR);
            // this node's share of the sum the lattice kernels take their per-sample offset from
            esum += fmaxf((u < tp.U ? fmaxf(cb, cy) : cb) - lse, OFFSET_FLOOR);
        }
    }
    esum = wave_sum(esum);
    if constexpr (RB == 2) {
        if (lane == 0 && present) a.ls.tile_esum[tile] = esum;
    } else {
        if (lane == 0) esum_lds[wave] = esum;
        __syncthreads();
        if (lane == 0 && (wave & 1) == 0 && present) a.ls.tile_esum[tile] = esum + esum_lds[wave + 1];
    }
}

template <int MODE, int KK, int RB, int WPS, int WAVES = 4>
hipError_t launch_scores_t(ScoreArgs a, size_t part_bytes, hipStream_t stream) {
    constexpr int TW = WAVES / 2 * RB, SLOTS = 256 * 4 * WPS / WAVES;
    const int n = (a.tile1 - a.tile0 + TW - 1) / TW;
    constexpr size_t smem = score_smem_bytes(KK, WPS, WAVES);
    static bool configured = false;
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_scores<MODE, KK, RB, WPS, WAVES>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
        configured = true;
    }
    int vs = 1;
    // (kept scores leave in pairs of blocks, two pairs at a time)
    if (MODE == 1 || n <= SC_SPLIT_MAX_WG) vs = score_split(n, SLOTS, a.pr.V, MODE != 1, MODE == 2 ? 4 : 2).parts;
    if (MODE != 1 && (size_t)score_segments(a.pr.V) * n * TW * 64 * sizeof(f32x4) > part_bytes) vs = 1;
    k_scores<MODE, KK, RB, WPS, WAVES><<<dim3((unsigned)n, (unsigned)vs), dim3(64 * WAVES), smem, stream>>>(a);
    return hipGetLastError();
}

// Joint size 640, half tiles per wave (RB = 1) instead of whole ones: twice the workgroups of half the cost each.  A whole tile's workgroup reads half
// as much from LDS per MFMA, but a small launch of them has to split the vocabulary to fill the chip, and then every part builds the
// joint rows again, which costs as much as 8 blocks.  A call with V = 1024: one sample of 250 x 50 176 -> 147 us, two of 120 x 24 148 -> 116,
// eight 195 -> 179, 32 619 -> 567; sixteen, where the rule leaves the whole tiles, 361 -> 362; V = 4096: one sample 319 -> 269 us.
bool half_tiles_pay(int tiles, int V, bool statistics) {
    const long long c2 = 2 * score_split((tiles + 3) / 4, 256, V, statistics).cost, c1 = score_split((tiles + 1) / 2, 256, V, statistics).cost;
    return c1 * 10 < c2 * 9;
}

// Joint sizes 384 and 512: one workgroup of eight waves per compute unit instead of two of four.  W_out^T crosses from the L2 once for all eight
// waves and its stages are twice as long (half the hand-overs); on the other hand nothing stands beside the start and end of a workgroup,
// which weigh less the longer the vocabulary.  Losses alone, 64 samples of 400 x 80: H = 384 V = 1024 951 -> 950 us, 2048 1703 -> 1657, 8192
// 6253 -> 5922; H = 512 V = 1024 1156 -> 1169, 2048 2072 -> 2069, 4096 3944 -> 3888.  In the backward form the stores of dH push W_out^T out of the L2
// where it comes near the 4 MiB of an XCD, so there the line lies at H V.  Calls with both kernels in eight waves, 64 samples of 400 x 80: H = 384
// V = 2048 6874 -> 6975 us, 4096 13354 -> 13268 (the forward kernel alone gains 125), 8192 30.4 -> 29.8 ms; H = 512 V = 1024 4448 -> 4487 us, 2048 8189
// -> 8298, 4096 15.54 -> 15.38 ms, 8192 30.7 -> 30.1 (256 samples of up to 800 x 240: 198.6 -> 191.1 ms).  Joint sizes 128 and 256, whose
// stages are no longer with eight waves, lose 1 to 18 %.  So do launches that leave most of the chip idle (a few workgroups per XCD, the vocabulary
// split): H = 512, 12 tiles, V = 5376 134 -> 167 us a call, 100 tiles, V = 6144 219 -> 239; below half a round (512 tiles) it is four waves.
bool eight_waves_pay(int mode, const Problem& pr, int tiles) {
    if (tiles < 512) return false;
    return mode == 0 ? pr.V >= (pr.H == 384 ? 2048 : 4096) : (long long)pr.H * pr.V >= 1 << 21;
}

}  // namespace

// Joint sizes up to 512: two workgroups per compute unit (one's joint rows are built beside the other's MFMAs), or one of eight waves; 640: whole
// tiles per wave (half the LDS reads per MFMA) where they fill the chip; above: 32 rows per wave fill the registers.
hipError_t launch_fwd_bf16(const Problem& pr, const void* Wpack, const SampleTable& st, const LatticeState& ls, int tile0,
                           int tile1, void* part, size_t part_bytes, hipStream_t stream) {
    if (tile1 <= tile0) return hipSuccess;
    const ScoreArgs a{pr, st, ls, (const bf16_t*)Wpack, tile0, tile1, nullptr, nullptr, nullptr, EVERY_TILE, (f32x4*)part};
    switch (pr.H) {
        case 128: return launch_scores_t<0, 8, 1, 2>(a, part_bytes, stream);
        case 256: return launch_scores_t<0, 16, 1, 2>(a, part_bytes, stream);
        case 384:
            return eight_waves_pay(0, pr, tile1 - tile0) ? launch_scores_t<0, 24, 1, 2, 8>(a, part_bytes, stream)
                                          : launch_scores_t<0, 24, 1, 2>(a, part_bytes, stream);
        case 512:
            return eight_waves_pay(0, pr, tile1 - tile0) ? launch_scores_t<0, 32, 1, 2, 8>(a, part_bytes, stream)
                                          : launch_scores_t<0, 32, 1, 2>(a, part_bytes, stream);
        case 640:
            return half_tiles_pay(tile1 - tile0, pr.V, true) ? launch_scores_t<0, 40, 1, 1>(a, part_bytes, stream)
                                                       : launch_scores_t<0, 40, 2, 1>(a, part_bytes, stream);
        case 768: return launch_scores_t<0, 48, 1, 1>(a, part_bytes, stream);
        case 896: return launch_scores_t<0, 56, 1, 1>(a, part_bytes, stream);
        case 1024: return launch_scores_t<0, 64, 1, 1>(a, part_bytes, stream);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_bwd_scores_bf16(const Problem& pr, const void* Wpack, const SampleTable& st, const LatticeState& ls, int tile0,
                                  int tile1, void* dH, void* Z, const ActiveTiles& at, hipStream_t stream) {
    if (tile1 <= tile0) return hipSuccess;
    const ScoreArgs a{pr, st, ls, (const bf16_t*)Wpack, tile0, tile1, (unsigned char*)dH, (unsigned char*)Z, nullptr, at, nullptr};
    switch (pr.H) {
        case 128: return launch_scores_t<1, 8, 1, 2>(a, 0, stream);
        case 256: return launch_scores_t<1, 16, 1, 2>(a, 0, stream);
        case 384:
            return eight_waves_pay(1, pr, tile1 - tile0) ? launch_scores_t<1, 24, 1, 2, 8>(a, 0, stream) : launch_scores_t<1, 24, 1, 2>(a, 0, stream);
        case 512:
            return eight_waves_pay(1, pr, tile1 - tile0) ? launch_scores_t<1, 32, 1, 2, 8>(a, 0, stream) : launch_scores_t<1, 32, 1, 2>(a, 0, stream);
        case 640:
            return half_tiles_pay(tile1 - tile0, pr.V, false) ? launch_scores_t<1, 40, 1, 1>(a, 0, stream)
                                                       : launch_scores_t<1, 40, 2, 1>(a, 0, stream);
        case 768: return launch_scores_t<1, 48, 1, 1>(a, 0, stream);
        case 896: return launch_scores_t<1, 56, 1, 1>(a, 0, stream);
        case 1024: return launch_scores_t<1, 64, 1, 1>(a, 0, stream);
    }
    return hipErrorInvalidValue;
}

// Kept scores: two workgroups per compute unit up to 384 (the stores of one stand beside the other's MFMAs; against
// one, 64 samples of 500 x 100, V = 1024: H = 256 4.85 -> 4.21 ms a call, H = 384 6.71 -> 6.09 ms; 16 samples, H = 256, V = 4096
// 4.88 -> 4.32 ms).  At 512 the two further score blocks that wait for their pair leave no registers for a second one (13 would spill).
// A small launch splits the vocabulary as the forward kernel without kept scores does (one sample of 250 x 50, V = 1024: H = 256 144 -> 135 us a
// call, H = 384 160 -> 150, H = 640 188 -> 173, H = 1024 213 -> 194).
hipError_t launch_fwd_keep_bf16(const Problem& pr, const void* Wpack, const SampleTable& st, const LatticeState& ls, int tile0,
                                int tile1, void* kept, void* Z, float* kept_max, void* part, size_t part_bytes, hipStream_t stream) {
    if (tile1 <= tile0) return hipSuccess;
    const ScoreArgs a{pr, st, ls, (const bf16_t*)Wpack, tile0, tile1, (unsigned char*)kept, (unsigned char*)Z, kept_max, EVERY_TILE,
                      (f32x4*)part};
    switch (pr.H) {
        case 128: return launch_scores_t<2, 8, 1, 2>(a, part_bytes, stream);
        case 256: return launch_scores_t<2, 16, 1, 2>(a, part_bytes, stream);
        case 384: return launch_scores_t<2, 24, 1, 2>(a, part_bytes, stream);
        case 512: return launch_scores_t<2, 32, 1, 1>(a, part_bytes, stream);
        case 640: return launch_scores_t<2, 40, 1, 1>(a, part_bytes, stream);
        case 768: return launch_scores_t<2, 48, 1, 1>(a, part_bytes, stream);
        case 896: return launch_scores_t<2, 56, 1, 1>(a, part_bytes, stream);
        case 1024: return launch_scores_t<2, 64, 1, 1>(a, part_bytes, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace rnnt
