// dz GEMM of the bf16 backward pass (Alg. 1 lines 10, 11):
//   dz = dH W_out^T   (dH [rows,V] from the chunk buffer, contraction over the vocabulary),
//   dx = dz (1 - z^2),  d_enc[t] += sum_u dx,  d_pred[u] += sum_t dx  per lattice tile (64 rows: 8 frames x 8 labels or 16 x 4).
//
// 256x256 output tile (4 lattice tiles x 256 hidden) per workgroup; 512 threads = 8 waves in 2 x 4, two per SIMD, each 128 x 64 = 4 x 2
// accumulator tiles (short vocabularies, dz_waves: 128x256 and 4 waves, two workgroups per compute unit, three stages of 24 KiB each), so that one k16-step is 6 LDS fragment reads for 8 MFMAs, and one wave's waits and epilogue stand beside the other's
// work.  (Four waves of 128 x 128, one per SIMD, read a third less from LDS and were slower, see below.)  Where only 128 hidden columns are left
// (H not a multiple of 256) the waves stand 4 x 2, each 64 x 64.
// Both operands lie in memory as MFMA fragments of 1 KiB (dH: device_common.h; W_out: the packed copy
// [V/16][H/32]), so stages of 32 vocabulary entries (16 fragments of each) travel global -> LDS
// asynchronously in whole cache lines, five (three) stages deep, and are read back without bank conflicts.  Fragments are read one
// k16-step ahead of their MFMAs, also across the stage hand-over.
//
// Epilogue: 1 - z^2 = 4 r (1 - r) with r = 1 / (1 + e^{2 enc} e^{2 pred}), one reciprocal per
// element from per-row exponentials; the input rows they come from are loaded before the main loop.  Everything after the product
// is linear in dz, so the vocabulary may be split over workgroups: a launch that leaves the chip partly idle, or its last
// round partly filled, does that.
// What bounds it: of 9.6 ms (H = 512, V = 1024, 13 M nodes, 0.58 of the tiles) the MFMAs alone take 5.3 (1.6 PFLOP/s, power), the epilogue 2.7 (0.7 of it
// its atomics, 0.3 the reciprocals), the copies 1.1 and the LDS reads 0.3.  Four waves instead of eight, four stages deep: 10.7; V = 8192, 3.7 M nodes 19.3 ms
// against 18.6; H = 640, V = 1024, 32 k rows 654 us against 620.  No copies past the last stage, by a branch around them: 9.8 and 19.2.
#include "device_common.h"
#include "gemm_dw_tile.h"
#include "plan.h"

namespace rnnt {

namespace {

constexpr int ZT = 256;       // tile edge
constexpr int ZK = 32;        // vocabulary entries per stage
constexpr int z_stages(int WAVES) { return WAVES == 8 ? 5 : 3; }
constexpr unsigned z_a_bytes(int WAVES) { return WAVES * 2048u; }                 // dH's part of a stage
constexpr unsigned z_stage_bytes(int WAVES) { return z_a_bytes(WAVES) + 16u * 1024u; }
constexpr int Z_EP = 264;     // pitch (floats) of the epilogue's rows in LDS
constexpr int Z_ROWS = 20;    // input rows of a lattice tile: 8 + 8 or 16 + 4

struct DzArgs {
    const unsigned char* dH;
    const unsigned char* Wq;
    Problem pr;
    SampleTable st;
    int tile0, tile1;
    float* d_enc;
    float* d_pred;
    int n_tiles;              // hidden tiles, the half one included
    int edge;                 // their width: 256, or 128 (half tiles only)
    int v_splits;             // parts of the vocabulary
    int per_part;             // workgroups per part, a multiple of 8
    ActiveTiles at;           // which tiles the chunk's 64-row slots hold (see kernels.h)
};

// HALF: the last hidden tile, 128 columns; vs: part of the vocabulary
template <bool HALF, int WAVES>
__device__ __forceinline__ void dz_tile(const DzArgs& g, unsigned char* dz_smem, int bx, int n0, int n_slots, int vs) {
    constexpr int MT = HALF ? 2 : 4;                  // 32-row blocks per wave
    constexpr int DMAS = 2 + (HALF ? 8 : 16) / WAVES; // copies per wave and stage
    constexpr int TILES = WAVES / 2, ZST = z_stages(WAVES), NB = 8 / WAVES * (HALF ? 1 : 2);      // NB: hidden blocks of an entry half a wave copies
    constexpr int NI = HALF || WAVES == 8 ? 2 : 3;    // issues per stage
    constexpr unsigned Z_OPER = z_a_bytes(WAVES), Z_STAGE = z_stage_bytes(WAVES);
    const int tid = threadIdx.x;
    const int lane = tid & 63, l32 = lane & 31, hb = lane >> 5;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = HALF ? wv >> 1 : wv >> 2, wn = HALF ? wv & 1 : wv & 3;
    const int H = g.pr.H, V = g.pr.V;
    const unsigned smem_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)dz_smem;

    // global -> LDS: a stage is, per operand, blocks of 32 rows (lattice rows / hidden columns) x 2 fragments of 16 entries.
    // LDS order: A [WAVES row blocks][entry half], B [entry half][8 hidden blocks].  Wave w moves row block w (lattice tile w / 2) and, of entry half
    // w / TILES, NB hidden blocks from NB (w % TILES) on: 2 with eight waves, 4 with four (HALF: 1 and 2).  Everything but the lane's 16 bytes is
    // wave-uniform.  Slots past the list's end read the last listed tile again; their products are never stored.
    const size_t DB = chunk_block_bytes(V);   // bytes of a block of 32 rows of dH
    const unsigned lane_b = (unsigned)lane * 16u;
    const int wt = wv >> 1;                           // lattice tile whose copies and input rows are this wave's
    const bool present = bx * TILES + wt < n_slots;
    const int entry = present ? bx * TILES + wt : n_slots - 1;
    const int tile = __builtin_amdgcn_readfirstlane(g.at.active ? g.at.active[g.at.group_tile0 + g.at.cbase + entry] : g.tile0 + entry);
    // (kept scores: wherever the forward pass has put the listed tile)
    const int slot = (g.at.active && g.at.slot_tile0 >= 0) ? tile - g.at.slot_tile0 : entry;
    const int nsteps = V / ZK / g.v_splits, step0 = vs * nsteps;
    const unsigned char* As = g.dH + (size_t)(2 * slot + (wv & 1)) * DB + (size_t)step0 * 2048;
    const size_t WB = (size_t)(H / 32) * 1024;        // bytes of 16 entries of Wq
    const unsigned char* Bs = g.Wq + (size_t)step0 * 2 * WB + (size_t)(wv / TILES) * WB + (size_t)(n0 / 32 + NB * (wv % TILES)) * 1024;
    // The copies of stage gstep into LDS buffer buf, NI issues: both entry halves of the row block (j = 0), the hidden blocks (1; four of them: 1 and 2).
    // (In pairs: M0 and its wait state once.)
    auto issue = [&](int gstep, unsigned buf, auto j_tag) {
        constexpr int j = decltype(j_tag)::value;
        const unsigned sb = smem_base + buf * Z_STAGE;
        const unsigned bdst = sb + Z_OPER + (unsigned)((wv / TILES) * 8 + NB * (wv % TILES)) * 1024u;
        if constexpr (j == 0) lds_dma16_pair<0>(As + (size_t)gstep * 2048, lane_b, sb + (unsigned)wv * 2048u);
        else if constexpr (NB == 1) lds_dma16_s(Bs + (size_t)gstep * 2 * WB, lane_b, bdst);
        else lds_dma16_pair<(j - 1) * 2048>(Bs + (size_t)gstep * 2 * WB, lane_b, bdst);
    };
    const int last = nsteps - 1;
#pragma unroll
    for (int s5 = 0; s5 < ZST; ++s5)
        static_for<0, NI>([&](auto j) { issue(s5 < last ? s5 : last, (unsigned)s5, j); });

    // the epilogue's input rows, half of a lattice tile's per wave: lane = 8 columns of every second (HALF: fourth) row (zero outside the sample)
    const TilePos tp = locate_tile(g.st, tile);
    constexpr int NC = HALF ? 16 : 32, RPS = 64 / NC, NR = (Z_ROWS / RPS + 1) / 2;      // 8-column pieces per row, rows per step, steps
    bf16x8 in[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int r = lane / NC + RPS * (NR * (wv & 1) + i), c = lane % NC, th = 64 >> tp.us, u = tp.u0 + r - th;
        const bool is_enc = r < th, ok = is_enc ? tp.t0 + r < tp.T : (r - th < tp.uw && u <= tp.U);
        const bf16_t* src = is_enc ? reinterpret_cast<const bf16_t*>(g.pr.enc) + ((size_t)tp.s * g.pr.T_max + tp.t0 + r) * H
                                   : reinterpret_cast<const bf16_t*>(g.pr.pred) + ((size_t)tp.s * (g.pr.U_max + 1) + u) * H;
        in[i] = bf16x8{};
        if (ok) in[i] = *reinterpret_cast<const bf16x8*>(src + n0 + c * 8);
    }

    // fragment of a row block, k16-step kk (= entry half): dH lies with its rows permuted (frag_granule), W_out in lane order
    const unsigned a_off[2] = {frag_granule(lane, 0), frag_granule(lane, 1)};
    f32x16 acc[MT][2];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x16{0};
    bf16x8 fa[2][MT], fb[2][2];
    auto frag_a = [&](unsigned buf, int kk, int mt) {
        return *reinterpret_cast<const bf16x8*>(dz_smem + buf * Z_STAGE + (wm * MT + mt) * 2048 + kk * 1024 + a_off[kk]);
    };
    auto frag_b = [&](unsigned buf, int kk, int nt) {
        return *reinterpret_cast<const bf16x8*>(dz_smem + buf * Z_STAGE + Z_OPER + kk * 8192 + (wn * 2 + nt) * 1024 + lane_b);
    };
    // The MFMAs of one k16-step (register set `set`).  Behind each of the first ones, one fragment of the following k16-step is
    // read into the other set; behind two of the last ones of the second step go the copies of a later stage.
    auto multiply = [&](auto set_tag, unsigned next_buf, auto next_kk_tag, int it, unsigned buf) {
        constexpr int set = decltype(set_tag)::value, next_kk = decltype(next_kk_tag)::value;
        static_for<0, 2 * MT>([&](auto idx_tag) {
            constexpr int idx = decltype(idx_tag)::value, mt = idx >> 1, nt = idx & 1;
            acc[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][mt], fb[set][nt], acc[mt][nt], 0, 0, 0);
            if constexpr (idx < MT) fa[set ^ 1][idx] = frag_a(next_buf, next_kk, idx);
            else if constexpr (idx < MT + 2) fb[set ^ 1][idx - MT] = frag_b(next_buf, next_kk, idx - MT);
            if constexpr (set == 1 && idx >= 2 * MT - 2 * NI && idx % 2 == 0)
                issue(it + ZST < last ? it + ZST : last, buf, std::integral_constant<int, (idx - (2 * MT - 2 * NI)) / 2>{});
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    // All stages in flight before the first one is consumed.  The hand-over to the next stage (wait for this wave's copies, then for
    // everyone's) sits in the middle of a stage; there every wave has read all its fragments of the present one, whose buffer may be
    // refilled.  Beyond the last stage the pipeline re-loads the last one into buffers nobody reads
    // any more, which keeps the loop free of branches and the number of copies in flight constant.  The waits for LDS reads are placed by hand (as the builtin the compiler's own counter tracking understands) before the
    // reads of the following step are issued: the counter completes in order, so a wait placed after them would wait for them too.
    typedef std::integral_constant<int, 0> I0;
    typedef std::integral_constant<int, 1> I1;
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((ZST - 1) * DMAS) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < MT; ++i) fa[0][i] = frag_a(0, 0, i);
#pragma unroll
    for (int i = 0; i < 2; ++i) fb[0][i] = frag_b(0, 0, i);
    unsigned buf = 0;                                 // of stage it
    for (int it = 0; it < nsteps; ++it) {
        const unsigned next = buf + 1 == ZST ? 0 : buf + 1;
        __builtin_amdgcn_s_waitcnt(WAIT_LGKM0);
        __builtin_amdgcn_sched_barrier(0);
        multiply(I0{}, buf, I1{}, 0, 0u);
        __builtin_amdgcn_s_waitcnt(WAIT_LGKM0);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((ZST - 2) * DMAS) : "memory");  // of stage it + 1; the later ones stay in flight
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        multiply(I1{}, next, I0{}, it, buf);
        buf = next;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();                                  // the stages become the epilogue's scratch

    // ---- epilogue.  Per lattice tile Z_ROWS rows of e^{2x}: the tile's frames, behind them its label positions; where an input lies beyond
    // +-40 (the product of two exponentials could overflow, or cancel as inf * 0) the tile's rows are the inputs themselves.
    float* ex = reinterpret_cast<float*>(dz_smem);                // [TILES][Z_ROWS][Z_EP]
    struct TileInfo {
        int s, T, U, t0, u0, us;
        int far[2];                                   // an input of the first, second half of the rows lies beyond the limit
    };
    TileInfo* info = reinterpret_cast<TileInfo*>(dz_smem + TILES * Z_ROWS * Z_EP * sizeof(float));
    {
        constexpr float K2 = 2.0f * LOG2E_F;
        float big = 0.0f;
#pragma unroll
        for (int i = 0; i < NR; ++i)
#pragma unroll
            for (int k = 0; k < 8; ++k) big = fmaxf(big, fabsf((float)in[i][k]));
        const bool far = __any(!(big <= 115.0f / K2));
        if (lane == 0) info[wt].far[wv & 1] = far;
        __syncthreads();
        const bool by_sum = (info[wt].far[0] | info[wt].far[1]) != 0;
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const int r = lane / NC + RPS * (NR * (wv & 1) + i);
            if (r >= Z_ROWS) continue;
            float* dst = ex + (wt * Z_ROWS + r) * Z_EP + (lane % NC) * 8;
            f32x4 lo, hi;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                lo[k] = (float)in[i][k];
                hi[k] = (float)in[i][4 + k];
                if (!by_sum) {
                    lo[k] = __builtin_amdgcn_exp2f(lo[k] * K2);
                    hi[k] = __builtin_amdgcn_exp2f(hi[k] * K2);
                }
            }
            *reinterpret_cast<f32x4*>(dst) = lo;
            *reinterpret_cast<f32x4*>(dst + 4) = hi;
        }
        if (lane == 0 && (wv & 1) == 0) {
            TileInfo& ti = info[wt];
            ti.s = present ? tp.s : -1;
            ti.T = tp.T; ti.U = tp.U; ti.t0 = tp.t0; ti.u0 = tp.u0; ti.us = tp.us;
        }
    }
    __syncthreads();
    // Accumulator register 4j+i of row block 2*lt + m2 is row r = 32 m2 + 8j + 4 hb + i of lattice tile lt, hidden column l32: in an 8 x 8
    // tile frame 4 m2 + j, label 4 hb + i; in a 16 x 4 tile frame 8 m2 + 2j + hb, label i.  One copy of the loop nest per shape.
    auto tile_epilogue = [&](auto lt_tag) {
        constexpr int lt = decltype(lt_tag)::value;
        const int t4 = HALF ? wm : wm * 2 + lt;
        const TileInfo ti = info[t4];
        const int s = __builtin_amdgcn_readfirstlane(ti.s), us = __builtin_amdgcn_readfirstlane(ti.us);
        const bool by_sum = __builtin_amdgcn_readfirstlane(ti.far[0] | ti.far[1]) != 0;
        if (s < 0) return;
        float* d_enc = g.d_enc + (size_t)s * g.pr.T_max * H;
        float* d_prd = g.d_pred + (size_t)s * (g.pr.U_max + 1) * H;
        const float* er = ex + (t4 * Z_ROWS) * Z_EP;
        auto reduce = [&](auto wide_tag, auto sum_tag) {
            constexpr bool WIDE = decltype(wide_tag)::value, SUM = decltype(sum_tag)::value;
            constexpr int TH = WIDE ? 8 : 16;
            const int ulb = WIDE ? 4 * hb : 0;              // first of this lane's four label positions
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                const int hc = wn * 64 + nt * 32 + l32, h = n0 + hc;        // column inside the tile, hidden column
                float qv[4], pu[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int i = 0; i < 4; ++i) qv[i] = er[(TH + ulb + i) * Z_EP + hc];
#pragma unroll
                for (int m2 = 0; m2 < 2; ++m2) {
                    float se[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float ev = er[(WIDE ? 4 * m2 + j : 8 * m2 + 2 * j + hb) * Z_EP + hc];
                        se[j] = 0.0f;
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            float w;                        // (1 - z^2) / 4
                            if (SUM) {
                                const float z = fast_tanh(ev + qv[i]);
                                w = fmaf(-0.25f * z, z, 0.25f);
                            } else {
                                const float r = __builtin_amdgcn_rcpf(fmaf(ev, qv[i], 1.0f));
                                w = fmaf(-r, r, r);
                            }
                            const float d = acc[2 * lt + m2][nt][4 * j + i];
                            se[j] = fmaf(d, w, se[j]);
                            pu[i] = fmaf(d, w, pu[i]);
                        }
                    }
                    if (WIDE) {
#pragma unroll
                        for (int j = 0; j < 4; j += 2) {    // a frame's eight labels lie in both lane halves; each half adds one frame
                            const float s0 = both_halves_sum(se[j]), s1 = both_halves_sum(se[j + 1]);
                            const int t = ti.t0 + 4 * m2 + j + hb;
                            if (t < ti.T) atomicAdd(&d_enc[(size_t)t * H + h], 4.0f * (hb ? s1 : s0));
                        }
                    } else {
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const int t = ti.t0 + 8 * m2 + 2 * j + hb;
                            if (t < ti.T) atomicAdd(&d_enc[(size_t)t * H + h], 4.0f * se[j]);
                        }
                    }
                }
                if (WIDE) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int u = ti.u0 + 4 * hb + i;
                        if (u <= ti.U) atomicAdd(&d_prd[(size_t)u * H + h], 4.0f * pu[i]);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 4; i += 2) {        // a label's sixteen frames lie in both lane halves; each half adds one label
                        const float s0 = both_halves_sum(pu[i]), s1 = both_halves_sum(pu[i + 1]);
                        const int u = ti.u0 + i + hb;
                        if (u <= ti.U) atomicAdd(&d_prd[(size_t)u * H + h], 4.0f * (hb ? s1 : s0));
                    }
                }
            }
        };
        if (us == 3) {
            if (by_sum) reduce(std::true_type{}, std::true_type{});
            else reduce(std::true_type{}, std::false_type{});
        } else {
            if (by_sum) reduce(std::false_type{}, std::true_type{});
            else reduce(std::false_type{}, std::false_type{});
        }
    };
    tile_epilogue(std::integral_constant<int, 0>{});
    if constexpr (!HALF) tile_epilogue(std::integral_constant<int, 1>{});
}

// L: workgroup of the v_splits * per_part
template <int WAVES>
__device__ __forceinline__ void dz_workgroup(const DzArgs& g, unsigned char* dz_smem, int L) {
    // XCD-aware order (ids that agree modulo 8 share an L2): the hidden tiles of one row tile are
    // neighbours on one XCD, so the rows of dH are fetched from HBM once.
    const int vs = L / g.per_part;
    L -= vs * g.per_part;
    const int xcd = L & 7, q = L >> 3;
    const int by = q % g.n_tiles, bx = xcd + 8 * (q / g.n_tiles);
    // slots of the chunk that hold a tile: all of the launch's, or what is left of the group's list
    int n_slots = g.tile1 - g.tile0;
    if (g.at.active) {
        const int left = *g.at.n_active - g.at.cbase;
        n_slots = left < n_slots ? left : n_slots;
    }
    if (bx * (WAVES / 2) >= n_slots) return;          // (uniform per workgroup)
    const int n0 = by * g.edge;
    if (g.edge < ZT || n0 + 128 >= g.pr.H) dz_tile<true, WAVES>(g, dz_smem, bx, n0, n_slots, vs);
    else dz_tile<false, WAVES>(g, dz_smem, bx, n0, n_slots, vs);
}

template <int WAVES>
__global__ __launch_bounds__(64 * WAVES, 2) void k_gemm_dz256(DzArgs g) {
    extern __shared__ __align__(16) unsigned char dz_smem[];   // [stages] x { A, B }
    dz_workgroup<WAVES>(g, dz_smem, blockIdx.x);
}

// Both GEMMs of a chunk: dW's workgroups, then dz's (they share nothing but what they read: dH).  The rule and what it gives: plan.h.
template <bool BY_TILE>
__global__ __launch_bounds__(512) void k_gemm_dz_dw(DzArgs z, DwArgs w, int nw) {
    extern __shared__ __align__(16) unsigned char smem[];
    if ((int)blockIdx.x < nw) dw_workgroup<BY_TILE>(w, smem, blockIdx.x);
    else dz_workgroup<8>(z, smem, blockIdx.x - nw);
}

constexpr size_t dz_smem_bytes(int WAVES) { return (size_t)z_stages(WAVES) * z_stage_bytes(WAVES); }

DzArgs dz_args(const DzForm& f, const Problem& pr, const void* Wq, const SampleTable& st, int tile0, int tile1, const void* dH,
               float* d_enc, float* d_pred, const ActiveTiles& at, int waves) {
    const int m_tiles = (tile1 - tile0 + waves / 2 - 1) / (waves / 2), n_tiles = (pr.H + f.edge - 1) / f.edge;
    return DzArgs{(const unsigned char*)dH, (const unsigned char*)Wq, pr, st, tile0, tile1, d_enc, d_pred, n_tiles, f.edge, f.vs,
                  (m_tiles + 7) / 8 * 8 * n_tiles, at};
}

}  // namespace

template <int WAVES>
static hipError_t launch_dz(const DzArgs& g, hipStream_t stream) {
    constexpr size_t smem = dz_smem_bytes(WAVES);
    static bool configured = false;
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_dz256<WAVES>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)smem);
        if (e != hipSuccess) return e;
        configured = true;
    }
    k_gemm_dz256<WAVES><<<dim3((unsigned)(g.v_splits * g.per_part)), dim3(64 * WAVES), smem, stream>>>(g);
    return hipGetLastError();
}

hipError_t launch_gemm_dz_bf16(const Problem& pr, const void* Wq, const SampleTable& st, int tile0, int tile1, const void* dH,
                               float* d_enc, float* d_pred, const ActiveTiles& at, hipStream_t stream) {
    const int n = tile1 - tile0;
    if (n <= 0) return hipSuccess;
    if (pr.V % (4 * ZK) != 0) return hipErrorInvalidValue;
    const int waves = dz_waves(pr.H, pr.V);
    const DzArgs g = dz_args(dz_alone(pr.H, pr.V, n), pr, Wq, st, tile0, tile1, dH, d_enc, d_pred, at, waves);
    return waves == 4 ? launch_dz<4>(g, stream) : launch_dz<8>(g, stream);
}

hipError_t launch_gemm_dz_dw_bf16(const Problem& pr, const void* Wq, const SampleTable& st, int tile0, int tile1, const void* Z,
                                  const void* dH, float* d_enc, float* d_pred, int splits, int first, float* slots, float* db,
                                  const ActiveTiles& at, hipStream_t stream) {
    const long long rows = (long long)(tile1 - tile0) * JT_ROWS;
    if (rows <= 0 || splits <= 0 || pr.V % (4 * ZK) != 0) return hipErrorInvalidValue;
    const DzArgs z = dz_args(dz_one_grid(pr.H, pr.V, tile1 - tile0, splits), pr, Wq, st, tile0, tile1, dH, d_enc, d_pred, at, 8);
    const DwArgs w = dw_args(pr.H, pr.V, rows, splits, first, Z, dH, slots, db, at);
    constexpr size_t smem = dz_smem_bytes(8) > DW_SMEM ? dz_smem_bytes(8) : DW_SMEM;
    static bool configured = false;
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_dz_dw<false>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_dz_dw<true>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
        configured = true;
    }
    const int nw = dw_grid(pr.H, pr.V, splits);
    const dim3 grid((unsigned)(nw + z.v_splits * z.per_part));
    if (at.active && at.slot_tile0 >= 0) k_gemm_dz_dw<true><<<grid, dim3(512), smem, stream>>>(z, w, nw);
    else k_gemm_dz_dw<false><<<grid, dim3(512), smem, stream>>>(z, w, nw);
    return hipGetLastError();
}

}  // namespace rnnt
