// The dW GEMM's workgroup (device code): used by its own launch and by the one it shares with the dz GEMM.
#pragma once
#include "device_common.h"

namespace rnnt {

namespace {

constexpr int JT_ROWS = 64;       // rows of a lattice tile

// ------------------------------------------------------------------------------------------------
// dW += Z^T dH and db += column sums of dH (Alg. 1 line 8) as one split-K GEMM with 256x256 tiles.
// 512 threads = 8 waves in 2 (hidden) x 4 (vocabulary), two per SIMD; each wave owns 128 x 64 = 4 x 2
// accumulator tiles, so that a k16-step reads 6 fragments from LDS for 8
// MFMAs and every byte of a stage feeds 128 flops.  Both operands, Z [rows,H] and dH [rows,V], lie in 1 KiB fragments of
// 32 rows x 16 columns (device_common.h), eight columns of a row together, so the 256 columns of a tile are 16 KiB in one piece, and the
// contraction index (the chunk's rows) is the slow one inside a fragment.  Stages of 32 rows travel global -> LDS asynchronously (global_load_lds, no registers), five stages deep, and lie
// in LDS as in memory; MFMA fragments, which need 8 consecutive rows of one column per lane,
// come from the transposing LDS read (ds_read_b64_tr_b16): within 16 lanes, lane 4j+c supplies 4
// columns of row j and lane i receives rows 0..3 of column i.  The fragments' row order puts the 16 rows a 32-lane read touches
// into different banks.
// The workgroups of the first hidden-tile row also sum their B fragments over the rows (the bias
// gradient) with packed bf16 dot products against ones.
// What bounds it: of 7.45 ms (H = 512, V = 1024, 13 M nodes, 0.58 of the tiles) the MFMAs alone take 5.4 (1.6 PFLOP/s, power), the copies 1.2, the sums
// of the chunks before 0.4, the LDS reads 0.4.  Four waves of 128 x 128 with a stage less in flight: 8.05; eight with a stage less 7.7; V = 8192, 3.7 M nodes 20.2 ms
// against 18.6.
// ------------------------------------------------------------------------------------------------
constexpr int WT = 256;       // tile edge
constexpr int WK = 32;        // rows per pipeline stage
constexpr int WST = 5;        // pipeline stages (LDS buffers)

struct DwArgs {
    const unsigned char* Z;
    const unsigned char* dH;
    long long K, k_per_split;
    float* slots;    // [splits][tiles][4 waves][4][4][4][64 lanes] float4: partial sums, accumulator layout
    float* db;
    int first;       // overwrite the slot instead of adding to it
    int H, V;
    int mt, nt;      // output tiles along H and V
    int splits;
    ActiveTiles at;  // at.active set: the chunk holds 64 * (*at.n_active - at.cbase) rows if that is less than K
};
// BY_TILE (at.slot_tile0 >= 0): the 64 rows of the list's entry i lie in slot (tile - at.slot_tile0) of both chunk
// buffers instead of slot i.  A stage of 32 rows lies inside one slot, so only the first row of a stage changes;
// the list entry of a stage is read (a scalar load) one loop iteration before the stage's copies are issued.

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ bf16x8 lds_read_tr_frag(const unsigned char* lo_p, const unsigned char* hi_p) {
    // rows +0..3 and +4..7 of this lane's column
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(lo_p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(hi_p));
    const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}

// HALF: the last hidden tile of 128 columns; the waves stand 2 (hidden) x 4 as for a whole tile, each 64 x 64
template <bool BY_TILE, bool HALF>
__device__ __forceinline__ void dw_tile(const DwArgs& g, unsigned char* dw_smem, int split, int tile) {
    constexpr int MT = HALF ? 2 : 4;                  // 32-column blocks of the hidden side per wave
    constexpr int AF = HALF ? 1 : 2;                  // fragments of Z a wave copies per stage
    constexpr int DMAS = AF + 2;                      // copies per wave and stage
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63, l32 = lane & 31, hb = lane >> 5;
    const int wm = wave >> 2, wn = wave & 3;
    const int ntile = g.mt * g.nt;
    const int bm = tile % g.mt, bn = tile / g.mt;
    const long long m0 = (long long)bm * WT, n0 = (long long)bn * WT;
    long long K = g.K, k_per_split = g.k_per_split;
    if (g.at.active) {
        long long act = (long long)*g.at.n_active - g.at.cbase;
        act = act < 0 ? 0 : act * JT_ROWS;
        if (act < K) {
            K = act;
            const long long per = (K + g.splits - 1) / g.splits;
            k_per_split = (per + WK - 1) / WK * WK;
        }
    }
    const long long ks = (long long)split * k_per_split;
    const long long ke = ks + k_per_split < K ? ks + k_per_split : K;
    const bool do_db = (bm == 0) && (wm == 0);
    constexpr unsigned STAGE_BYTES = 2u * WK * WT * 2u;
    constexpr unsigned OPER_BYTES = (unsigned)WK * WT * 2u;
    const unsigned smem_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)dw_smem;

    // global -> LDS: one DMA instruction moves one fragment; wave w moves fragments 2 w, 2 w + 1 of dH
    // and AF w .. of Z.  Everything but
    // the lane's 16 bytes is wave-uniform and lives in scalar registers, so issuing a DMA costs no vector instruction.
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    const size_t ZB = chunk_block_bytes(g.H), DB = chunk_block_bytes(g.V);   // bytes of a block of 32 rows
    const unsigned char* Zs = g.Z + (size_t)(ks / WK) * ZB + (size_t)(m0 / 16 + AF * wv) * 1024;
    const unsigned char* Ds = g.dH + (size_t)(ks / WK) * DB + (size_t)(n0 / 16 + 2 * wv) * 1024;
    const unsigned dst_a = smem_base + (unsigned)(AF * wv) * 1024u, dst_b = smem_base + OPER_BYTES + (unsigned)(2 * wv) * 1024u;
    const unsigned lane_b = (unsigned)lane * 16u;
    // Block of 32 rows of stage gstep of the split, relative to the split's first; `entry` is the list entry of the stage's slot
    // (BY_TILE only).
    // (read through the constant address space: the list was written before this launch, and only such a load
    // becomes a scalar load that stays clear of the vector-memory counter the copies below are tracked with)
    typedef const int __attribute__((address_space(4))) * list_ptr;
    const list_ptr lst = BY_TILE ? (list_ptr)(g.at.active + g.at.group_tile0 + g.at.cbase) : nullptr;
    auto stage_entry = [&](long long gstep) { return BY_TILE ? lst[(ks + gstep * WK) >> 6] : 0; };
    auto stage_block = [&](long long gstep, int entry) -> long long {
        if (!BY_TILE) return gstep;
        return ((long long)(entry - g.at.slot_tile0) << 1) + (((ks + gstep * WK) >> 5) & 1) - ks / WK;
    };
    // Copies of dH (j = 0) or Z (1) of the stage whose rows are block blk, into LDS buffer buf (in pairs: M0 and its wait state once)
    auto issue_pair = [&](long long blk, unsigned buf, auto j_tag) {
        constexpr int j = decltype(j_tag)::value;
        if constexpr (j == 0) lds_dma16_pair<0>(Ds + blk * (long long)DB, lane_b, dst_b + buf * STAGE_BYTES);
        else if constexpr (HALF) lds_dma16_s(Zs + blk * (long long)ZB, lane_b, dst_a + buf * STAGE_BYTES);
        else lds_dma16_pair<0>(Zs + blk * (long long)ZB, lane_b, dst_a + buf * STAGE_BYTES);
    };
    // fragment addresses: lane = 16 g + 4 j + c supplies row 8*(g/2) + j, columns 16*(g%2) + 4c .. +3 of a 32-column tile: granule
    // (row, c/2) of fragment 2 * tile + g % 2, at position 32 (c/2) + (row ^ 4 (2 (g % 2) + c/2))
    const int fg = lane >> 4, fj = (lane >> 2) & 3, fc = lane & 3;
    const int fswz = 4 * (2 * (fg & 1) + (fc >> 1));
    const unsigned fbase = (unsigned)((fg & 1) * 1024 + (fc >> 1) * 512 + (fc & 1) * 8);
    const unsigned f_lo = fbase + (unsigned)(((8 * (fg >> 1)) ^ fswz) + fj) * 16u;
    const unsigned f_hi = fbase + (unsigned)(((8 * (fg >> 1) + 4) ^ fswz) + fj) * 16u;
    const unsigned a_lo = f_lo + (unsigned)(wm * MT) * 2048u, a_hi = f_hi + (unsigned)(wm * MT) * 2048u;
    const unsigned b_lo = f_lo + OPER_BYTES + (unsigned)wn * 4096u, b_hi = f_hi + OPER_BYTES + (unsigned)wn * 4096u;

    f32x16 acc[MT][2];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x16{0};
    float dbs[2] = {0.0f, 0.0f};
    const bf16x2 ones = {(bf16_t)1.0f, (bf16_t)1.0f};

    const long long nsteps = ke > ks ? (ke - ks) / WK : 0;   // a split beyond the chunk still writes its slot
    if (nsteps == 0 && !g.first) return;                     // ... unless the slot already holds a sum: nothing to add
    static_assert(WK == 32, "the loop below is written for two k16-steps per stage");
    bf16x8 fa[2][MT], fb[2][2];
    auto read_frags = [&](int set, unsigned buf, int kk) {
        const unsigned char* st = dw_smem + buf * STAGE_BYTES + kk * 256;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) fa[set][mt] = lds_read_tr_frag(st + a_lo + mt * 2048, st + a_hi + mt * 2048);
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) fb[set][nt] = lds_read_tr_frag(st + b_lo + nt * 2048, st + b_hi + nt * 2048);
    };
    // The 2 MT MFMAs of one k16-step (register set `set`); behind each of the first MT + 2, one fragment of the
    // following k16-step is read into the other set.  An MFMA keeps the matrix pipe busy for 32 clocks but
    // the issue port only briefly: the reads go out in its shadow.  Behind two of the last four of a stage's second step go the copies of a later
    // stage.
    auto multiply = [&](auto set_tag, unsigned next_buf, int next_kk, long long dma_block, unsigned dma_buf) {
        constexpr int set = decltype(set_tag)::value;
        const unsigned char* st = dw_smem + next_buf * STAGE_BYTES + next_kk * 256;
        static_for<0, 2 * MT>([&](auto idx_tag) {
            constexpr int idx = decltype(idx_tag)::value, mt = idx >> 1, nt = idx & 1;
            acc[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][mt], fb[set][nt], acc[mt][nt], 0, 0, 0);
            if constexpr (idx < MT) fa[set ^ 1][idx] = lds_read_tr_frag(st + a_lo + idx * 2048, st + a_hi + idx * 2048);
            else if constexpr (idx < MT + 2)
                fb[set ^ 1][idx - MT] = lds_read_tr_frag(st + b_lo + (idx - MT) * 2048, st + b_hi + (idx - MT) * 2048);
            if constexpr (set == 1 && idx >= 2 * MT - 4 && idx % 2 == 0)
                issue_pair(dma_block, dma_buf, std::integral_constant<int, (idx - (2 * MT - 4)) / 2>{});
            __builtin_amdgcn_sched_barrier(0);
        });
        if (do_db) {
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int q2 = 0; q2 < 4; ++q2) {
                    const bf16x2 pr2 = {fb[set][nt][2 * q2], fb[set][nt][2 * q2 + 1]};
                    dbs[nt] = __builtin_amdgcn_fdot2_f32_bf16(pr2, ones, dbs[nt], false);
                }
        }
    };
    // Five stages in flight before the first one is consumed (DMAS copies per wave and stage).  The hand-over to the next stage (wait
    // for this wave's copies, then for everyone's) sits in the middle of a stage; there every wave has read all its fragments of the
    // present one, whose buffer may be refilled.  Beyond the last stage the pipeline keeps re-loading the
    // last one into buffers nobody reads any more, which keeps the loop free of branches and the number of
    // copies in flight constant.
    if (nsteps > 0) {
        const long long last = nsteps - 1;
#pragma unroll
        for (int s5 = 0; s5 < WST; ++s5) {
            const long long gs = s5 < last ? s5 : last;
            const long long blk = stage_block(gs, stage_entry(gs));
            static_for<0, 2>([&](auto j) { issue_pair(blk, (unsigned)s5, j); });
        }
        int entry_ahead = stage_entry(WST < last ? WST : last);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((WST - 1) * DMAS) : "memory");
        __syncthreads();
        read_frags(0, 0, 0);
        unsigned buf = 0;                               // of stage it
        for (long long it = 0; it < nsteps; ++it) {
            const unsigned next = buf + 1 == WST ? 0 : buf + 1;
            __builtin_amdgcn_s_waitcnt(WAIT_LGKM0);     // set 0 landed (read behind the first MFMAs of the step before)
            __builtin_amdgcn_sched_barrier(0);
            const long long dma_block = stage_block(it + WST < last ? it + WST : last, entry_ahead);
            entry_ahead = stage_entry(it + WST + 1 < last ? it + WST + 1 : last);      // arrives during this iteration
            multiply(std::integral_constant<int, 0>{}, buf, 1, 0, 0);
            __builtin_amdgcn_s_waitcnt(WAIT_LGKM0);     // set 1 landed
            // stage it + 1 landed; the later ones stay in flight
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((WST - 2) * DMAS) : "memory");
            __syncthreads();
            __builtin_amdgcn_sched_barrier(0);
            multiply(std::integral_constant<int, 1>{}, next, 0, dma_block, buf);
            buf = next;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // no copy may land after the workgroup has ended
    }
    // Partial sums go to this workgroup's own slot, in accumulator order (one 16-byte store per lane
    // and four accumulator rows): no atomics, and the same workgroup adds the next chunk's product.
    {
        f32x4* slot = reinterpret_cast<f32x4*>(g.slots) +
                      (((size_t)split * ntile + tile) * 4 + (wm * 2 + (wn >> 1))) * (size_t)(4 * 4 * 4 * 64) + (wn & 1) * (2 * 4 * 64) + lane;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    f32x4 v = {acc[mt][nt][4 * j], acc[mt][nt][4 * j + 1], acc[mt][nt][4 * j + 2],
                               acc[mt][nt][4 * j + 3]};
                    f32x4* q = slot + ((mt * 4 + nt) * 4 + j) * 64;
                    if (!g.first) v += *q;
                    *q = v;
                }
    }
    if (do_db) {
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
            float v = dbs[nt] + __shfl_xor(dbs[nt], 32, 64);
            if (hb == 0) atomicAdd(&g.db[n0 + wn * 64 + nt * 32 + l32], v);
        }
    }
}

// Workgroup ids are dealt round-robin to the 8 XCDs, each with its own L2.  An XCD takes a contiguous range of the (split, tile)
// pairs, so the output tiles that read the same rows of Z and dH run side by side on one XCD (or on neighbours) and the rows
// come from HBM once or little more.  Whole tiles go first, the half ones (H not a multiple of 256) fill the gaps of the last round.
// L: workgroup of the dw_grid.
template <bool BY_TILE>
__device__ __forceinline__ void dw_workgroup(const DwArgs& g, unsigned char* dw_smem, int L) {
    const int fm = g.H / WT, full = fm * g.nt, half = (g.mt - fm) * g.nt;     // whole and half tiles of a split
    const int xcd = L & 7, q = L >> 3;
    const int nf = g.splits * full, nh = g.splits * half, f8 = (nf + 7) >> 3, h8 = (nh + 7) >> 3;
    if (q < f8) {
        const int w = xcd * f8 + q;
        if (w >= nf) return;
        const int t = w % full;
        dw_tile<BY_TILE, false>(g, dw_smem, w / full, t / fm * g.mt + t % fm);
    } else {
        const int w = xcd * h8 + (q - f8);
        if (w >= nh) return;
        dw_tile<BY_TILE, true>(g, dw_smem, w / half, w % half * g.mt + fm);
    }
}
inline int dw_grid(int H, int V, int splits) {
    const int nt = V / WT, nf = H / WT * nt * splits, nh = (H + WT - 1) / WT * nt * splits - nf;
    return 8 * ((nf + 7) / 8 + (nh + 7) / 8);
}
inline DwArgs dw_args(int H, int V, long long rows, int splits, int first, const void* Z, const void* dH, float* slots, float* db,
                      const ActiveTiles& at) {
    DwArgs g{(const unsigned char*)Z, (const unsigned char*)dH, rows, 0, slots, db, first, H, V, (H + WT - 1) / WT, V / WT, splits, at};
    // a split past the end of a short chunk only touches its slot
    const long long per = (rows + splits - 1) / splits;
    g.k_per_split = (per + WK - 1) / WK * WK;
    return g;
}
constexpr size_t DW_SMEM = (size_t)WST * 2 * WK * WT * 2;      // [WST] x { A [WK][256], B [WK][256] } bf16

}  // namespace

}  // namespace rnnt
