// bf16 path (gfx950): kept scores -> score gradients, and the dW_out GEMM over the chunk buffers (layout: device_common.h).
//
// MFMA operand layouts (v_mfma_f32_32x32x16_bf16, D = A B + C, wave64):
//   A (32 x 16): lane l holds row l%32, k = 8*(l/32) .. +7        (8 bf16)
//   B (16 x 32): lane l holds column l%32, k = 8*(l/32) .. +7     (8 bf16)
//   C/D (32x32): lane l holds column l%32; register 4*j+i is row 8*j + 4*(l/32) + i
#include "device_common.h"
#include "gemm_dw_tile.h"

namespace rnnt {

// ------------------------------------------------------------------------------------------------
// Kept scores -> score gradients, in place (f^W_4 without the second score GEMM):
//   dh[r,v] = exp(t[r,v] + m[r, v/64] - lse[r] + ln gamma[r]) - [v = blank] B[r] - [v = y_u] Y[r].
// A wave takes half a lattice tile (32 rows, a row per lane and its partner); the forward kernel left a block of 32 entries as
// 2 KiB (register by register of its accumulators), which become the two bf16 fragments of the same entries.  HBM bound
// (4 bytes per score); four waves of a workgroup share a half's vocabulary.
// ------------------------------------------------------------------------------------------------
struct KeptArgs {
    Problem pr;
    SampleTable st;
    LatticeState ls;
    int tile0, tile1;
    unsigned char* kept;
    const float* kept_max;
    ActiveTiles at;
};
__global__ __launch_bounds__(256) void k_kept_to_dh(KeptArgs a) {
    typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
    const int V = a.pr.V;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, hb = lane >> 5;
    const int half = blockIdx.x & 1;
    int tile = a.tile0 + (int)(blockIdx.x >> 1);
    if (a.at.active) {
        // listed tiles only (uniform per workgroup); the kept scores of a tile lie at its position in the launch
        const int ci = a.at.cbase + (int)(blockIdx.x >> 1);
        if (ci >= *a.at.n_active) return;
        tile = a.at.active[a.at.group_tile0 + ci];
    }
    const int slot = tile - a.tile0;
    const TilePos tp = locate_tile(a.st, tile);
    const int r = 32 * half + l32, t = tp.t0 + (r >> tp.us), u = tp.u0 + (r & (tp.uw - 1)), b = tp.s;
    const int lab = (t < tp.T && u < tp.U) ? a.pr.labels[(size_t)b * a.pr.U_max + u] : -1;
    float g = RNNT_NEG_INF, vB = 0.0f, vY = 0.0f;
    if (t < tp.T && u <= tp.U) {
        const long long idx = (a.st.row_off[b] - a.ls.row_base) + lattice_index(tp.T, tp.U + 1, t, u);
        const RowDh rd = row_score_gradient(a.ls, idx, t, u, tp.T, tp.U, b, lab, a.pr.blank);
        g = rd.g;
        vB = rd.at_blank;
        vY = rd.at_label;
    }
    unsigned char* base = a.kept + (size_t)(slot * 2 + half) * chunk_block_bytes(V);
    const float* mx = a.kept_max + (size_t)slot * (V / 64) * 64 + r;
    // pairs of blocks (64 entries, 4 KiB): wave w takes pairs w, w + 4, ...; the next pair's loads run ahead
    const int np = V / 64;
    u32x4 nx[4];
    float mn = 0.0f;
    auto fetch = [&](int p) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            nx[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(base + (size_t)p * 4096 + i * 1024 + lane * 16));
        mn = mx[(size_t)p * 64];
    };
    if (wave < np) fetch(wave);
    for (int p = wave; p < np; p += 4) {
        u32x4 cur[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) cur[i] = nx[i];
        const float e = fmaf(mn, LOG2E_F, g);
        if (p + 4 < np) fetch(p + 4);
#pragma unroll
        for (int blk = 0; blk < 2; ++blk) {
            f32x16 d;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const f16x8 tv = __builtin_bit_cast(f16x8, cur[2 * blk + h]);
#pragma unroll
                for (int i = 0; i < 8; ++i) d[8 * h + i] = __builtin_amdgcn_exp2f(fmaf((float)tv[i], LOG2E_F, e));
            }
            const int vbase = p * 64 + blk * 32;
            int relb = a.pr.blank - vbase, rely = lab - vbase;
            if (__any((unsigned)rely < 32u) || (unsigned)relb < 32u) {
                relb -= 4 * hb;
                rely -= 4 * hb;
                asm volatile("" : "+v"(relb), "+v"(rely)::"memory");
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int vloc = 8 * (i >> 2) + (i & 3);
                    if (vloc == relb) d[i] = vB;
                    if (vloc == rely) d[i] = vY;
                }
            }
#pragma unroll
            for (int h = 0; h < 2; ++h)
                __builtin_nontemporal_store(fragment_from_scores(d, h),
                                            reinterpret_cast<u32x4*>(base + (size_t)p * 4096 + (2 * blk + h) * 1024 +
                                                                     frag_granule(lane, h)));
        }
    }
}

hipError_t launch_kept_to_dh_bf16(const Problem& pr, const SampleTable& st, const LatticeState& ls, int tile0, int tile1,
                                  void* kept, const float* kept_max, const ActiveTiles& at, hipStream_t stream) {
    const int n = tile1 - tile0;
    if (n <= 0) return hipSuccess;
    const KeptArgs a{pr, st, ls, tile0, tile1, (unsigned char*)kept, kept_max, at};
    k_kept_to_dh<<<dim3((unsigned)n * 2), dim3(256), 0, stream>>>(a);
    return hipGetLastError();
}

template <bool BY_TILE>
__global__ __launch_bounds__(512) void k_gemm_dw256(DwArgs g) {
    extern __shared__ __align__(16) unsigned char dw_smem[];
    dw_workgroup<BY_TILE>(g, dw_smem, blockIdx.x);
}

hipError_t launch_gemm_dw_bf16(int H, int V, long long rows, int splits, int first, const void* Z, const void* dH,
                               float* slots, float* db, const ActiveTiles& at, hipStream_t stream) {
    if (rows <= 0 || splits <= 0 || rows % WK != 0) return hipErrorInvalidValue;
    const DwArgs g = dw_args(H, V, rows, splits, first, Z, dH, slots, db, at);
    static bool configured = false;
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_dw256<false>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)DW_SMEM);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_dw256<true>),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)DW_SMEM);
        if (e != hipSuccess) return e;
        configured = true;
    }
    const dim3 grid((unsigned)dw_grid(H, V, splits));
    if (at.active && at.slot_tile0 >= 0) k_gemm_dw256<true><<<grid, dim3(512), DW_SMEM, stream>>>(g);
    else k_gemm_dw256<false><<<grid, dim3(512), DW_SMEM, stream>>>(g);
    return hipGetLastError();
}

// dW (+)= sum over the splits of the slots.  One thread per float4 of a tile's slot (four consecutive
// hidden rows of one vocabulary column), decoded back from the accumulator order of k_gemm_dw256.
__global__ __launch_bounds__(256) void k_dw_reduce(const f32x4* __restrict__ slots, float* __restrict__ dW, int H, int V,
                                                   int mt_tiles, int ntile, int splits, int accumulate) {
    const int tile = blockIdx.y;
    const int e = blockIdx.x * 256 + threadIdx.x;          // 0 .. 16383
    const int bm = tile % mt_tiles, bn = tile / mt_tiles;
    const int wave = e >> 12, mt = (e >> 10) & 3, nt = (e >> 8) & 3, j = (e >> 6) & 3, lane = e & 63;
    const int wm_cols = bm * WT + 128 >= H ? 64 : 128;     // hidden columns of a wave: half tile, whole tile
    if (mt * 32 >= wm_cols) return;
    f32x4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int s = 0; s < splits; ++s) sum += slots[((size_t)s * ntile + tile) * 16384 + e];
    const int m = bm * WT + (wave >> 1) * wm_cols + mt * 32 + 8 * j + 4 * (lane >> 5);
    const int n = bn * WT + (wave & 1) * 128 + nt * 32 + (lane & 31);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float* q = dW + (size_t)(m + i) * V + n;
        *q = accumulate ? *q + sum[i] : sum[i];
    }
}

hipError_t launch_dw_reduce(int H, int V, int splits, const float* slots, float* dW, int accumulate,
                            hipStream_t stream) {
    const int mt = (H + WT - 1) / WT, nt = V / WT;
    k_dw_reduce<<<dim3(64, (unsigned)(mt * nt)), dim3(256), 0, stream>>>((const f32x4*)slots, dW, H, V, mt, mt * nt, splits,
                                                                      accumulate);
    return hipGetLastError();
}

}  // namespace rnnt
