// Device helpers shared by the HIP kernels of this library (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "kernels.h"

namespace rnnt {

constexpr float LOG2E_F = 1.4426950408889634f;
constexpr float LN2_F = 0.6931471805599453f;
#define RNNT_NEG_INF (-__builtin_huge_valf())
// s_waitcnt operand (gfx9 encoding: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt[15:14]) that waits for
// every outstanding LDS / scalar-memory operation of the wave and for nothing else.
constexpr int WAIT_LGKM0 = 0xC07F;

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Largest s in [lo, hi) with off[s] <= x  (off is non-decreasing, off[lo] <= x < off[hi]).
template <typename T>
__device__ __forceinline__ int find_segment(const T* __restrict__ off, int lo, int hi, T x) {
    while (hi - lo > 1) {
        int mid = (lo + hi) >> 1;
        if (off[mid] <= x) lo = mid; else hi = mid;
    }
    return lo;
}

// Position of a lattice tile: sample, first frame, first label position, and the sample's tile shape
// (uw = 8 or 4 label positions, us = log2 uw; row r of the tile is frame t0 + (r >> us), label u0 + (r & (uw-1))).
struct TilePos {
    int s, T, U, t0, u0, uw, us;
};

__device__ __forceinline__ TilePos locate_tile(const SampleTable& st, int tile) {
    TilePos p;
    p.s = st.tile_sample[tile];
    p.T = st.T[p.s];
    p.U = st.U[p.s];
    p.uw = tile_label_width(p.T, p.U);
    p.us = p.uw == 8 ? 3 : 2;
    const int tiles_u = (p.U + p.uw) >> p.us;     // ceil((U+1)/uw)
    const int lt = tile - st.tile_off[p.s];
    const int tb = lt / tiles_u;
    p.t0 = tb * (64 >> p.us);
    p.u0 = (lt - tb * tiles_u) << p.us;
    return p;
}

// tanh through one exp and one reciprocal; absolute error ~1e-7, saturates cleanly at +-1.
__device__ __forceinline__ float fast_tanh(float x) {
    float e = __builtin_amdgcn_exp2f(x * (2.0f * LOG2E_F));
    return 1.0f - 2.0f * __builtin_amdgcn_rcpf(1.0f + e);
}

// Eight joint activations z = tanh(e + q), rounded to bf16.
__device__ __forceinline__ bf16x8 joint_tanh8(bf16x8 e, bf16x8 q) {
    bf16x8 z;
#pragma unroll
    for (int j = 0; j < 8; ++j) z[j] = (bf16_t)fast_tanh((float)e[j] + (float)q[j]);
    return z;
}

__device__ __forceinline__ float2 emissions(float blank, float label) {
    // (comparisons that keep NaN)
    return make_float2(blank < EMISSION_FLOOR ? EMISSION_FLOOR : blank, label < EMISSION_FLOOR ? EMISSION_FLOOR : label);
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// Posterior weights of one lattice node (f^W_4): ln gamma, and the occupation of its blank and
// label transitions.  alpha/beta/lnP carry the per-sample emission offset `shift`, which cancels.
// With per-sample loss weights all three are those of w_s * loss_s.
struct RowPost {
    float log_gamma, Bk, Yk;
};
__device__ __forceinline__ RowPost row_posteriors(const LatticeState& ls, long long idx, int t, int u,
                                                   int T, int U, int s) {
    const float a = ls.alpha[idx], lnP = ls.lnP[s], c = ls.shift[s];
    RowPost r;
    r.log_gamma = a + ls.beta[idx] - lnP;
    const float2 em = ls.em[idx];
    const float ab = a + em.x + c - lnP;
    const float* __restrict__ next = ls.beta + idx + next_diagonal_step(T, U + 1, t + u);
    if (t < T - 1) r.Bk = __expf(ab + next[0]);
    else r.Bk = (u == U) ? __expf(ab) : 0.0f;
    r.Yk = (u < U) ? __expf(a + em.y + c - lnP + next[1]) : 0.0f;
    if (ls.weight) {
        // gradients of sum_b w_b loss_b: every posterior weight of sample s is scaled by w_s >= 0; one of weight 0 contributes nothing, whatever its
        // posteriors are (without a possible alignment they are infinite)
        const float w = ls.weight[s];
        r.log_gamma = w > 0.0f ? r.log_gamma + __logf(w) : RNNT_NEG_INF;
        r.Bk = w > 0.0f ? r.Bk * w : 0.0f;
        r.Yk = w > 0.0f ? r.Yk * w : 0.0f;
    }
    return r;
}

// What turns a row of scores h into its score gradient dh = gamma softmax - posteriors (f^W_4): dh = exp2(h log2 e + g)
// except at the blank and the label entry, whose final values follow from the stored log-probabilities (so the per-element path
// needs no indicator logic; the owning lane overwrites those two entries).
struct RowDh {
    float g, at_blank, at_label;
};
__device__ __forceinline__ RowDh row_score_gradient(const LatticeState& ls, long long idx, int t, int u, int T, int U, int s,
                                                    int label, int blank) {
    const RowPost rp = row_posteriors(ls, idx, t, u, T, U, s);
    const float both = (label == blank) ? 1.0f : 0.0f;
    RowDh r;
    r.g = (rp.log_gamma - ls.lse[idx]) * LOG2E_F;
    r.at_blank = __expf(rp.log_gamma + ls.em[idx].x) - rp.Bk - both * rp.Yk;
    r.at_label = (label >= 0) ? __expf(rp.log_gamma + ls.em[idx].y) - rp.Yk - both * rp.Bk : 0.0f;
    return r;
}

// Asynchronous global -> LDS copy of 16 bytes per lane (global_load_lds_dwordx4): lane l's 16 bytes, at sbase + voff (a wave-uniform
// 64-bit base and a 32-bit byte offset per lane), land at LDS byte address lds_base + 16*l (lds_base wave-uniform, passed
// in M0).  Completion is tracked by the wave's vmcnt counter; the compiler does not see these loads, so the waits are explicit below.
// A load that takes its LDS address from M0 may not follow the scalar write of M0 directly: one wait state in between, which the
// compiler does not add inside assembler text.  Here and in the other copies the s_nop is that wait state.
__device__ __forceinline__ void lds_dma16_s(const void* sbase, unsigned voff, unsigned lds_base) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase), "s"(lds_base)
                 : "memory", "m0");
}


// ---- chunk buffers: MFMA fragments ------------------------------------------------------------------------
// dH [rows, V] and Z [rows, H] (bf16) lie in fragments of 32 rows x 16 columns (1 KiB): block of 32 rows (half a lattice
// tile) after block, in a block fragment after fragment along the columns, in a fragment 64 granules of 8 columns (16
// bytes).  Granule (row r, column half o) of fragment f lies at position 32 o + (r ^ (4 (2 (f & 1) + o))).  A wave that holds
// an MFMA operand fragment (lane l: row l % 32, columns 8 (l / 32) .. +7) writes or reads it as 1 KiB of whole cache
// lines; the dW GEMM, which contracts over the rows, reads the same bytes with transposing LDS reads, and the xor spreads
// the 16 rows such a read touches over all banks.  A block is 64 n + 4096 bytes (32 rows of chunk_pitch(n) elements), so that
// blocks of a power-of-two length do not all start in the same memory channel.
__host__ __device__ inline size_t chunk_block_bytes(int n) { return (size_t)64 * chunk_pitch(n); }
// byte offset of this lane's granule in a fragment of parity par (lane as above)
__device__ __forceinline__ unsigned frag_granule(int lane, int par) {
    const int o = lane >> 5;
    return (unsigned)((o * 32 + ((lane & 31) ^ (4 * (2 * par + o)))) * 16);
}

template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<I + 1, N>(f);
    }
}

// The same copy as lds_dma16_s with an immediate offset, which moves both addresses: OFF bytes from sbase and from lds_base.
template <int OFF>
__device__ __forceinline__ void lds_dma16_imm(const void* sbase, unsigned voff, unsigned lds_base) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:%3" ::"v"(voff), "s"(sbase), "s"(lds_base),
                 "n"(OFF)
                 : "memory", "m0");
}
// Two of them, OFF and OFF + 1024, for one write of M0.
template <int OFF>
__device__ __forceinline__ void lds_dma16_pair(const void* sbase, unsigned voff, unsigned lds_base) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 offset:%3\n\t"
                 "global_load_lds_dwordx4 %0, %1 offset:%4" ::"v"(voff), "s"(sbase), "s"(lds_base), "n"(OFF), "n"(OFF + 1024)
                 : "memory", "m0");
}
// 4 bytes per lane: word at sbase + voff of lane l -> lds_base + 4 l (64 words; lanes with equal voff write equal words)
__device__ __forceinline__ void lds_dma4_s(const void* sbase, unsigned voff, unsigned lds_base) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(voff), "s"(sbase), "s"(lds_base)
                 : "memory", "m0");
}

// Exchange between the two halves of a wave: returns {x of the lower half in both, ...}: the upper half of x changes
// places with the lower half of y.
__device__ __forceinline__ void swap_halves(unsigned& x, unsigned& y) {
    const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
    x = r[0];
    y = r[1];
}
__device__ __forceinline__ float both_halves_max(float v) {
    unsigned a = __float_as_uint(v), b = a;
    swap_halves(a, b);
    return fmaxf(__uint_as_float(a), __uint_as_float(b));
}
__device__ __forceinline__ float both_halves_sum(float v) {
    unsigned a = __float_as_uint(v), b = a;
    swap_halves(a, b);
    return __uint_as_float(a) + __uint_as_float(b);
}

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
// acc += A B with the B fragment in accumulation registers (AGPR) or in vector registers.  Written as assembler text
// because the compiler copies operands that live in AGPRs to vector registers first (four moves per MFMA: the power
// and the issue slots of this kernel).  The compiler places no wait states for it, so the code around it keeps the
// required distances itself: a vector instruction that writes an operand stands at least two instructions ahead
// (mfma_after_valu), and the result is not read before the whole depth of the matrix pipe has passed (mfma_result_ready, or at least
// two further MFMAs in between).  Both waits name the accumulators, so that no move of them can be placed behind the wait.
template <bool AGPR>
__device__ __forceinline__ void mfma_zb(f32x16& acc, const u32x4& w, const u32x4& z) {
    if constexpr (AGPR) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(w), "a"(z));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(w), "v"(z));
}
// Eight values of one half of a score block (registers 8 p .. 8 p + 7 of its accumulator: columns 16 p + {4 hb .. +3, 8 + 4 hb .. +3}
// of the lane's row) -> this lane's granule of the 32 x 16 bf16 fragment p (columns 16 p + 8 hb .. +7)
__device__ __forceinline__ u32x4 fragment_from_scores(const f32x16& d, int p) {
    typedef __bf16 pair __attribute__((ext_vector_type(2)));
    unsigned x[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const pair v = {(bf16_t)d[8 * p + 2 * i], (bf16_t)d[8 * p + 2 * i + 1]};
        x[i] = __builtin_bit_cast(unsigned, v);
    }
    swap_halves(x[0], x[2]);
    swap_halves(x[1], x[3]);
    return u32x4{x[0], x[1], x[2], x[3]};
}
__device__ __forceinline__ void mfma_after_valu(f32x16 (&acc)[1]) { asm volatile("s_nop 3" : "+v"(acc[0])::"memory"); }
__device__ __forceinline__ void mfma_after_valu(f32x16 (&acc)[2]) { asm volatile("s_nop 3" : "+v"(acc[0]), "+v"(acc[1])::"memory"); }
__device__ __forceinline__ void mfma_result_ready(f32x16& acc) { asm volatile("s_nop 15\n\ts_nop 7" : "+v"(acc)); }

// The joint rows of one wave as MFMA B fragments: z[kk] of lane (l32, hb) holds row l32, columns 16 kk + 8 hb .. +7.
// The wave's 32 rows need 12 input rows (4 frames + 8 labels, or 8 + 4).  All their loads are sent at once (JointInputs): a workgroup has
// one or two waves per SIMD and nothing else would hide their latency.
// tanh(x) = 1 - 2 / (e^{2x} + 1) with e^{2(e+q)} = e^{2e} e^{2q}: the exponentials of the 12 input rows are formed
// once per column (128 columns at a time, in the wave's own LDS scratch) and an element costs one reciprocal.  Inputs
// beyond +-40 (exponents beyond +-115, where the product could overflow): everything is computed from the sums.
constexpr int JR_PITCH = 144;                 // floats per row of the scratch (128 columns; 64 bytes of padding against bank conflicts)
constexpr int JR_SCRATCH = 12 * JR_PITCH * 4;     // bytes per wave
template <int KK>
struct JointInputs {
    bf16x8 x[KK / 8][3];
    // enc / prd: the sample's rows
    __device__ __forceinline__ void load(const bf16_t* __restrict__ enc, const bf16_t* __restrict__ prd, int H, const TilePos& tp,
                                         int half, int lane) {
        const int nT = 32 >> tp.us;                       // frames of the wave: 4 (8 x 8 tile) or 8 (16 x 4)
        const int tb = tp.t0 + half * nT;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const int vec = (lane >> 4) + 4 * i, c = lane & 15;
            const int t = tb + vec, u = tp.u0 + vec - nT;
            const bf16_t* src = (vec < nT ? enc + (size_t)(t < tp.T ? t : tp.T - 1) * H : prd + (size_t)(u <= tp.U ? u : tp.U) * H) + c * 8;
#pragma unroll
            for (int ch = 0; ch < KK / 8; ++ch) x[ch][i] = *reinterpret_cast<const bf16x8*>(src + ch * 128);
        }
    }
};
// FIRST: index of the wave's first fragment here (those below AGPR_FRAGS are moved to accumulation registers).
// zout: this wave's block of the Z chunk buffer, or null.
template <int KK, int FIRST, int AGPR_FRAGS>
__device__ __forceinline__ void build_joint_rows(u32x4 (&z)[KK], const JointInputs<KK>& in, float* scratch,
                                                 const bf16_t* __restrict__ enc, const bf16_t* __restrict__ prd, int H,
                                                 const TilePos& tp, int half, int lane, unsigned char* zout) {
    constexpr float K2 = 2.0f * LOG2E_F;
    const int l32 = lane & 31, hb = lane >> 5;
    const int nT = 32 >> tp.us;
    const int ra = l32 >> tp.us, rb = l32 & (tp.uw - 1);
    const float* ea = scratch + ra * JR_PITCH + 8 * hb;
    const float* qa = scratch + (nT + rb) * JR_PITCH + 8 * hb;
    float big = 0.0f;
#pragma unroll
    for (int ch = 0; ch < KK / 8; ++ch)
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int k = 0; k < 8; ++k) big = fmaxf(big, fabsf((float)in.x[ch][i][k]));
    if (__any(!(big <= 115.0f / K2))) {
        const int t = tp.t0 + half * nT + ra, u = tp.u0 + rb;
        const bf16_t* er = enc + (size_t)(t < tp.T ? t : tp.T - 1) * H + 8 * hb;
        const bf16_t* qr = prd + (size_t)(u <= tp.U ? u : tp.U) * H + 8 * hb;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            z[kk] = __builtin_bit_cast(u32x4, joint_tanh8(*reinterpret_cast<const bf16x8*>(er + kk * 16),
                                                          *reinterpret_cast<const bf16x8*>(qr + kk * 16)));
            if (FIRST + kk < AGPR_FRAGS) asm volatile("" : "+a"(z[kk]));
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
#pragma unroll
        for (int ch = 0; ch < KK / 8; ++ch) {
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                float* dst = scratch + ((lane >> 4) + 4 * i) * JR_PITCH + (lane & 15) * 8;
                f32x4 lo, hi;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    lo[k] = __builtin_amdgcn_exp2f((float)in.x[ch][i][k] * K2);
                    hi[k] = __builtin_amdgcn_exp2f((float)in.x[ch][i][4 + k] * K2);
                }
                *reinterpret_cast<f32x4*>(dst) = lo;
                *reinterpret_cast<f32x4*>(dst + 4) = hi;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int k8 = 0; k8 < 8; ++k8) {
                f32x4 e[2], q[2];
#pragma unroll
                for (int p = 0; p < 2; ++p) {
                    e[p] = *reinterpret_cast<const f32x4*>(ea + k8 * 16 + 4 * p);
                    q[p] = *reinterpret_cast<const f32x4*>(qa + k8 * 16 + 4 * p);
                }
                bf16x8 zv;
#pragma unroll
                for (int p = 0; p < 2; ++p)
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        zv[4 * p + k] = (bf16_t)(1.0f - 2.0f * __builtin_amdgcn_rcpf(fmaf(e[p][k], q[p][k], 1.0f)));
                z[ch * 8 + k8] = __builtin_bit_cast(u32x4, zv);
                if (k8 & 1) __builtin_amdgcn_sched_barrier(0);     // (keeps the loads of later steps from piling up in registers)
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int k8 = 0; k8 < 8; ++k8)
                if (FIRST + ch * 8 + k8 < AGPR_FRAGS) asm volatile("" : "+a"(z[ch * 8 + k8]));
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (zout != nullptr) {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
            __builtin_nontemporal_store(z[kk], reinterpret_cast<u32x4*>(zout + kk * 1024 + frag_granule(lane, kk & 1)));
    }
}

}  // namespace rnnt
