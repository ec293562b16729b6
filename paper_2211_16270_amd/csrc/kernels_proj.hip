// The two linear maps inside the tanh of the joint network (Eq. 4): enc = hA W_A + b_Z, pred = hL W_L,
// and their backward (Algorithm 1 line 9 for W_A, b_Z, W_L; lines 10-11 continued to hA, hL).
//
// All of them are one GEMM shape family  C[m,n] (+)= sum_k A(m,k) B(k,n)  over row-major arrays whose
// operands differ only in which index is contiguous in memory:
//   forward      enc[r,h]   = sum_k hA[r,k]   W_A[k,h] + b_Z[h]     A k-contiguous, B k-slow
//   d input      d_hA[r,k]  = sum_h d_enc[r,h] W_A[k,h]             A k-contiguous, B k-contiguous
//   d weights    dW_A[k,h] += sum_r hA[r,k]   d_enc[r,h]            A k-slow, B k-slow (split over r)
// Rows r = b*T_max + t beyond a sample's length are padding: their input may hold anything (NaN
// included) and is read as zero.
//
// bf16 path: 128x128 output tile per workgroup, 4 waves x (64x64 = 2x2 MFMA 32x32x16 tiles), K-step 64.
// A k-contiguous operand lies in LDS as [row][k] and gives fragments by plain 16-byte reads; a k-slow
// operand lies there as in memory ([k][row], 16-byte chunks XOR-swizzled) and gives fragments by the
// transposing LDS read.  Both maps of a direction are one launch (forward: k_proj_forward; backward: k_proj_backward, the four products and db_Z).
// What bounds it: at the sizes of a training step (8000 + 1632 rows, D = H = 512: 15 GFLOP in all) the latency of a K-step's loads and the number of
// launches; a large batch, the bytes.  So loads run two K-steps ahead in registers and are not touched before they go to LDS (masks and the rounding of
// fp32 operands are applied there).  32 samples of 250 x 50, D = H = 512: forward 18.6 us, backward 47,
// where seven launches that waited for each step's loads took 55 and 172; a call 1161 -> 1012 us.
// fp32 path: the tile GEMM of the fp32 joint path where rows are 16-byte aligned (D, H multiples of 4);
// else one thread per output element.
#include "device_common.h"
#include "kernels.h"

#include <algorithm>
#include <cmath>

namespace rnnt {

namespace {

constexpr int PT = 128;        // output tile edge
constexpr int PK = 64;         // K-step
constexpr int PP = PK + 8;     // LDS row pitch (bf16 elements): 144 bytes, conflict-free 16-byte reads
constexpr int PQ = PT * PK / 8 / 256;   // 8-element chunks per thread, operand and step
constexpr unsigned P_OPER = PT * PP;    // elements of one operand's stage (PT*PP >= PK*PT: either layout fits)
constexpr size_t P_SMEM = (size_t)4 * P_OPER * sizeof(bf16_t);      // two stages of two operands
static_assert(PT * PP >= PK * PT, "LDS tile size");

// source row s is real data iff there is no mask or (s % period) < len[s / period] + extra
__device__ __forceinline__ bool row_is_data(const RowMask& m, long long s) {
    if (m.len == nullptr) return true;
    const long long b = s / m.period;
    return (int)(s - b * m.period) < m.len[b] + m.extra;
}

// Eight elements as they lie in memory (the caller's arrays need no more than their element's alignment), and as bf16.
template <typename T>
struct Chunk8;
template <>
struct Chunk8<bf16_t> {
    typedef bf16x8 any_aligned __attribute__((aligned(2)));
    bf16x8 v;
    __device__ __forceinline__ void load(const bf16_t* p) { v = *reinterpret_cast<const any_aligned*>(p); }
    __device__ __forceinline__ bf16x8 rounded() const { return v; }
};
typedef f32x4 f32x4_any __attribute__((aligned(4)));
template <>
struct Chunk8<float> {
    f32x4 a, b;
    __device__ __forceinline__ void load(const float* p) {
        a = *reinterpret_cast<const f32x4_any*>(p);
        b = *reinterpret_cast<const f32x4_any*>(p + 4);
    }
    __device__ __forceinline__ bf16x8 rounded() const {
        bf16x8 r;
#pragma unroll
        for (int j = 0; j < 4; ++j) { r[j] = (bf16_t)a[j]; r[4 + j] = (bf16_t)b[j]; }
        return r;
    }
};

// One operand of the tile product.  KSLOW = false: element (i, k) at p[i*ld + k]; true: at p[k*ld + i].
// i runs over the tile's 128 rows (m for A, n for B) starting at i0.  Each of the 256 threads fetches PQ chunks of 8 elements along the contiguous index.
template <typename T, bool KSLOW>
struct Operand {
    const T* base;         // of this thread's chunks
    long long ld, last;    // KSLOW: last valid k
    const T* row[PQ];      // !KSLOW: its rows (those beyond n_i: the last one again, whose products are not stored)

    __device__ __forceinline__ Operand(const T* p, long long ld_, long long i0, long long n_i, long long n_k, int tid) : ld(ld_), last(n_k - 1) {
        if (KSLOW) {
            base = p + i0 + (tid & 15) * 8;                     // 16 chunks of 8 along i per k
        } else {
            base = nullptr;
#pragma unroll
            for (int q = 0; q < PQ; ++q) {
                const long long i = i0 + (tid >> 3) + 32 * q;   // 8 chunks of 8 along k per row
                row[q] = p + (i < n_i ? i : n_i - 1) * ld + (tid & 7) * 8;
            }
        }
    }
    __device__ __forceinline__ void fetch(Chunk8<T> (&v)[PQ], long long k0, int tid) const {
#pragma unroll
        for (int q = 0; q < PQ; ++q) {
            if (KSLOW) {
                const long long k = k0 + (tid >> 4) + 16 * q;
                v[q].load(base + (k < last ? k : last) * ld);
            } else {
                v[q].load(row[q] + k0);
            }
        }
    }
    // LDS image of the tile.  !KSLOW: [i][k], pitch PP (k contiguous).  KSLOW: as in memory, [k][i] with
    // 128 elements per row, 16-byte chunk c of row k at position c ^ 4*(k%4) (conflict-free for the
    // transposing read that turns it into MFMA fragments); row k is read as zero where bit k of `live` is not set.
    static __device__ __forceinline__ void stage(const Chunk8<T> (&v)[PQ], bf16_t* tile, int tid, unsigned long long live) {
#pragma unroll
        for (int q = 0; q < PQ; ++q) {
            const bf16x8 x = v[q].rounded();
            if (!KSLOW) {
                *reinterpret_cast<bf16x8*>(tile + ((tid >> 3) + 32 * q) * PP + (tid & 7) * 8) = x;
            } else {
                const int kk = (tid >> 4) + 16 * q, c = tid & 15;
                u32x4 w = __builtin_bit_cast(u32x4, x);
                w &= (live >> kk) & 1 ? ~0u : 0u;
                *reinterpret_cast<u32x4*>(tile + kk * PT + ((c ^ ((kk & 3) << 2)) << 3)) = w;
            }
        }
    }
    // MFMA fragment of rows [i_base, i_base + 32), k16-step kk: lane l holds row i_base + l%32, k = 8*(l/32)..+7
    static __device__ __forceinline__ bf16x8 fragment(const bf16_t* tile, int i_base, int kk, int lane) {
        if (!KSLOW) {
            return *reinterpret_cast<const bf16x8*>(tile + (i_base + (lane & 31)) * PP + kk * 16 + (lane >> 5) * 8);
        } else {
            // transposing read: within 16 lanes, lane 4j+c supplies 4 columns of row j and lane i receives
            // rows 0..3 of column i; lane = 16 g + 4 j + c reads row 8*(g/2) + j, columns 16*(g%2) + 4c .. +3
            typedef short s16x4 __attribute__((ext_vector_type(4)));
            typedef short s16x8 __attribute__((ext_vector_type(8)));
            const int fg = lane >> 4, fj = (lane >> 2) & 3, fc = lane & 3;
            const int row = kk * 16 + 8 * (fg >> 1) + fj;
            const int col = i_base + 16 * (fg & 1) + 4 * fc;
            const bf16_t* p = tile + row * PT + ((((col >> 3) ^ (fj << 2))) << 3) + (col & 7);
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p + 4 * PT));
            const s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            return __builtin_bit_cast(bf16x8, v);
        }
    }
};

struct TileJob {
    const void* A;
    const void* B;
    long long lda, ldb;
    void* C;
    long long ldc;
    const float* bias;       // per column n, or null
    float* col_sum;          // ROWS_K: += column sums of B over the rows of the split, or null
    RowMask mask;            // ROWS_K: of the source rows k of both operands
    long long M, N, K;       // N and K multiples of 128 (ROWS_K: N and M, any K)
};

// The tile (m0, n0) of C = A B, K from ks to ke.  ROWS_K: the operands are k-slow, k runs over source rows; C is added to with float atomics.
// OUT: element type of C.
template <typename TA, typename TB, bool B_KSLOW, bool ROWS_K, typename OUT>
__device__ __forceinline__ void proj_tile(const TileJob& g, unsigned char* smem, long long m0, long long n0, long long ks, long long ke) {
    typedef Operand<TA, ROWS_K> OpA;
    typedef Operand<TB, B_KSLOW> OpB;
    bf16_t* stages = reinterpret_cast<bf16_t*>(smem);                 // [2][A, B]
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, hb = lane >> 5;
    const int wm = wave >> 1, wn = wave & 1;
    const OpA A((const TA*)g.A, g.lda, m0, g.M, g.K, tid);
    const OpB B((const TB*)g.B, g.ldb, n0, g.N, g.K, tid);

    f32x16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x16{0};
    float sum[8] = {};
    const bool summing = ROWS_K && g.col_sum != nullptr;              // (uniform)

    Chunk8<TA> va[2][PQ];
    Chunk8<TB> vb[2][PQ];
    int len[2] = {}, pos[2] = {};                 // ROWS_K: of source row k0 + lane: its sample's length, its place in the sample
    const long long k_last = ks + (ke - ks - 1) / PK * PK;            // the last step
    auto fetch = [&](auto set_tag, long long k0) {
        constexpr int s = decltype(set_tag)::value;
        k0 = k0 < k_last ? k0 : k_last;           // (past the end: the last step again, not used)
        A.fetch(va[s], k0, tid);
        B.fetch(vb[s], k0, tid);
        if (ROWS_K) {
            const unsigned r = (unsigned)(k0 + lane), b = (r < (unsigned)g.K ? r : (unsigned)g.K - 1u) / (unsigned)g.mask.period;
            pos[s] = (int)(r - b * (unsigned)g.mask.period);
            len[s] = g.mask.len[b];
        }
    };
    auto stage = [&](auto set_tag, long long k0) {
        constexpr int s = decltype(set_tag)::value;
        unsigned long long live = ~0ull;
        if (ROWS_K) live = __builtin_amdgcn_ballot_w64(pos[s] < len[s] + g.mask.extra && k0 + lane < ke);
        bf16_t* t = stages + s * 2 * P_OPER;
        OpA::stage(va[s], t, tid, live);
        OpB::stage(vb[s], t + P_OPER, tid, live);
        if constexpr (ROWS_K)
            if (summing) {
#pragma unroll
                for (int q = 0; q < PQ; ++q) {
                    const bool ok = (live >> ((tid >> 4) + 16 * q)) & 1;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        sum[j] += ok ? vb[s][q].a[j] : 0.0f;
                        sum[4 + j] += ok ? vb[s][q].b[j] : 0.0f;
                    }
                }
            }
    };
    // A step: the next one's operands, loaded two steps before, go to the other stage, which every wave has left at the barrier; the loads of the
    // step after the next but one are sent; the MFMAs.
    auto step = [&](auto set_tag, long long k0) {
        constexpr int s = decltype(set_tag)::value;
        typedef std::integral_constant<int, s ^ 1> Other;
        stage(Other{}, k0 + PK);                  // (past the end: a stage nobody reads)
        __builtin_amdgcn_sched_barrier(0);        // (loads stay in this order: their waits are by count)
        fetch(Other{}, k0 + 3 * PK);
        __builtin_amdgcn_sched_barrier(0);
        const bf16_t* As = stages + s * 2 * P_OPER;
        const bf16_t* Bs = As + P_OPER;
#pragma unroll
        for (int kk = 0; kk < PK / 16; ++kk) {
            bf16x8 fa[2], fb[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) fa[i] = OpA::fragment(As, wm * 64 + i * 32, kk, lane);
#pragma unroll
            for (int j = 0; j < 2; ++j) fb[j] = OpB::fragment(Bs, wn * 64 + j * 32, kk, lane);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    // (added to C: lanes along n, whole lines of atomics; stored: lanes along m, a lane holds runs of four columns)
                    acc[i][j] = ROWS_K ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0)
                                       : __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
        }
        __syncthreads();
    };
    typedef std::integral_constant<int, 0> I0;
    typedef std::integral_constant<int, 1> I1;
    fetch(I0{}, ks);
    __builtin_amdgcn_sched_barrier(0);
    fetch(I1{}, ks + PK);
    __builtin_amdgcn_sched_barrier(0);
    stage(I0{}, ks);
    __builtin_amdgcn_sched_barrier(0);
    fetch(I0{}, ks + 2 * PK);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    // (two steps without a branch between them, so that the waits for loads stay by count: K is a multiple of 128, and rows from ke on are zeros)
    for (long long k0 = ks; k0 < ke; k0 += 2 * PK) {
        step(I0{}, k0);
        step(I1{}, k0 + PK);
    }

    f32x4 bias[2][4];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) bias[j][q] = f32x4{0};
    if (!ROWS_K && g.bias != nullptr) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) bias[j][q] = *reinterpret_cast<const f32x4_any*>(g.bias + n0 + wn * 64 + j * 32 + 4 * hb + 8 * q);
    }
    // accumulator register 4q+r of tile (i,j): place 8q + 4hb + r of its first operand's rows, l32 of the second's
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if constexpr (ROWS_K) {
                float* c = (float*)g.C + (m0 + wm * 64 + i * 32 + 4 * hb) * g.ldc + n0 + wn * 64 + j * 32 + l32;
#pragma unroll
                for (int q = 0; q < 16; ++q) atomicAdd(c + (8 * (q >> 2) + (q & 3)) * g.ldc, acc[i][j][q]);
            } else {
                const long long m = m0 + wm * 64 + i * 32 + l32, n = n0 + wn * 64 + j * 32 + 4 * hb;
                if (m >= g.M) continue;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    f32x4 v;
#pragma unroll
                    for (int r = 0; r < 4; ++r) v[r] = acc[i][j][4 * q + r] + bias[j][q][r];
                    if constexpr (std::is_same_v<OUT, float>) {
                        *reinterpret_cast<f32x4_any*>((float*)g.C + m * g.ldc + n + 8 * q) = v;
                    } else {
                        bf16x4 o;
#pragma unroll
                        for (int r = 0; r < 4; ++r) o[r] = (bf16_t)v[r];
                        *reinterpret_cast<bf16x4*>((bf16_t*)g.C + m * g.ldc + n + 8 * q) = o;
                    }
                }
            }
        }
    if constexpr (ROWS_K)
        if (summing) {
            float* red = reinterpret_cast<float*>(smem);              // [16 row groups][128 columns] (the last step ended with a barrier)
#pragma unroll
            for (int j = 0; j < 8; ++j) red[(tid >> 4) * PT + (tid & 15) * 8 + j] = sum[j];
            __syncthreads();
            if (tid < PT) {
                float t = 0.0f;
#pragma unroll
                for (int r = 0; r < 16; ++r) t += red[r * PT + tid];
                atomicAdd(g.col_sum + n0 + tid, t);
            }
        }
}

// Workgroups of a launch are numbered so that those which agree modulo 8 share an L2: the tiles that read the same rows (of h or d_out) are neighbours
// on one XCD.  Each part of a launch takes a multiple of 8 workgroups.
struct RowTiles {
    int m_tiles, n_tiles;
    __host__ __device__ int workgroups() const { return (m_tiles + 7) / 8 * 8 * n_tiles; }
};

struct ForwardArgs {
    TileJob job[2];
    RowTiles t[2];
    float* clear[3];         // cleared by the workgroups behind the tiles (the backward launch adds to them)
    long long clear_n[3];
    int clear_wgs;
};
__global__ __launch_bounds__(256, 2) void k_proj_forward(ForwardArgs a) {
    extern __shared__ __align__(16) unsigned char proj_smem[];
    int L = blockIdx.x;
    const int n_a = a.t[0].workgroups();
    if (L >= n_a + a.t[1].workgroups()) {
        L -= n_a + a.t[1].workgroups();
#pragma unroll
        for (int r = 0; r < 3; ++r)
            for (long long i = (long long)L * 256 + threadIdx.x; i < a.clear_n[r]; i += (long long)a.clear_wgs * 256) a.clear[r][i] = 0.0f;
        return;
    }
    const int side = L >= n_a;
    if (side) L -= n_a;
    const RowTiles t = side ? a.t[1] : a.t[0];
    const TileJob& g = side ? a.job[1] : a.job[0];
    const int q = L >> 3, m = (L & 7) + 8 * (q / t.n_tiles), n = q % t.n_tiles;
    if (m >= t.m_tiles) return;
    proj_tile<bf16_t, bf16_t, true, false, bf16_t>(g, proj_smem, (long long)m * PT, (long long)n * PT, 0, g.K);
}

struct BackwardArgs {
    TileJob weight[2], input[2];
    int tiles[2], n_tiles;   // weight: output tiles, of which n_tiles along n
    int splits[2];
    long long per_split[2];
    RowTiles t[2];
};
__global__ __launch_bounds__(256, 2) void k_proj_backward(BackwardArgs a) {
    extern __shared__ __align__(16) unsigned char proj_smem[];
    int L = blockIdx.x;
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        const int n = (a.splits[side] + 7) / 8 * 8 * a.tiles[side];
        if (L < n) {
            const int q = L >> 3, split = (L & 7) + 8 * (q / a.tiles[side]), tile = q % a.tiles[side];
            TileJob g = a.weight[side];
            const long long ks = split * a.per_split[side], ke = ks + a.per_split[side] < g.K ? ks + a.per_split[side] : g.K;
            if (split >= a.splits[side] || ks >= ke) return;
            const int m = tile / a.n_tiles;
            if (m != 0) g.col_sum = nullptr;
            proj_tile<bf16_t, float, true, true, float>(g, proj_smem, (long long)m * PT, (long long)(tile % a.n_tiles) * PT, ks, ke);
            return;
        }
        L -= n;
    }
    const int side = L >= a.t[0].workgroups();
    if (side) L -= a.t[0].workgroups();
    const RowTiles t = side ? a.t[1] : a.t[0];
    const TileJob& g = side ? a.input[1] : a.input[0];
    const int q = L >> 3, m = (L & 7) + 8 * (q / t.n_tiles), n = q % t.n_tiles;
    if (m >= t.m_tiles) return;
    proj_tile<float, bf16_t, false, false, float>(g, proj_smem, (long long)m * PT, (long long)n * PT, 0, g.K);
}

template <typename ARGS>
hipError_t launch_proj(void (*kernel)(ARGS), const ARGS& a, long long workgroups, hipStream_t stream) {
    if (workgroups > 0x7fffffffLL) return hipErrorInvalidValue;
    static bool configured = false;          // one flag per instantiation, i.e. kernel
    if (!configured) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)P_SMEM);
        if (e != hipSuccess) return e;
        configured = true;
    }
    kernel<<<dim3((unsigned)workgroups), dim3(256), P_SMEM, stream>>>(a);
    return hipGetLastError();
}

// ---- fp32: one thread per output element ---------------------------------------------------
// A(m,k) at a[m*sam + k*sak], B(k,n) at b[k*sbk + n*sbn]; masked: rows k of both operands
__global__ void k_proj_gemm_f32(const float* __restrict__ a, long long sam, long long sak, const float* __restrict__ b,
                                long long sbk, long long sbn, float* __restrict__ c, long long ldc,
                                const float* __restrict__ bias, long long M, long long N, long long K, RowMask mask,
                                int accumulate) {
    const long long idx = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= M * N) return;
    const long long m = idx / N, n = idx - m * N;
    float s = bias ? bias[n] : 0.0f;
    for (long long k = 0; k < K; ++k) {
        if (!row_is_data(mask, k)) continue;
        s = fmaf(a[m * sam + k * sak], b[k * sbk + n * sbn], s);
    }
    c[m * ldc + n] = accumulate ? c[m * ldc + n] + s : s;
}

// out[c] (+)= sum over all rows of x[r, c]   (x fp32 [rows, cols]); 256 columns x one slice of rows per workgroup
__global__ __launch_bounds__(256) void k_col_sum(const float* __restrict__ x, long long rows, int cols, long long rows_per,
                                                 float* __restrict__ out) {
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= cols) return;
    const long long r0 = (long long)blockIdx.y * rows_per;
    const long long r1 = r0 + rows_per < rows ? r0 + rows_per : rows;
    float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;
    long long r = r0;
    for (; r + 3 < r1; r += 4) {
        s0 += x[r * cols + c];
        s1 += x[(r + 1) * cols + c];
        s2 += x[(r + 2) * cols + c];
        s3 += x[(r + 3) * cols + c];
    }
    for (; r < r1; ++r) s0 += x[r * cols + c];
    atomicAdd(&out[c], (s0 + s1) + (s2 + s3));
}

// Rows per split of a weight gradient's sum: a multiple of 128, at least 256, for about 256 workgroups where that costs no accuracy, else as many as keep
// the sum's error down.  A split of n rows is n / 16 additions of the matrix instruction, S splits are as many atomics.  Rounded additions of terms of
// random sign leave u sqrt(n / 32 + S / 2) of the result, least at n = 4 sqrt(rows); of terms of one sign u sqrt(n / (48 S) + S / 3), least at
// n = 2 rows^(2/3).  Between the two one grows as the other falls; there the splits are those of 512 workgroups.  Relative error of dW, inputs of either
// sign (of one sign), 320 k rows, with 256 workgroups, with 512 of them and with this rule: D = H = 512 6.7e-7, 4.8e-7, 4.6e-7 (1.8e-7, 1.2e-7, 1.2e-7);
// D = H = 1024 1.5e-6, 1.0e-6, 5.0e-7 (7.6e-7, 3.6e-7, 1.2e-7).  Time of a call with 256 workgroups and with this rule: that one 9300 -> 8215 us, D = H = 512
// 3300 -> 3370, 64 samples of 1000 x 3, D = 1024, H = 640 1162 -> 1198; 8000 rows, D = H = 512 as before.
long long proj_split_rows(int tiles, long long rows) {
    const double n = (double)rows, fill = n * tiles / 256, low = 4.0 * std::sqrt(n), high = 2.0 * std::cbrt(n * n);
    const double best = fill * fill <= 2.0 * low * low ? fill : std::max(low, std::min(0.5 * fill, high));      // (as far from low as half of it)
    return std::max(256LL, ((long long)best + 64) / 128 * 128);
}

}  // namespace

static hipError_t proj_forward_f32(const ProjSide& s, int H, hipStream_t stream) {
    const RowMask none{nullptr, 1, 0};
    if (gemm_f32_edge_fits(s.h, s.D, s.W, H, s.D, H))
        return launch_gemm_f32_masked(0, 1, (const float*)s.h, s.D, none, (const float*)s.W, H, none, (float*)s.out, H, s.bias, 0, s.rows, H, s.D, 1,
                                      stream);
    const long long total = s.rows * H;
    k_proj_gemm_f32<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream>>>(
        (const float*)s.h, s.D, 1, (const float*)s.W, H, 1, (float*)s.out, H, s.bias, s.rows, H, s.D, none, 0);
    return hipGetLastError();
}

static hipError_t proj_backward_f32(const ProjSide& s, int H, hipStream_t stream) {
    // padded rows of d_out are zero, so d_in is zero there without a mask; dW is added to with float atomics
    const RowMask none{nullptr, 1, 0};
    const float *h = (const float*)s.h, *W = (const float*)s.W;
    hipError_t e;
    if (gemm_f32_edge_fits(s.d_out, H, s.W, H, H, H)) {
        e = launch_gemm_f32_masked(0, 0, s.d_out, H, none, W, H, none, s.d_in, s.D, nullptr, 0, s.rows, s.D, H, 1, stream);
    } else {
        const long long total = s.rows * s.D;
        k_proj_gemm_f32<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream>>>(
            s.d_out, H, 1, W, 1, H, s.d_in, s.D, nullptr, s.rows, s.D, H, none, 0);
        e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
    if (gemm_f32_edge_fits(s.h, s.D, s.d_out, H, s.D, H)) {
        e = launch_gemm_f32_masked(1, 1, h, s.D, s.mask, s.d_out, H, s.mask, s.dW, H, nullptr, 1, s.D, H, s.rows,
                                   k_splits_f32(s.D, H, s.rows), stream);
    } else {
        const long long total = (long long)s.D * H;
        k_proj_gemm_f32<<<dim3((unsigned)((total + 255) / 256)), dim3(256), 0, stream>>>(
            h, 1, s.D, s.d_out, H, 1, s.dW, H, nullptr, s.D, H, s.rows, s.mask, 1);
        e = hipGetLastError();
    }
    if (e != hipSuccess || s.db == nullptr) return e;
    return launch_col_sum(s.d_out, s.rows, H, s.db, stream);
}

hipError_t launch_proj_forward(int bf16, const ProjSide (&s)[2], int H, bool clear, hipStream_t stream) {
    if (!bf16) {
        if (clear) {
            PrepArgs pa{};
            for (int i = 0; i < 2; ++i) {
                pa.zero_ptr[i] = s[i].dW;
                pa.zero_n[i] = (size_t)s[i].D * H;
            }
            pa.zero_ptr[2] = s[0].db;
            pa.zero_n[2] = (size_t)H;
            const hipError_t e = launch_prepare(pa, stream);
            if (e != hipSuccess) return e;
        }
        for (const ProjSide& x : s) {
            const hipError_t e = proj_forward_f32(x, H, stream);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    ForwardArgs a{};
    for (int i = 0; i < 2; ++i) {
        const ProjSide& x = s[i];
        a.job[i] = TileJob{x.h, x.W, x.D, H, x.out, H, x.bias, nullptr, RowMask{nullptr, 1, 0}, x.rows, H, x.D};
        a.t[i] = RowTiles{(int)((x.rows + PT - 1) / PT), H / PT};
        if (clear) {
            a.clear[i] = x.dW;
            a.clear_n[i] = (long long)x.D * H;
        }
    }
    if (clear) {
        a.clear[2] = s[0].db;
        a.clear_n[2] = H;
        a.clear_wgs = 64;
    }
    return launch_proj(k_proj_forward, a, (long long)a.t[0].workgroups() + a.t[1].workgroups() + a.clear_wgs, stream);
}

hipError_t launch_proj_backward(int bf16, const ProjSide (&s)[2], int H, hipStream_t stream) {
    if (!bf16) {
        for (const ProjSide& x : s) {
            const hipError_t e = proj_backward_f32(x, H, stream);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    BackwardArgs a{};
    a.n_tiles = H / PT;
    long long wgs = 0;
    for (int i = 0; i < 2; ++i) {
        const ProjSide& x = s[i];
        a.weight[i] = TileJob{x.h, x.d_out, x.D, H, x.dW, H, nullptr, x.db, x.mask, x.D, H, x.rows};
        a.input[i] = TileJob{x.d_out, x.W, H, H, x.d_in, x.D, nullptr, nullptr, RowMask{nullptr, 1, 0}, x.rows, x.D, H};
        a.tiles[i] = x.D / PT * a.n_tiles;
        a.per_split[i] = proj_split_rows(a.tiles[i], x.rows);
        a.splits[i] = (int)((x.rows + a.per_split[i] - 1) / a.per_split[i]);
        a.t[i] = RowTiles{(int)((x.rows + PT - 1) / PT), x.D / PT};
        wgs += (long long)(a.splits[i] + 7) / 8 * 8 * a.tiles[i] + a.t[i].workgroups();
    }
    return launch_proj(k_proj_backward, a, wgs, stream);
}

hipError_t launch_col_sum(const float* x, long long rows, int cols, float* out, hipStream_t stream) {
    if (rows <= 0 || cols <= 0) return hipSuccess;
    long long slices = (rows + 31) / 32;
    if (slices > 1024) slices = 1024;
    const long long per = (rows + slices - 1) / slices;
    k_col_sum<<<dim3((unsigned)((cols + 255) / 256), (unsigned)((rows + per - 1) / per)), dim3(256), 0, stream>>>(
        x, rows, cols, per, out);
    return hipGetLastError();
}

}  // namespace rnnt
