// fp32 path.  Two forms:
//  * plain FMA kernels for any H, V (the small fp32 workloads);
//  * for H and V multiples of 4 from 64 on, the same steps over chunks of lattice nodes as matrix GEMMs of fp32
//    precision (operands as three bf16 parts, k_gemm_f32) with row kernels between them:
//      Z = tanh(enc_t + pred_u)              (Eq. 4)            k_rows_z_f32
//      S = Z W + b                            (Eq. 6)            k_gemm_f32 <A k-contiguous, B k-slow>
//      lse, emissions per row                 (f^W_1)            k_rows_stats_f32
//      dh = gamma softmax - posteriors        (f^W_4)            k_rows_dh_f32 (in place of S)
//        db += column sums of dh              (Alg. 1 line 8)
//      dW += Z^T dh                           (Alg. 1 line 8)    k_gemm_f32 <A k-slow, B k-slow>, split over the rows
//      dZ = dh W^T                            (Alg. 1 l. 10-11)  k_gemm_f32 <A k-contiguous, B k-contiguous>
//      d_enc, d_pred += dZ (1 - Z^2)                             k_rows_dz_f32
//    The chunk buffers S [rows, V], Z and dZ [rows, H] live in the workspace; rows beyond the chunk's
//    last node (up to the next multiple of 128) are zero.  The throughput path is the bf16 one.
#include <algorithm>
#include <cstdint>

#include "device_common.h"

namespace rnnt {

__global__ void k_copy_f32(const float4* __restrict__ src, float4* __restrict__ dst, size_t n4) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n4; i += stride) dst[i] = src[i];
}

hipError_t launch_copy_f32(const float* src, float* dst, size_t n, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    k_copy_f32<<<dim3(4096), dim3(256), 0, stream>>>((const float4*)src, (float4*)dst, n / 4);
    return hipGetLastError();
}

struct NodePos {
    int s, T, U, t, u;
    long long idx;  // index into the group's lattice arrays
};

__device__ __forceinline__ NodePos locate_node(const SampleTable& st, long long row_base, int s0, int s1,
                                               long long r) {
    NodePos p;
    const long long rg = r + row_base;
    p.s = find_segment<long long>(st.row_off, s0, s1, rg);
    p.T = st.T[p.s];
    p.U = st.U[p.s];
    const int local = (int)(rg - st.row_off[p.s]);
    p.t = local / (p.U + 1);
    p.u = local - p.t * (p.U + 1);
    p.idx = st.row_off[p.s] - row_base + lattice_index(p.T, p.U + 1, p.t, p.u);
    return p;
}

// ---- plain kernels, any H and V: a workgroup takes `nodes` lattice nodes, their joint rows and scores lie in LDS, and W_out too where it is small.
// Threads stand in rows of G (a power of two, at most 64) over the vocabulary resp. the hidden columns.  What bounds them: latency; these are calls of
// a few thousand nodes at most.  One node per wavefront before: every node added its H V products to dW_out with atomics of its own, here
// a workgroup's nodes are summed first.  A call, H = 32, V = 16, 240 nodes 46.7 -> 25.0 us (43.4 with the present sweep and the old kernels); H = 63,
// V = 99, 8 k nodes 755 -> 108; H = 301, V = 1001, 240 nodes 1246 -> 508; H = 1023, V = 4097, 32 k nodes 585 -> 284 ms.

namespace {

constexpr int PLAIN_NODES = 16;            // most nodes per workgroup
constexpr int PLAIN_SUM = 64;              // entries of the vocabulary per partial sum of dz
constexpr size_t PLAIN_W = 24 * 1024;      // bytes of W_out that are kept in LDS
constexpr size_t PLAIN_ROWS = 64 * 1024;   // bytes of rows, for more than one node
constexpr long long WIDE_WGS = 512;        // workgroups of k_fwd_f32_wide before a thread takes more than one node
constexpr long long WIDE_LDS = 40 * 1024;

struct PlainShape {
    int nodes;                             // per workgroup
    int w_pitch;                           // floats per row of W_out in LDS (odd: rows start in different banks), 0: W_out stays in memory
    int gv, gh;                            // log2 of the thread rows over the vocabulary, the hidden columns
    size_t smem;
};
// Few nodes: small workgroups, so that there are enough of them (240 nodes: 60).
inline PlainShape plain_shape(int H, int V, long long rows) {
    auto log2_up = [](int n) { int g = 0; while (g < 6 && (1 << g) < n) ++g; return g; };
    PlainShape s{};
    s.nodes = rows >= 4096 ? 16 : rows >= 1024 ? 8 : 4;
    const size_t row = (size_t)(H + V) * 4;
    while (s.nodes > 1 && s.nodes * row > PLAIN_ROWS) s.nodes /= 2;
    s.w_pitch = (size_t)H * (V | 1) * 4 <= PLAIN_W ? V | 1 : 0;
    s.gv = log2_up(V);
    s.gh = log2_up(H);
    s.smem = s.nodes * row + (size_t)H * s.w_pitch * 4;
    return s;
}

// z[i][H] = tanh(enc_t + pred_u), h[i][V] = scores of the workgroup's n nodes; W: W_out as the caller reads it (LDS or memory, pitch ldw)
struct PlainRows {
    float* z;
    float* h;
    const float* W;
    int ldw;
};
__device__ __forceinline__ PlainRows plain_scores(const Problem& pr, const PlainShape& sh, const NodePos* node, int n, float* smem) {
    const int H = pr.H, V = pr.V, tid = threadIdx.x;
    const float* Wg = (const float*)pr.W;
    PlainRows r{smem, smem + (size_t)sh.nodes * H, Wg, V};
    const int rv = tid >> sh.gv, cv = tid & ((1 << sh.gv) - 1), nv = 256 >> sh.gv;
    if (sh.w_pitch) {
        float* Wl = r.h + (size_t)sh.nodes * V;
        for (int k = rv; k < H; k += nv)
            for (int v = cv; v < V; v += 1 << sh.gv) Wl[k * sh.w_pitch + v] = Wg[(size_t)k * V + v];
        r.W = Wl;
        r.ldw = sh.w_pitch;
    }
    __syncthreads();                       // (the nodes, too)
    for (int i = tid >> sh.gh; i < n; i += 256 >> sh.gh) {
        const float* enc = (const float*)pr.enc + ((size_t)node[i].s * pr.T_max + node[i].t) * H;
        const float* prd = (const float*)pr.pred + ((size_t)node[i].s * (pr.U_max + 1) + node[i].u) * H;
        for (int k = tid & ((1 << sh.gh) - 1); k < H; k += 1 << sh.gh) r.z[i * H + k] = tanhf(enc[k] + prd[k]);
    }
    __syncthreads();
    for (int i = rv; i < n; i += nv)
        for (int v = cv; v < V; v += 1 << sh.gv) {
            float acc = 0.0f;
#pragma unroll 8
            for (int k = 0; k < H; ++k) acc = fmaf(r.z[i * H + k], r.W[(size_t)k * r.ldw + v], acc);
            r.h[i * V + v] = acc + pr.b_out[v];
        }
    return r;
}
// -1: no label here, or one outside the vocabulary, which can not be emitted (a label indexes a row of scores: never beyond its end)
__device__ __forceinline__ int node_label(const Problem& pr, const NodePos& p) {
    const int y = p.u < p.U ? pr.labels[(size_t)p.s * pr.U_max + p.u] : -1;
    return (unsigned)y < (unsigned)pr.V ? y : -1;
}

}  // namespace

// Eq. (4), Eq. (6), f^W_1
__global__ __launch_bounds__(256) void k_fwd_f32(Problem pr, SampleTable st, LatticeState ls, int s0, int s1, long long rows,
                                                 PlainShape sh) {
    extern __shared__ float smem[];
    __shared__ NodePos node[PLAIN_NODES];
    const long long r0 = (long long)blockIdx.x * sh.nodes;
    const int n = rows - r0 < sh.nodes ? (int)(rows - r0) : sh.nodes, V = pr.V;
    if ((int)threadIdx.x < n) node[threadIdx.x] = locate_node(st, ls.row_base, s0, s1, r0 + threadIdx.x);
    const PlainRows rw = plain_scores(pr, sh, node, n, smem);
    __syncthreads();
    const int lane = threadIdx.x & 63;
    for (int i = threadIdx.x >> 6; i < n; i += 4) {
        const float* h = rw.h + i * V;
        float m = RNNT_NEG_INF;
        for (int v = lane; v < V; v += 64) m = fmaxf(m, h[v]);
        const float M = wave_max(m);
        float ssum = 0.0f;
        for (int v = lane; v < V; v += 64) ssum += expf(h[v] - M);
        const float lse = M + logf(wave_sum(ssum));
        if (lane == 0) {
            const int label = node_label(pr, node[i]);
            ls.lse[node[i].idx] = lse;
            ls.em[node[i].idx] = emissions(h[pr.blank] - lse, label >= 0 ? h[label] - lse : EMISSION_FLOOR);
        }
    }
}

// The same where W_out stays in memory: a thread takes an entry of the vocabulary for NB nodes at once, so that W_out is read once for them, and keeps
// running statistics instead of scores (a workgroup then needs 4 H bytes of LDS per node, and several share a compute unit).  Threads stand in rows of
// 64, 128 or 256 over the vocabulary, a row has NB nodes of its own.
// What bounds it: the loads of W_out from L1 and L2, one 256-byte line per wavefront for NB multiply-adds.  Losses alone, one node per wavefront, scores in LDS as
// above, this kernel: H = 1023, V = 4097, 32 k nodes 23.2, 56.0, 7.0 ms; 2 k nodes 4.57, 5.28, 0.90 ms; H = 65, V = 16383, 2 k nodes 1257, 3124, 242 us; H = 30, V = 4097,
// 32 k nodes 730, 1435, 304 us; H = 127, V = 255, 32 k nodes 194, 203, 118 us; H = 301, V = 1001, 240 nodes 180, 137, 48 us.
struct WideShape {
    int g;                                 // log2 of a thread row
    int pitch;                             // floats per joint row in LDS
    int nodes;                             // per workgroup
};
template <int NB>
__global__ __launch_bounds__(256) void k_fwd_f32_wide(Problem pr, SampleTable st, LatticeState ls, int s0, int s1, long long rows, WideShape sh) {
    extern __shared__ __align__(16) float zs[];      // [nodes][pitch]
    __shared__ NodePos node[4 * NB];
    __shared__ float4 part[4][NB];         // per wavefront: maximum, sum, blank, label
    const long long r0 = (long long)blockIdx.x * sh.nodes;
    const int n = rows - r0 < sh.nodes ? (int)(rows - r0) : sh.nodes, H = pr.H, V = pr.V, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid < sh.nodes) node[tid] = locate_node(st, ls.row_base, s0, s1, r0 + (tid < n ? tid : n - 1));
    __syncthreads();
    for (int i = wave; i < sh.nodes; i += 4) {
        const float* enc = (const float*)pr.enc + ((size_t)node[i].s * pr.T_max + node[i].t) * H;
        const float* prd = (const float*)pr.pred + ((size_t)node[i].s * (pr.U_max + 1) + node[i].u) * H;
        for (int k = lane; k < sh.pitch; k += 64) zs[i * sh.pitch + k] = k < H ? tanhf(enc[k] + prd[k]) : 0.0f;
    }
    __syncthreads();
    const int row = tid >> sh.g, G = 1 << sh.g;
    const float* z = zs + row * NB * sh.pitch;
    float m[NB], sum[NB], cap_b[NB], cap_y[NB];
    int label[NB];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        m[i] = -3.402823466e38f;           // (finite: entries that are masked out add nothing to it)
        sum[i] = 0.0f;
        cap_b[i] = cap_y[i] = RNNT_NEG_INF;
        label[i] = node_label(pr, node[row * NB + i]);
    }
    for (int v = tid & (G - 1); v < V; v += G) {
        const float* w = (const float*)pr.W + v;
        float acc[NB] = {};
        int k = 0;
#pragma unroll 2
        for (; k + 4 <= H; k += 4, w += 4 * (size_t)V) {
            float wk[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) wk[j] = w[j * (size_t)V];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const f32x4 zk = *reinterpret_cast<const f32x4*>(z + i * sh.pitch + k);
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i] = fmaf(zk[j], wk[j], acc[i]);
            }
        }
        for (; k < H; ++k, w += V)
#pragma unroll
            for (int i = 0; i < NB; ++i) acc[i] = fmaf(z[i * sh.pitch + k], *w, acc[i]);
        const float b = pr.b_out[v];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const float h = acc[i] + b, d = h - m[i], e = expf(-fabsf(d));
            sum[i] = d > 0.0f ? fmaf(sum[i], e, 1.0f) : sum[i] + e;
            m[i] = fmaxf(m[i], h);
            if (v == pr.blank) cap_b[i] = h;
            if (v == label[i]) cap_y[i] = h;
        }
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const float M = wave_max(m[i]), S = wave_sum(sum[i] * expf(m[i] - M));
        cap_b[i] = wave_max(cap_b[i]);
        cap_y[i] = wave_max(cap_y[i]);
        if (lane == 0) part[wave][i] = make_float4(M, S, cap_b[i], cap_y[i]);
    }
    __syncthreads();
    if (tid < n) {
        // the wavefronts of the node's row
        const int w0 = (tid / NB) << (sh.g - 6), nw = 1 << (sh.g - 6), i = tid % NB;
        float4 p = part[w0][i];
        for (int w = 1; w < nw; ++w) {
            const float4 q = part[w0 + w][i];
            const float M = fmaxf(p.x, q.x);
            p = make_float4(M, p.y * expf(p.x - M) + q.y * expf(q.x - M), fmaxf(p.z, q.z), fmaxf(p.w, q.w));
        }
        const float lse = p.x + logf(p.y) + (p.x - p.x);                   // (an infinite score: NaN)
        ls.lse[node[tid].idx] = lse;
        ls.em[node[tid].idx] = emissions(p.z - lse, node_label(pr, node[tid]) >= 0 ? p.w - lse : EMISSION_FLOOR);
    }
}

// f^W_4 and Algorithm 1 lines 8, 10, 11
__global__ __launch_bounds__(256) void k_bwd_f32(Problem pr, SampleTable st, LatticeState ls, GradOut go, int s0, int s1, long long rows,
                                                 PlainShape sh) {
    extern __shared__ float smem[];
    __shared__ NodePos node[PLAIN_NODES];
    __shared__ RowPost post[PLAIN_NODES];
    __shared__ float lse[PLAIN_NODES];
    __shared__ int label[PLAIN_NODES];
    const long long r0 = (long long)blockIdx.x * sh.nodes;
    const int n = rows - r0 < sh.nodes ? (int)(rows - r0) : sh.nodes, tid = threadIdx.x, H = pr.H, V = pr.V;
    if (tid < n) {
        const NodePos p = locate_node(st, ls.row_base, s0, s1, r0 + tid);
        node[tid] = p;
        post[tid] = row_posteriors(ls, p.idx, p.t, p.u, p.T, p.U, p.s);
        lse[tid] = ls.lse[p.idx];
        label[tid] = node_label(pr, p);
    }
    const PlainRows rw = plain_scores(pr, sh, node, n, smem);
    const int rv = tid >> sh.gv, cv = tid & ((1 << sh.gv) - 1), nv = 256 >> sh.gv;
    // (each thread the scores it has formed itself)
    for (int i = rv; i < n; i += nv) {
        const float off = post[i].log_gamma - lse[i];
        for (int v = cv; v < V; v += 1 << sh.gv) {
            float d = expf(rw.h[i * V + v] + off);
            if (v == pr.blank) d -= post[i].Bk;
            if (v == label[i]) d -= post[i].Yk;
            rw.h[i * V + v] = d;
        }
    }
    __syncthreads();
    for (int v = tid; v < V; v += 256) {
        float sum = 0.0f;
        for (int i = 0; i < n; ++i) sum += rw.h[i * V + v];
        atomicAdd(&go.db[v], sum);
    }
    for (int k = rv; k < H; k += nv)
        for (int v = cv; v < V; v += 1 << sh.gv) {
            float sum = 0.0f;
            for (int i = 0; i < n; ++i) sum = fmaf(rw.z[i * H + k], rw.h[i * V + v], sum);
            atomicAdd(&go.dW[(size_t)k * V + v], sum);
        }
    for (int i = tid >> sh.gh; i < n; i += 256 >> sh.gh) {
        float* d_enc = go.d_enc + ((size_t)node[i].s * pr.T_max + node[i].t) * H;
        float* d_prd = go.d_pred + ((size_t)node[i].s * (pr.U_max + 1) + node[i].u) * H;
        for (int k = tid & ((1 << sh.gh) - 1); k < H; k += 1 << sh.gh) {
            // (in blocks of four sums: one chain over the vocabulary would round at the full size of the sum all along; V = 16383: d_enc 2.9e-6 off,
            // 5.2e-7 with a lane per entry before and 5.2e-7 now)
            float dz = 0.0f;
            for (int v0 = 0; v0 < V; v0 += PLAIN_SUM) {
                const int v1 = v0 + PLAIN_SUM < V ? v0 + PLAIN_SUM : V;
                const float* h = rw.h + i * V;
                const float* w = rw.W + (size_t)k * rw.ldw;
                float part[4] = {};
                int v = v0;
#pragma unroll 2
                for (; v + 4 <= v1; v += 4)
#pragma unroll
                    for (int j = 0; j < 4; ++j) part[j] = fmaf(h[v + j], w[v + j], part[j]);
                for (; v < v1; ++v) part[0] = fmaf(h[v], w[v], part[0]);
                dz += (part[0] + part[1]) + (part[2] + part[3]);
            }
            const float zk = rw.z[i * H + k], dx = dz * (1.0f - zk * zk);
            atomicAdd(&d_enc[k], dx);
            atomicAdd(&d_prd[k], dx);
        }
    }
}

namespace {
template <int NB>
hipError_t launch_fwd_f32_wide(const Problem& pr, const SampleTable& st, const LatticeState& ls, int s0, int s1, long long rows, WideShape sh,
                               hipStream_t stream) {
    sh.nodes = NB * (256 >> sh.g);
    k_fwd_f32_wide<NB><<<dim3((unsigned)((rows + sh.nodes - 1) / sh.nodes)), dim3(256), (size_t)sh.nodes * sh.pitch * 4, stream>>>(pr, st, ls, s0, s1,
                                                                                                                         rows, sh);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_fwd_f32(const Problem& pr, const SampleTable& st, const LatticeState& ls, int s0, int s1,
                          long long rows, hipStream_t stream) {
    if (rows <= 0) return hipSuccess;
    const PlainShape sh = plain_shape(pr.H, pr.V, rows);
    if (sh.w_pitch == 0) {
        // as many nodes at once as leave WIDE_WGS workgroups, and at least four of them on a compute unit
        WideShape w{pr.V <= 64 ? 6 : pr.V <= 128 ? 7 : 8, (pr.H + 3) & ~3, 0};
        const long long rows_wg = 256 >> w.g;
        int nb = 8;
        while (nb > 1 && (rows < WIDE_WGS * rows_wg * nb || rows_wg * nb * w.pitch * 4 > WIDE_LDS)) nb /= 2;
        if (nb == 8) return launch_fwd_f32_wide<8>(pr, st, ls, s0, s1, rows, w, stream);
        if (nb == 4) return launch_fwd_f32_wide<4>(pr, st, ls, s0, s1, rows, w, stream);
        if (nb == 2) return launch_fwd_f32_wide<2>(pr, st, ls, s0, s1, rows, w, stream);
        return launch_fwd_f32_wide<1>(pr, st, ls, s0, s1, rows, w, stream);
    }
    k_fwd_f32<<<dim3((unsigned)((rows + sh.nodes - 1) / sh.nodes)), dim3(256), sh.smem, stream>>>(pr, st, ls, s0, s1, rows, sh);
    return hipGetLastError();
}

hipError_t launch_bwd_f32(const Problem& pr, const SampleTable& st, const LatticeState& ls, const GradOut& go,
                          int s0, int s1, long long rows, hipStream_t stream) {
    if (rows <= 0) return hipSuccess;
    const PlainShape sh = plain_shape(pr.H, pr.V, rows);
    k_bwd_f32<<<dim3((unsigned)((rows + sh.nodes - 1) / sh.nodes)), dim3(256), sh.smem, stream>>>(pr, st, ls, go, s0, s1, rows, sh);
    return hipGetLastError();
}

// ---- fp32 GEMM path ---------------------------------------------------------------------

namespace {

constexpr int FT = 128;       // output tile: 128 rows x TN columns
constexpr int FK = 16;        // K-step
constexpr int FLIP = 1024;    // depth after which the sum changes its sign

// C = A B in fp32 precision on the bf16 matrix instruction.  An fp32 value is the exact sum of three bf16 values, each the rounded rest
// of the ones before: x = h + m + l with |m| <= 2^-9 |x|, |l| <= 2^-18 |x|.  A product takes the six pairs h h, h m, m h, h l, m m, l h; what is
// left out is below 2^-26 of it, a quarter of an fp32 rounding, and 16 products are added per rounding of the accumulator where the fp32
// instruction adds two.  The accumulation rounds towards minus infinity, a mean of 5e-11 of the result's size per unit of depth, alike for all results: sums over
// many of them would show it (d_pred at V = 16384: a mean of -8e-7 of its size, twice the error of the fp32 instruction).  So every FLIP of depth the sum
// changes its sign, and A enters with the other one: what is lost goes the other way (that mean then: 2e-8; 1.1 % of a call's time, 2 % with 256).  Error
// against 64 bits over that of v_mfma_f32_32x32x2_f32, whole calls, 24 seeds each of seven shapes from H = 64, V = 2048 to H = 4096, V = 64: d_enc 0.69 to 0.96, d_pred
// 0.66 to 1.01, dW_out 0.62 to 1.00.  Operands are exact from 2^-110 on; below, what lies under 2^-134 is lost.  Values beyond the largest bf16, 3.39e38, and
// infinities: see the end of the kernel.
// The bf16 instruction does sixteen times the work of the fp32 one, a sixth of it still 2.7 times.  What bounds it: power (1.7 GHz, matrix pipes busy
// 64 to 67 % of the time; 200 TFLOP/s against 123 to 130 with the fp32 instruction).  H = 1024, V = 4096, 131 k nodes: a call 37.2 -> 22.8 ms.
// The parts are formed on the way into LDS, so the operands stay as they are in memory.
// One part of two values, which leave as what remains of them.
__device__ __forceinline__ unsigned split_part(float& x0, float& x1) {
    unsigned p;
    // (as text: the compiler otherwise converts the first of the two once more by itself)
    asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(p) : "v"(x0), "v"(x1));
    x0 -= __uint_as_float(p << 16);
    x1 -= __uint_as_float(p & 0xffff0000u);
    return p;
}

// One operand of the tile product, ROWS rows (m for A, n for B) x FK.  KSLOW = false: element (i, k) at p[i*ld + k]; true: at p[k*ld + i].
// EDGE: elements with i >= n_i or k >= n_k, and those of a padded source row (the row index is i if !KSLOW, k if KSLOW; see RowMask), read as
// zero.  The extent along the contiguous index is a multiple of 4, so a 16-byte piece is inside or outside as a whole.  Branch-free: a
// piece outside is loaded from the operand's first element and cleared.
// In LDS: blocks of 32 rows, each three MFMA fragments of 1 KiB (the three parts), in a fragment 64 granules of 16 bytes: 8 consecutive k (half kh) of
// one row, the row's place r at granule 32 kh + (r ^ 12 kh) (the xor spreads a write of both halves over all banks).  The place of row
// i is i for a k-contiguous operand; a k-slow one, whose threads hold four consecutive rows of two k, puts row i at i / 4 + 8 (i % 4), so that eight
// threads write 128 bytes in one piece.
template <bool KSLOW, bool EDGE, int ROWS>
struct OperandF32 {
    const float* p;
    long long ld;
    long long n_i, n_k;
    RowMask mask;
    static constexpr int NQ = ROWS / 64;              // 16-byte pieces per thread and step
    // 16-byte piece q of the step at k0 (i0, k0 uniform)
    __device__ __forceinline__ f32x4 piece(long long i0, long long k0, int q, int tid) const {
        const int lane = tid & 63, wave = tid >> 6;
        const int di = KSLOW ? wave * 32 + (lane & 7) * 4 : tid >> 2, dk = KSLOW ? (lane >> 3) * 2 : (tid & 3) * 4;
        i0 += KSLOW ? (q >> 1) * 128 : q * 64;
        k0 += KSLOW ? q & 1 : 0;
        if constexpr (!EDGE) {
            const unsigned voff = (unsigned)(KSLOW ? dk * (int)ld + di : di * (int)ld + dk) * 4u;
            const float* base = p + (KSLOW ? k0 * ld + i0 : i0 * ld + k0);
            return *reinterpret_cast<const f32x4*>(reinterpret_cast<const char*>(base) + voff);
        }
        const long long i = i0 + di, k = k0 + dk, off = !KSLOW ? i * ld + k : k * ld + i;
        const bool ok = i < n_i && k < n_k;
        bool keep = ok;
        if (mask.len != nullptr) {
            const long long src = ok ? (!KSLOW ? i : k) : 0, b = src / mask.period;
            keep = ok && (int)(src - b * mask.period) < mask.len[b] + mask.extra;
        }
        u32x4 w = __builtin_bit_cast(u32x4, *reinterpret_cast<const f32x4*>(p + (ok ? off : 0)));
        w &= keep ? ~0u : 0u;
        return __builtin_bit_cast(f32x4, w);
    }
    __device__ __forceinline__ void fetch(f32x4 (&v)[NQ], long long i0, long long k0, int tid) const {
#pragma unroll
        for (int q = 0; q < NQ; ++q) v[q] = piece(i0, k0, q, tid);
    }
    // The work of bringing a step's pieces into LDS, cut into units of about five vector instructions and one LDS write: part n / 3 ... of two values
    // (k-contiguous operands: every second unit, with ten, of four).  The last unit of a piece loads that of the step at k2.
    // The values enter with the sign bit of `sign` flipped.
    static constexpr int UNITS = 6 * NQ;
    template <int U>
    __device__ __forceinline__ void unit(f32x4 (&v)[NQ], unsigned char* tile, int tid, long long i0, long long k2, unsigned sign) const {
        auto flip = [&](float x) { return __uint_as_float(__float_as_uint(x) ^ sign); };
        if constexpr (!KSLOW) {
            if constexpr (U % 2 == 0) {
                constexpr int q = U / 6, part = U % 6 / 2;
                const int r = (tid >> 2) & 31, kp = tid & 3, kh = kp >> 1;
                float x[4] = {v[q][0], v[q][1], v[q][2], v[q][3]};
                if constexpr (part == 0)
#pragma unroll
                    for (int j = 0; j < 4; ++j) x[j] = flip(x[j]);
                const unsigned a = split_part(x[0], x[1]), b = split_part(x[2], x[3]);
                v[q] = f32x4{x[0], x[1], x[2], x[3]};
                *reinterpret_cast<uint2*>(tile + (tid >> 7) * 3072 + q * 6144 + part * 1024 + kh * 512 + (r ^ (12 * kh)) * 16 + (kp & 1) * 8) =
                    make_uint2(a, b);
                if constexpr (part == 2) v[q] = piece(i0, k2, q, tid);
            }
        } else {
            constexpr int q = U / 12 * 2, c = U % 12 / 3, part = U % 3;
            const int lane = tid & 63, wave = tid >> 6, kp = lane >> 3, kh = kp >> 2;
            float x0 = v[q][c], x1 = v[q + 1][c];
            if constexpr (part == 0) {
                x0 = flip(x0);
                x1 = flip(x1);
            }
            *reinterpret_cast<unsigned*>(tile + wave * 3072 + q * 6144 + part * 1024 + kh * 512 +
                                         (((lane & 7) ^ (4 * kh)) + ((8 * c) ^ (8 * kh))) * 16 + (kp & 3) * 4) = split_part(x0, x1);
            v[q][c] = x0;
            v[q + 1][c] = x1;
            if constexpr (U % 12 == 11) {
                v[q] = piece(i0, k2, q, tid);
                v[q + 1] = piece(i0, k2, q + 1, tid);
            }
        }
    }
    // one value as it is
    __device__ __forceinline__ float value(long long i, long long k) const {
        bool keep = !EDGE || (i < n_i && k < n_k);
        if (EDGE && mask.len != nullptr) {
            const long long src = keep ? (!KSLOW ? i : k) : 0, b = src / mask.period;
            keep = keep && (int)(src - b * mask.period) < mask.len[b] + mask.extra;
        }
        const float x = p[keep ? (!KSLOW ? i * ld + k : k * ld + i) : 0];
        return keep ? x : 0.0f;
    }
    // row of a block that stands at place r
    static __device__ __forceinline__ int row_at(int r) { return KSLOW ? (r & 7) * 4 + (r >> 3) : r; }
};

// C[m, n] (+)= sum_k A(m, k) B(k, n) (+ bias[n]) in fp32.  128 x TN output tile per workgroup, 4 waves x (64 x TN/2) = 2 x TN/64 MFMA tiles of
// 32 x 32, six MFMAs of depth 16 each per K-step; two LDS buffers, one barrier per K-step, global loads two K-steps ahead of their MFMAs in registers.
// Two workgroups per compute unit (72 KiB of LDS and 256 registers each; three of 128 x 128): one's splitting stands beside the other's MFMAs.
// grid (M/128, N/TN, splits); a split covers k_per_split (a multiple of 16) of K.  atomic != 0: the tile
// is added to C with float atomics (split over K, or C accumulates over calls).
template <int TN, class OpA, class OpB>
__global__ __launch_bounds__(256, TN == 256 ? 2 : 3) void k_gemm_f32(OpA A, OpB B, float* __restrict__ C, long long ldc,
                                                     const float* __restrict__ bias, int atomic, long long M,
                                                     long long N, long long K, long long k_per_split) {
    constexpr int NT = TN / 64;                       // MFMA tiles of a wave along N
    constexpr unsigned A_BYTES = FT / 32 * 3072, BUF = A_BYTES + TN / 32 * 3072;
    __shared__ __align__(16) unsigned char smem[2 * BUF];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, hb = lane >> 5;
    const int wm = wave >> 1, wn = wave & 1;
    const long long m0 = (long long)blockIdx.x * FT, n0 = (long long)blockIdx.y * TN;
    const long long ks = (long long)blockIdx.z * k_per_split;
    const long long ke = ks + k_per_split < K ? ks + k_per_split : K;
    if (ks >= ke) return;
    f32x16 acc[2][NT];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = f32x16{0};
    f32x4 va[OpA::NQ], vb[OpB::NQ];
    const unsigned frag = hb * 512u + (unsigned)(l32 ^ (12 * hb)) * 16u;
    const unsigned char* fa0 = smem + wm * 2 * 3072 + frag;
    const unsigned char* fb0 = smem + A_BYTES + wn * NT * 3072 + frag;
    const long long last = ks + (ke - ks - 1) / FK * FK;
    // unit w of a step: of B's, then of A's (with `sign`); into buffer `buf`; the loads that follow them take the step at k2
    constexpr int UNITS = OpA::UNITS + OpB::UNITS;
    auto unit = [&](auto w_tag, unsigned buf, long long k2, unsigned sign) {
        constexpr int w = decltype(w_tag)::value;
        if constexpr (w < OpB::UNITS) B.template unit<w>(vb, smem + buf + A_BYTES, tid, n0, k2, 0u);
        else A.template unit<w - OpB::UNITS>(va, smem + buf, tid, m0, k2, sign);
    };
    auto negate = [&] {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[i][j] = -acc[i][j];
    };
    A.fetch(va, m0, ks, tid);
    B.fetch(vb, n0, ks, tid);
    static_for<0, UNITS>([&](auto w) { unit(w, 0u, ks + FK < last ? ks + FK : last, 0u); });
    __syncthreads();
    unsigned cur = 0;
    for (long long k0 = ks; k0 < ke; k0 += FK, cur ^= BUF) {
        // (past the end: the last step again, into a buffer nobody reads any more)
        const long long k2 = k0 + 2 * FK < last ? k0 + 2 * FK : last;
        if (k0 > ks && ((k0 - ks) & (FLIP - 1)) == 0) negate();
        const unsigned sign = ((k0 - ks + FK) & FLIP) ? 0x80000000u : 0u;        // of the step being staged
        bf16x8 fa[2][3], fb[2][3];
        auto frag_b = [&](auto j_tag, int c) {
            constexpr int j = decltype(j_tag)::value;
            fb[j & 1][c] = *reinterpret_cast<const bf16x8*>(fb0 + cur + (j * 3 + c) * 1024);
        };
#pragma unroll
        for (int c = 2; c >= 0; --c) {
            fa[0][2 - c] = *reinterpret_cast<const bf16x8*>(fa0 + cur + (2 - c) * 1024);
            frag_b(std::integral_constant<int, 0>{}, c);
            fa[1][2 - c] = *reinterpret_cast<const bf16x8*>(fa0 + cur + (3 + 2 - c) * 1024);
        }
        // Behind each MFMA (it holds the matrix pipe for 32 clocks and the issue port for four) a share of the next step's staging: the buffer's last
        // readers have passed the barrier that ended the step before.
        static_for<0, 12 * NT>([&](auto g_tag) {
            constexpr int g = decltype(g_tag)::value, j = g / 12, i = g & 1, pr = g % 12 / 2;
            // the small products first: (part of A, part of B)
            constexpr int pa[6] = {0, 1, 2, 0, 1, 0}, pb[6] = {2, 1, 0, 1, 0, 0};
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i][pa[pr]], fb[j & 1][pb[pr]], acc[i][j], 0, 0, 0);
            if constexpr (j + 1 < NT && g % 12 >= 3 && g % 12 < 6) frag_b(std::integral_constant<int, j + 1>{}, 5 - g % 12);
            constexpr int w0 = g * UNITS / (12 * NT), w1 = (g + 1) * UNITS / (12 * NT);
            static_for<w0, w1>([&](auto w) { unit(w, cur ^ BUF, k2, sign); });
            __builtin_amdgcn_sched_barrier(0);
        });
        __syncthreads();
    }
    if ((ke - ks - 1) & FLIP) negate();
    // accumulator register 4q+r of tile (i,j): place 8q + 4hb + r along M, l32 along N
    auto store = [&](const f32x16& d, int i, int j) {
        const long long n = n0 + (wn * NT + j) * 32 + OpB::row_at(l32);
        if (n >= N) return;
        const float bv = (bias != nullptr && blockIdx.z == 0) ? bias[n] : 0.0f;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const long long m = m0 + wm * 64 + i * 32 + OpA::row_at(8 * (q >> 2) + 4 * hb + (q & 3));
            if (m >= M) continue;
            const float v = d[q] + bv;
            if (atomic) atomicAdd(C + m * ldc + n, v);
            else C[m * ldc + n] = v;
        }
    };
    // An operand that is infinite, or beyond the largest bf16, has no three parts: its rest is infinite or NaN, and so is every sum it enters.  A wave
    // that holds such a sum forms its sums again, of the values as they are, on the fp32 instruction, tile after tile, unless NaN among its operands are
    // the reason (padding, which may hold anything; a sample without an alignment): they give NaN either way.  (Projections of 400 frames, D = 512, whose
    // padding is NaN: a call 390 -> 418 us; without the search for NaN 831.)
    float odd = 0.0f;                                 // NaN if one is infinite or NaN
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int q = 0; q < 16; ++q) odd = fmaf(acc[i][j][q], 0.0f, odd);
    bool again = __any(odd != 0.0f);
    int place = l32;
    asm volatile("" : "+v"(place));                   // (nothing below is formed ahead of the main loop)
    if (again) {
        // a bit per place: the infinite and NaN sums of this lane's column (tile by tile), NaN found so far in the rows of A, the columns of B
        unsigned sums[2][NT], nan_a[2] = {}, nan_b[NT] = {};
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) {
                unsigned m = 0;
#pragma unroll
                for (int q = 0; q < 16; ++q) m |= fabsf(acc[i][j][q]) < -RNNT_NEG_INF ? 0u : 1u << (8 * (q >> 2) + (q & 3));
                sums[i][j] = m << (4 * hb);
            }
        auto places = [](bool x) {
            const unsigned long long m = __builtin_amdgcn_ballot_w64(x);
            return (unsigned)m | (unsigned)(m >> 32);
        };
        auto unexplained = [&] {
            unsigned u = 0;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j) u |= (nan_b[j] >> place) & 1u ? 0u : sums[i][j] & ~nan_a[i];
            return (bool)__any(u != 0);
        };
        long long k0 = ks;
        while (k0 < ke && (again = unexplained())) {
            const long long k1 = k0 + 64 < ke ? k0 + 64 : ke;
            bool na[2] = {}, nb[NT] = {};
#pragma unroll 1
            for (long long k = k0; k < k1; k += 2) {
#pragma unroll
                for (int i = 0; i < 2; ++i) na[i] |= __builtin_isnan(A.value(m0 + wm * 64 + i * 32 + OpA::row_at(place), k + hb));
#pragma unroll
                for (int j = 0; j < NT; ++j) nb[j] |= __builtin_isnan(B.value(n0 + (wn * NT + j) * 32 + OpB::row_at(place), k + hb));
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) nan_a[i] |= places(na[i]);
#pragma unroll
            for (int j = 0; j < NT; ++j) nan_b[j] |= places(nb[j]);
            k0 = k1;
        }
        if (again) again = unexplained();
    }
    if (again) {
#pragma unroll 1
        for (int t = 0; t < 2 * NT; ++t) {
            const int i = t & 1, j = t >> 1;
            const long long m = m0 + wm * 64 + i * 32 + OpA::row_at(place), n = n0 + (wn * NT + j) * 32 + OpB::row_at(place);
            f32x16 d = f32x16{0};
#pragma unroll 1
            for (long long k = ks; k < ke; k += 2)    // (beyond the end of a sum: zeros of both operands)
                d = __builtin_amdgcn_mfma_f32_32x32x2f32(A.value(m, k + hb), B.value(n, k + hb), d, 0, 0, 0);
            store(d, i, j);
        }
    } else {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) store(acc[i][j], i, j);
    }
}

struct GemmF32 {
    const float* A;
    long long lda;
    RowMask ma;
    const float* B;
    long long ldb;
    RowMask mb;
    float* C;
    long long ldc;
    const float* bias;
    int atomic;
    long long M, N, K;
    int splits;
};

template <bool AK, bool BK, bool EDGE, int TN>
hipError_t launch_gemm_f32_t(const GemmF32& g, hipStream_t stream) {
    long long per = (g.K + g.splits - 1) / g.splits;
    per = (per + FK - 1) / FK * FK;
    const long long nz = (g.K + per - 1) / per, gm = (g.M + FT - 1) / FT, gn = (g.N + TN - 1) / TN;
    if (gm > 0x7fffffffLL || gn > 65535 || nz > 65535) return hipErrorInvalidValue;
    const OperandF32<AK, EDGE, FT> a{g.A, g.lda, g.M, g.K, g.ma};
    const OperandF32<BK, EDGE, TN> b{g.B, g.ldb, g.N, g.K, g.mb};
    k_gemm_f32<TN><<<dim3((unsigned)gm, (unsigned)gn, (unsigned)nz), dim3(256), 0, stream>>>(a, b, g.C, g.ldc, g.bias, g.atomic, g.M, g.N,
                                                                                        g.K, per);
    return hipGetLastError();
}

// Splits of a sum over K rows: about 512 workgroups of 128 x 128 in all, at least 128 rows each; long sums (4096 rows and more per split) in as many as
// 512 workgroups of 128 x 256 take (H = 1024, V = 4096, 33 k rows: 1323 -> 1190 us; with 4500 rows, H = 512, V = 1024, the atomics of so many splits
// cost more: a call 245 -> 260 us); at most 16384 rows per split, so that no sum's rounding grows beyond that of the longest one over the vocabulary
// (and whole rounds of those workgroups: H = 1024, V = 4096, 73 k rows, five splits in three rounds of narrow tiles -> eight in two of wide ones: a call of 16 samples of up to
// 500 x 100 in a workspace that holds such chunks 79.9 -> 78.7 ms).
}  // namespace
int k_splits_f32(long long M, long long N, long long K) {
    const long long rows = (M + FT - 1) / FT, narrow = rows * ((N + 127) / 128), wide = rows * ((N + 255) / 256);
    long long s = std::min((512 + narrow - 1) / narrow, (K + FT - 1) / FT);
    const long long full = (512 + wide - 1) / wide;
    if (K >= 4096 * s) s = std::max(s, full);
    if (K > 16384 * s) s = ((K + 16383) / 16384 + full - 1) / full * full;
    return (int)std::max(1LL, s);
}
namespace {

// Tiles of 256 or 128 columns: the fewer rounds of the chip (two workgroups per compute unit), a narrow one costing 0.6 of a wide one.
inline bool wide_tiles_pay(long long M, long long N, int splits) {
    const long long rows = (M + FT - 1) / FT * splits;
    const long long wide = (rows * ((N + 255) / 256) + 511) / 512, narrow = (rows * ((N + 127) / 128) + 511) / 512;
    return 10 * wide <= 6 * narrow;
}

// Without edge handling where M, N, K are multiples of the tile and no row is masked, else with it.
template <bool AK, bool BK>
hipError_t launch_gemm_f32(const GemmF32& g, hipStream_t stream) {
    if (g.M <= 0 || g.N <= 0 || g.K <= 0) return hipSuccess;
    // 16-byte pieces along each operand's contiguous index
    const bool fits = g.lda % 4 == 0 && g.ldb % 4 == 0 && (AK ? g.M : g.K) % 4 == 0 && (BK ? g.N : g.K) % 4 == 0 &&
                      (uintptr_t)g.A % 16 == 0 && (uintptr_t)g.B % 16 == 0;
    if (!fits || g.splits < 1 || (g.splits > 1 && !g.atomic)) return hipErrorInvalidValue;
    const bool wide = wide_tiles_pay(g.M, g.N, g.splits);
    const bool edge = g.ma.len != nullptr || g.mb.len != nullptr || g.M % FT != 0 || g.N % (wide ? 256 : 128) != 0 || g.K % FK != 0;
    if (wide) return edge ? launch_gemm_f32_t<AK, BK, true, 256>(g, stream) : launch_gemm_f32_t<AK, BK, false, 256>(g, stream);
    return edge ? launch_gemm_f32_t<AK, BK, true, 128>(g, stream) : launch_gemm_f32_t<AK, BK, false, 128>(g, stream);
}

// Row i of the chunk is lattice node r0 + i of the group (i < n), or padding (n <= i < gridDim.x).
// Z[i, :] = tanh(enc_t + pred_u), zero in padding rows.
__global__ __launch_bounds__(256) void k_rows_z_f32(Problem pr, SampleTable st, LatticeState ls, int s0, int s1,
                                                    long long r0, long long n, float* __restrict__ Z) {
    const long long i = blockIdx.x;
    const int H = pr.H;
    float* z = Z + i * H;
    if (i >= n) {
        for (int k = threadIdx.x; k < H; k += 256) z[k] = 0.0f;
        return;
    }
    const NodePos p = locate_node(st, ls.row_base, s0, s1, r0 + i);
    const float* enc = (const float*)pr.enc + ((size_t)p.s * pr.T_max + p.t) * H;
    const float* prd = (const float*)pr.pred + ((size_t)p.s * (pr.U_max + 1) + p.u) * H;
    for (int k = threadIdx.x; k < H; k += 256) z[k] = tanhf(enc[k] + prd[k]);
}

// f^W_1 for one row of scores per wavefront (4 rows per workgroup): lse, emissions of node r0 + i.  Bound by reading the scores: once, where a row fits
// the registers of a wavefront (Q pieces of 16 bytes per lane; Q = 0: twice, whatever its length).  V = 4096, 31 k rows: 116 us (4.4 TB/s; two passes
// took 165).
template <int Q>
__global__ __launch_bounds__(256) void k_rows_stats_f32(Problem pr, SampleTable st, LatticeState ls, int s0, int s1,
                                                        long long r0, long long n, const float* __restrict__ S) {
    const long long i = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (i >= n) return;
    const int lane = threadIdx.x & 63, V = pr.V;
    const float* row = S + i * V;
    const f32x4* row4 = reinterpret_cast<const f32x4*>(row);      // V is a multiple of 4, rows are 16-byte aligned
    f32x4 x[Q ? Q : 1];
    float m = RNNT_NEG_INF;
    if constexpr (Q > 0) {
#pragma unroll
        for (int q = 0; q < Q; ++q) x[q] = lane + 64 * q < V / 4 ? row4[lane + 64 * q] : f32x4{RNNT_NEG_INF, RNNT_NEG_INF, RNNT_NEG_INF, RNNT_NEG_INF};
#pragma unroll
        for (int q = 0; q < Q; ++q) m = fmaxf(fmaxf(m, fmaxf(x[q][0], x[q][1])), fmaxf(x[q][2], x[q][3]));
    } else {
        for (int v = lane; v < V / 4; v += 64) {
            const f32x4 y = row4[v];
            m = fmaxf(fmaxf(m, fmaxf(y[0], y[1])), fmaxf(y[2], y[3]));
        }
    }
    const NodePos p = locate_node(st, ls.row_base, s0, s1, r0 + i);
    const int label = node_label(pr, p);
    const float M = wave_max(m);
    float ssum = 0.0f;
    auto add = [&](const f32x4& y) { ssum += (expf(y[0] - M) + expf(y[1] - M)) + (expf(y[2] - M) + expf(y[3] - M)); };
    if constexpr (Q > 0) {
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (lane + 64 * q < V / 4) add(x[q]);
    } else {
        for (int v = lane; v < V / 4; v += 64) add(row4[v]);
    }
    const float lse = M + logf(wave_sum(ssum));
    if (lane == 0) {
        ls.lse[p.idx] = lse;
        ls.em[p.idx] = emissions(row[pr.blank] - lse, label >= 0 ? row[label] - lse : EMISSION_FLOOR);
    }
}

// f^W_4 in place of the scores: dh = gamma softmax - posteriors, zero in padding rows; db += its column sums.  A workgroup takes 4 << lc columns and
// `rows` rows (a multiple of four per thread; the threads stand in rows of 1 << lc), so that the sums cost no further pass (31 k rows, V = 4096: 180 us,
// one pass for dh and one for the sums 178 and 133).
constexpr int DH_PER_THREAD = 128, DH_ROWS_MAX = DH_PER_THREAD * 16;
struct DhShape {
    int lc;                                           // threads over the vocabulary: 16 to 64
    int rows;                                         // per workgroup
};
// Rows: as many as leave about 128 workgroups down the chunk (additions to one address follow each other at about 0.1 us; with 1177 workgroups of 1024
// columns a call of 14 k rows, H = 256, V = 1024 took 376 us, now 267), at most 128 per thread.
inline DhShape dh_shape(int V, long long np) {
    DhShape s{4, 0};
    while (s.lc < 6 && (4 << s.lc) < V) ++s.lc;
    const long long groups = 256 >> s.lc;
    long long per = np / (128 * groups) / 4 * 4;
    per = per < 4 ? 4 : per > DH_PER_THREAD ? DH_PER_THREAD : per;
    s.rows = (int)(per * groups);
    return s;
}
__global__ __launch_bounds__(256) void k_rows_dh_f32(Problem pr, SampleTable st, LatticeState ls, int s0, int s1,
                                                     long long r0, long long n, long long n_padded, DhShape sh,
                                                     float* __restrict__ S, float* __restrict__ db) {
    __shared__ __align__(16) float row_data[DH_ROWS_MAX][4];      // offset of the exponent, what is taken off at the blank and the label, the label
    const long long i0 = (long long)blockIdx.x * sh.rows;
    const int tid = threadIdx.x, V = pr.V, rows = n_padded - i0 < sh.rows ? (int)(n_padded - i0) : sh.rows;
    for (int r = tid; r < rows; r += 256) {
        f32x4 d = f32x4{RNNT_NEG_INF, 0.0f, 0.0f, __int_as_float(-1)};
        if (i0 + r < n) {
            const NodePos p = locate_node(st, ls.row_base, s0, s1, r0 + i0 + r);
            const RowPost rp = row_posteriors(ls, p.idx, p.t, p.u, p.T, p.U, p.s);
            d = f32x4{rp.log_gamma - ls.lse[p.idx], rp.Bk, rp.Yk, __int_as_float(node_label(pr, p))};
        }
        *reinterpret_cast<f32x4*>(row_data[r]) = d;
    }
    __syncthreads();
    const int cols = 1 << sh.lc, groups = 256 >> sh.lc, c = tid & (cols - 1);
    const int v = ((int)blockIdx.y << (sh.lc + 2)) + c * 4;
    f32x4 sum = f32x4{0};
    if (v < V) {
        float* col = S + i0 * V + v;
        for (int q = tid >> sh.lc; q < rows; q += 4 * groups) {
            f32x4 x[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = q + j * groups < rows ? q + j * groups : q;     // (loads without branches between them)
                x[j] = *reinterpret_cast<const f32x4*>(col + (long long)r * V);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = q + j * groups;
                if (r >= rows) continue;
                const f32x4 rd = *reinterpret_cast<const f32x4*>(row_data[r]);
                const int label = __float_as_int(rd[3]);
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    float d = expf(x[j][k] + rd[0]);
                    if (v + k == pr.blank) d -= rd[1];
                    if (v + k == label) d -= rd[2];
                    x[j][k] = d;
                }
                if (i0 + r >= n) x[j] = f32x4{0};
                sum += x[j];
                *reinterpret_cast<f32x4*>(col + (long long)r * V) = x[j];
            }
        }
    }
    __syncthreads();                                  // row_data becomes [groups][4 cols] partial sums
    *reinterpret_cast<f32x4*>(row_data[tid]) = sum;
    __syncthreads();
    const float* part = &row_data[0][0];
    const int vt = ((int)blockIdx.y << (sh.lc + 2)) + tid;
    if (tid >= 4 * cols || vt >= V) return;
    float t = 0.0f;
    for (int g = 0; g < groups; ++g) t += part[g * 4 * cols + tid];
    atomicAdd(db + vt, t);
}

// d_enc[s, t, :] += dZ (1 - Z^2), d_pred[s, u, :] += the same: a lattice tile and 256 columns per workgroup (a wavefront takes every eighth frame, a lane
// four columns), summed over the tile's labels resp. frames before it leaves: 16 to 20 atomics a column and tile, where a node by itself takes 128
// (31 k nodes, H = 1024: 240 -> 60 us).  Nodes [r0, r0 + n) of the group have a row in Z and dZ; a tile may have others besides.  A wavefront's 8 nodes are
// loaded ahead of the first sum, so that a small call waits for memory once: with four wavefronts that took a frame at a time four samples of 30 x 8,
// H = 64, took 6.9 us, now 4.2, eight of 100 x 20, H = 512, 19.8, now 16.5.
// UW: the tile's label positions.
template <int UW>
__device__ __forceinline__ void rows_dz_tile(const Problem& pr, const TilePos& p, long long first, long long n, const float* __restrict__ Z,
                                             const float* __restrict__ dZ, float* __restrict__ d_enc, float* __restrict__ d_pred,
                                             float (&part)[8][8][256]) {
    constexpr int FRAMES = 8 / UW;                    // of a wavefront
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, H = pr.H;
    const int h0 = (int)blockIdx.y * 256, h = h0 + lane * 4;
    const bool col = h < H;
    f32x4 z[FRAMES][UW], g[FRAMES][UW];
    auto row = [&](int f) { return first + (long long)(p.t0 + wave + 8 * f) * (p.U + 1) + p.u0; };
#pragma unroll
    for (int f = 0; f < FRAMES; ++f)
#pragma unroll
        for (int u = 0; u < UW; ++u) {                // (loads without branches between them: what is not a row of the chunk reads another one)
            long long i = row(f) + u;
            i = i < 0 ? 0 : i < n ? i : n - 1;
            z[f][u] = *reinterpret_cast<const f32x4*>(Z + i * H + (col ? h : 0));
            g[f][u] = *reinterpret_cast<const f32x4*>(dZ + i * H + (col ? h : 0));
        }
    f32x4 pu[UW];
#pragma unroll
    for (int u = 0; u < UW; ++u) pu[u] = f32x4{0};
#pragma unroll
    for (int f = 0; f < FRAMES; ++f) {
        const int t = p.t0 + wave + 8 * f;
        f32x4 de = f32x4{0};
        bool any = false;
#pragma unroll
        for (int u = 0; u < UW; ++u) {
            const long long i = row(f) + u;
            const bool ok = t < p.T && p.u0 + u <= p.U && i >= 0 && i < n && col;
            any = any || ok;
            f32x4 dx = g[f][u] * (1.0f - z[f][u] * z[f][u]);
#pragma unroll
            for (int j = 0; j < 4; ++j) dx[j] = ok ? dx[j] : 0.0f;
            de += dx;
            pu[u] += dx;
        }
        // (through LDS, so that the lanes of an atomic lie side by side)
        *reinterpret_cast<f32x4*>(&part[wave][0][lane * 4]) = de;
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (__any(any)) {
            float* out = d_enc + ((size_t)p.s * pr.T_max + t) * H + h0;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (h0 + j * 64 + lane < H) atomicAdd(out + j * 64 + lane, part[wave][0][j * 64 + lane]);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
#pragma unroll
    for (int u = 0; u < UW; ++u) *reinterpret_cast<f32x4*>(&part[wave][u][lane * 4]) = pu[u];
    __syncthreads();
    const int c = threadIdx.x & 255, hc = h0 + c;
    if (hc >= H) return;
#pragma unroll
    for (int i = 0; i < UW / 2; ++i) {
        const int u = 2 * i + (int)(threadIdx.x >> 8);
        if (p.u0 + u <= p.U)
            atomicAdd(d_pred + ((size_t)p.s * (pr.U_max + 1) + p.u0 + u) * H + hc,
                      ((part[0][u][c] + part[1][u][c]) + (part[2][u][c] + part[3][u][c])) +
                          ((part[4][u][c] + part[5][u][c]) + (part[6][u][c] + part[7][u][c])));
    }
}
__global__ __launch_bounds__(512, 4) void k_rows_dz_f32(Problem pr, SampleTable st, LatticeState ls, int tile0,
                                                        long long r0, long long n, const float* __restrict__ Z,
                                                        const float* __restrict__ dZ, float* __restrict__ d_enc,
                                                        float* __restrict__ d_pred) {
    __shared__ __align__(16) float part[8][8][256];
    const TilePos p = locate_tile(st, tile0 + (int)blockIdx.x);
    const long long first = st.row_off[p.s] - ls.row_base - r0;        // row of the sample's first node
    if (p.uw == 8) rows_dz_tile<8>(pr, p, first, n, Z, dZ, d_enc, d_pred, part);
    else rows_dz_tile<4>(pr, p, first, n, Z, dZ, d_enc, d_pred, part);
}

}  // namespace

bool gemm_f32_edge_fits(const void* A, long long lda, const void* B, long long ldb, long long a_contig_extent,
                        long long b_contig_extent) {
    return lda % 4 == 0 && ldb % 4 == 0 && a_contig_extent % 4 == 0 && b_contig_extent % 4 == 0 &&
           (uintptr_t)A % 16 == 0 && (uintptr_t)B % 16 == 0;
}

hipError_t launch_gemm_f32_masked(int a_kslow, int b_kslow, const float* A, long long lda, const RowMask& ma,
                                  const float* B, long long ldb, const RowMask& mb, float* C, long long ldc,
                                  const float* bias, int atomic, long long M, long long N, long long K, int splits,
                                  hipStream_t stream) {
    const GemmF32 g{A, lda, ma, B, ldb, mb, C, ldc, bias, atomic, M, N, K, splits};
    if (!a_kslow && b_kslow) return launch_gemm_f32<false, true>(g, stream);
    if (!a_kslow && !b_kslow) return launch_gemm_f32<false, false>(g, stream);
    if (a_kslow && b_kslow) return launch_gemm_f32<true, true>(g, stream);
    return hipErrorInvalidValue;
}

namespace {
// The GEMM of the joint path (no padded source rows)
template <bool AK, bool BK>
hipError_t joint_gemm_f32(const float* A, long long lda, const float* B, long long ldb, float* C, long long ldc,
                          const float* bias, int atomic, long long M, long long N, long long K, int splits,
                          hipStream_t stream) {
    const RowMask none{nullptr, 1, 0};
    return launch_gemm_f32<AK, BK>(GemmF32{A, lda, none, B, ldb, none, C, ldc, bias, atomic, M, N, K, splits}, stream);
}
}  // namespace

hipError_t launch_fwd_f32_gemm(const Problem& pr, const SampleTable& st, const LatticeState& ls, int s0, int s1,
                               long long r0, long long n, float* S, float* Z, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    const long long np = (n + FT - 1) / FT * FT;
    k_rows_z_f32<<<dim3((unsigned)np), dim3(256), 0, stream>>>(pr, st, ls, s0, s1, r0, n, Z);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    e = joint_gemm_f32<false, true>(Z, pr.H, (const float*)pr.W, pr.V, S, pr.V, pr.b_out, 0, np, pr.V, pr.H, 1, stream);
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)((n + 3) / 4));
    if (pr.V <= 1024) k_rows_stats_f32<4><<<grid, dim3(256), 0, stream>>>(pr, st, ls, s0, s1, r0, n, S);
    else if (pr.V <= 4096) k_rows_stats_f32<16><<<grid, dim3(256), 0, stream>>>(pr, st, ls, s0, s1, r0, n, S);
    else k_rows_stats_f32<0><<<grid, dim3(256), 0, stream>>>(pr, st, ls, s0, s1, r0, n, S);
    return hipGetLastError();
}

hipError_t launch_bwd_f32_gemm(const Problem& pr, const SampleTable& st, const LatticeState& ls, const GradOut& go,
                               int s0, int s1, int tile0, int tile1, long long r0, long long n, bool have_scores, float* S, float* Z,
                               float* dZ, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    const long long np = (n + FT - 1) / FT * FT;
    const int H = pr.H, V = pr.V;
    const float* W = (const float*)pr.W;
    hipError_t e = hipSuccess;
    if (!have_scores) {
        k_rows_z_f32<<<dim3((unsigned)np), dim3(256), 0, stream>>>(pr, st, ls, s0, s1, r0, n, Z);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        e = joint_gemm_f32<false, true>(Z, H, W, V, S, V, pr.b_out, 0, np, V, H, 1, stream);
        if (e != hipSuccess) return e;
    }
    const DhShape sh = dh_shape(V, np);
    k_rows_dh_f32<<<dim3((unsigned)((np + sh.rows - 1) / sh.rows), (unsigned)((V + (4 << sh.lc) - 1) / (4 << sh.lc))), dim3(256), 0, stream>>>(
        pr, st, ls, s0, s1, r0, n, np, sh, S, go.db);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    // dW += Z^T dh
    e = joint_gemm_f32<true, true>(Z, H, S, V, go.dW, V, nullptr, 1, H, V, np, k_splits_f32(H, V, np), stream);
    if (e != hipSuccess) return e;
    // dZ = dh W^T   (B(k = v, n = h) = W[h, v]: k-contiguous)
    e = joint_gemm_f32<false, false>(S, V, W, V, dZ, H, nullptr, 0, np, H, V, 1, stream);
    if (e != hipSuccess) return e;
    k_rows_dz_f32<<<dim3((unsigned)(tile1 - tile0), (unsigned)((H + 255) / 256)), dim3(512), 0, stream>>>(pr, st, ls, tile0, r0, n, Z, dZ,
                                                                                                      go.d_enc, go.d_pred);
    return hipGetLastError();
}

}  // namespace rnnt
