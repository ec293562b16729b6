// Set-up work of one call in a single launch: clears the gradient outputs, writes the tile -> sample
// table and the two fragment-major copies of W_out.  Each workgroup reads its job from its index.
#include "device_common.h"
#include "kernels.h"

#include <cstring>
#include <type_traits>

namespace rnnt {

namespace {
struct PrepKernelArgs {
    PrepArgs a;
    unsigned zero_end[5];   // cumulative workgroup counts: clear region r is [zero_end[r-1], zero_end[r])
    unsigned ts_end;        // tile -> sample table: one workgroup per sample
    unsigned wp_end;        // W_out^T fragments for the score GEMM
    unsigned wq_end;        // W_out fragments for the dz GEMM
};
// The host tables of a small batch (about 125 samples), without a launch of their own ahead of this one.  A call: H = 32, V = 16, 240 nodes 33.9 ->
// 31.4 us (each waited for), one utterance of 250 x 50, H = 512, V = 1024 144.8 -> 141.6, four of 200 x 40 171.5 -> 167.6.
struct PrepTable {
    int v[PREP_TABLE_MAX];
};
struct NoTable {};

// TABLE = PrepTable: the last workgroup copies the table to its place, the others read it from the arguments
template <class TABLE>
__global__ __launch_bounds__(256) void k_prepare(PrepKernelArgs k, TABLE tab) {
    constexpr bool WITH_TABLE = std::is_same_v<TABLE, PrepTable>;
    const unsigned b = blockIdx.x;
    const int tid = threadIdx.x;
    if (b < k.zero_end[4]) {
        int r = 0;
        unsigned first = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (b >= k.zero_end[i]) { r = i + 1; first = k.zero_end[i]; }
        float* __restrict__ p = k.a.zero_ptr[r];
        const size_t n = k.a.zero_n[r];
        const size_t stride = (size_t)(k.zero_end[r] - first) * 256;
        for (size_t i = (size_t)(b - first) * 256 + tid; i < n; i += stride) p[i] = 0.0f;
    } else if (b < k.ts_end) {
        const int s = (int)(b - k.zero_end[4]);
        int first, e;
        if constexpr (WITH_TABLE) {
            first = tab.v[k.a.table_tile_off + s];
            e = tab.v[k.a.table_tile_off + s + 1];
        } else {
            first = k.a.tile_off[s];
            e = k.a.tile_off[s + 1];
        }
        for (int i = first + tid; i < e; i += 256) k.a.tile_sample[i] = s;
    } else if (b < k.wp_end) {
        // Wp[((vt*KK + kk)*64 + lane)*8 + j] = W[kk*16 + 8*(lane/32) + j][vt*32 + lane%32]:
        // one A fragment of the score GEMM is a contiguous 1 KiB block
        const int H = k.a.H, V = k.a.V, KK = H >> 4;
        const long long g = (long long)(b - k.ts_end) * 256 + tid;
        if (g >= (long long)(V >> 5) * KK * 64) return;
        const int lane = (int)(g & 63);
        const long long f = g >> 6;
        const int kk = (int)(f % KK), vt = (int)(f / KK);
        const int v = vt * 32 + (lane & 31);
        const int k0 = kk * 16 + 8 * (lane >> 5);
        const bf16_t* __restrict__ W = (const bf16_t*)k.a.W;
        bf16x8 o;
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = W[(size_t)(k0 + j) * V + v];
        *reinterpret_cast<bf16x8*>((bf16_t*)k.a.Wp + g * 8) = o;
    } else if (b < k.wq_end) {
        // Wq[((vk*(H/32) + ht)*64 + lane)*8 + j] = W[ht*32 + lane%32][vk*16 + 8*(lane/32) + j]
        const int H = k.a.H, V = k.a.V, HT = H >> 5;
        const long long g = (long long)(b - k.wp_end) * 256 + tid;
        if (g >= (long long)HT * (V >> 4) * 64) return;
        const int lane = (int)(g & 63);
        const long long f = g >> 6;
        const int vk = (int)(f / HT), ht = (int)(f - (long long)vk * HT);
        const bf16_t* src = (const bf16_t*)k.a.W + (size_t)(ht * 32 + (lane & 31)) * V + vk * 16 + 8 * (lane >> 5);
        *reinterpret_cast<bf16x8*>((bf16_t*)k.a.Wq + g * 8) = *reinterpret_cast<const bf16x8*>(src);
    } else if constexpr (WITH_TABLE) {
        for (int i = tid; i < k.a.table_n; i += 256) k.a.table_dst[i] = tab.v[i];
    }
}
}  // namespace

// dst[i] = bf16(src[i]) (round to nearest even), n a multiple of 8
__global__ __launch_bounds__(256) void k_f32_to_bf16(const float* __restrict__ src, bf16_t* __restrict__ dst, size_t n8) {
    const size_t stride = (size_t)gridDim.x * 256;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n8; i += stride) {
        const f32x4 lo = *reinterpret_cast<const f32x4*>(src + i * 8);
        const f32x4 hi = *reinterpret_cast<const f32x4*>(src + i * 8 + 4);
        bf16x8 o;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            o[j] = (bf16_t)lo[j];
            o[4 + j] = (bf16_t)hi[j];
        }
        *reinterpret_cast<bf16x8*>(dst + i * 8) = o;
    }
}

hipError_t launch_f32_to_bf16(const float* src, void* dst, size_t n, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    if (n % 8 != 0) return hipErrorInvalidValue;
    const size_t n8 = n / 8;
    const size_t blocks = (n8 + 255) / 256;
    k_f32_to_bf16<<<dim3((unsigned)(blocks > 16384 ? 16384 : blocks)), dim3(256), 0, stream>>>(src, (bf16_t*)dst, n8);
    return hipGetLastError();
}

hipError_t launch_prepare(const PrepArgs& a, hipStream_t stream) {
    PrepKernelArgs k{};
    k.a = a;
    unsigned end = 0;
    for (int r = 0; r < 5; ++r) {
        if (a.zero_ptr[r] != nullptr && a.zero_n[r] > 0) {
            size_t blocks = (a.zero_n[r] + 2047) / 2048;
            end += (unsigned)(blocks > 8192 ? 8192 : blocks);
        }
        k.zero_end[r] = end;
    }
    if (a.tile_sample != nullptr) end += (unsigned)a.B;
    k.ts_end = end;
    if (a.Wp != nullptr) end += (unsigned)(((long long)(a.V / 32) * (a.H / 16) * 64 + 255) / 256);
    k.wp_end = end;
    if (a.Wq != nullptr) end += (unsigned)(((long long)(a.H / 32) * (a.V / 16) * 64 + 255) / 256);
    k.wq_end = end;
    if (a.table_n > 0) {
        if (a.table_n > PREP_TABLE_MAX) return hipErrorInvalidValue;
        PrepTable tab;
        std::memcpy(tab.v, a.table, (size_t)a.table_n * 4);
        k_prepare<PrepTable><<<dim3(end + 1), dim3(256), 0, stream>>>(k, tab);
        return hipGetLastError();
    }
    if (end == 0) return hipSuccess;
    k_prepare<NoTable><<<dim3(end), dim3(256), 0, stream>>>(k, NoTable{});
    return hipGetLastError();
}

}  // namespace rnnt
