// Internal launch interface between the C-ABI layer (api.cpp) and the HIP kernels.
// Every function enqueues on `stream` and returns the launch status; none synchronises.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace rnnt {

// Device-resident description of the scheduled samples (one table per call).
struct SampleTable {
    const int* T;              // [B] T_len
    const int* U;              // [B] U_len
    const int* tile_off;       // [B+1] cumulative lattice-tile counts (64 nodes per tile)
    const int* tile_sample;    // [tiles] sample that owns each tile (filled by launch_prepare)
    const long long* row_off;  // [B+1] cumulative lattice-node counts
};

// Per-group lattice state; arrays are indexed by (row_off[s] - row_base) + lattice_index(T_s, U_s + 1, t, u).
// The nodes of a sample lie anti-diagonal after anti-diagonal (t + u = 0, 1, ...), on each by rising u: the lattice sweeps, which
// take one anti-diagonal per step, then read and write memory in one piece.  W = U + 1 columns.
__host__ __device__ inline int diagonal_offset(int T, int W, int k) {
    const int a = T < W ? T : W, b = T < W ? W : T;
    if (k <= a) return k * (k + 1) / 2;
    if (k <= b) return a * (a + 1) / 2 + (k - a) * a;
    const int r = T + W - 1 - k;
    return T * W - r * (r + 1) / 2;
}
__host__ __device__ inline int lattice_index(int T, int W, int t, int u) {
    const int k = t + u;
    return diagonal_offset(T, W, k) + u - (k >= T ? k - T + 1 : 0);
}
// Distance from node (t, u) to (t + 1, u); (t, u + 1) is the one behind that.
__host__ __device__ inline int next_diagonal_step(int T, int W, int k) {
    const int a = T < W ? T : W, r = T + W - 1 - k;
    int len = k + 1 < a ? k + 1 : a;
    len = len < r ? len : r;
    return len - (k + 1 >= T ? 1 : 0);
}
// Stands for ln 0 in the emissions: finite, so that the sums of two impossible ways are no NaN.  A sample whose alignments all take one
// has ln P below a tenth of it, however many they take and whatever else they do (no_alignment).
constexpr float EMISSION_FLOOR = -1e30f;
// A node's larger emission enters the sample's offset as at least this, so that an impossible one neither sets the offset nor is cancelled by
// it: T + U (at most 2^30 + 1023) offsets stay far below EMISSION_FLOOR.
constexpr float OFFSET_FLOOR = -1e9f;
// lnP: without the offset
__host__ __device__ inline bool no_alignment(double lnP) { return lnP < 0.1 * EMISSION_FLOOR; }

struct LatticeState {
    float* lse;    // ln of the softmax denominator (f^W_1)
    float2* em;    // log-probabilities of the blank (x) and of label y_u (y; EMISSION_FLOOR at u = U_s), not below EMISSION_FLOOR
    float* alpha;  // forward variable, offset by shift*(t+u)
    float* beta;   // backward variable, offset by shift*((T-t)+(U-u))
    float* lnP;    // [B] ln P(y|x) + shift*(T+U), per sample
    float* shift;  // [B] per-sample offset added to every emission log-probability
    const float* weight;  // [B] weight of loss[b] in the differentiated sum, or null (all ones)
    float* tile_esum;     // [tiles of the call] sum over a tile's nodes of max(blank, label, OFFSET_FLOOR) (without label where there is
                          // none), written by the bf16 forward kernels for the lattice kernels' offset; or null
    long long row_base;
};

struct Problem {
    int B, T_max, U_max, H, V, blank;
    const void* enc;
    const void* pred;
    const void* W;         // [H,V] as given by the caller
    const float* b_out;
    const int* labels;
};

struct GradOut {
    float* d_enc;
    float* d_pred;
    float* dW;
    float* db;
};

// Set-up of one call in a single launch: clears up to five float regions (null or empty ones are
// skipped), writes tile_sample[tile] = s for every tile of every sample (one lookup instead of a
// search per workgroup; skipped if tile_sample is null) and the fragment-major copies of W_out [H,V]
// (bf16): Wp for the A operand of the score GEMM, Wq for the dz GEMM (each skipped if null).
struct PrepArgs {
    float* zero_ptr[5];
    size_t zero_n[5];
    const int* tile_off;     // [B+1], device
    int* tile_sample;        // [tiles], device
    int B;
    const void* W;
    void* Wp;
    void* Wq;
    int H, V;
    // Host tables of at most PREP_TABLE_MAX ints that reach `table_dst` with this launch, as kernel arguments (table_n = 0: none;
    // tile_off then holds its values already); tile_off lies table_tile_off ints behind table_dst.
    const int* table;        // host
    int table_n, table_tile_off;
    int* table_dst;          // device
};
constexpr int PREP_TABLE_MAX = 800;
hipError_t launch_prepare(const PrepArgs& a, hipStream_t stream);
// dst[i] = bf16(src[i]), n a multiple of 8 (the gradients of a group, accumulated in fp32, on their way out)
hipError_t launch_f32_to_bf16(const float* src, void* dst, size_t n, hipStream_t stream);
// plain copy of n floats (n a multiple of 4): the known-size kernel the HBM counters are calibrated with
hipError_t launch_copy_f32(const float* src, float* dst, size_t n, hipStream_t stream);

// loop of workgroups x 4 waves x iters x 16 MFMAs (32x32x16 bf16) on the 32 x 1 KiB fragments at `frags`;
// writes workgroups x 256 floats to `out` (measurement support)
// every workgroup (256 threads) reads the same `bytes` (a multiple of 32 KiB) `iters` times; out: 4096 bytes per workgroup
hipError_t launch_stream_read(const void* src, size_t bytes, void* out, int workgroups, int iters, hipStream_t stream);
hipError_t launch_mfma_loop(const void* frags, float* out, int workgroups, int iters, hipStream_t stream);
// the same with the fp8 (e4m3) MFMA 32x32x64, unit scales: fragments of 64 lanes x 32 bytes (64 KiB in all)
hipError_t launch_mfma_loop_fp8(const void* frags, float* out, int workgroups, int iters, hipStream_t stream);

// ---- fp32 path (plain FMA kernels, any H, V) ------------------------------------------------
hipError_t launch_fwd_f32(const Problem& pr, const SampleTable& st, const LatticeState& ls,
                          int s0, int s1, long long rows, hipStream_t stream);
hipError_t launch_bwd_f32(const Problem& pr, const SampleTable& st, const LatticeState& ls,
                          const GradOut& go, int s0, int s1, long long rows, hipStream_t stream);

// fp32 GEMM form of the same two steps for H, V multiples of 4, over lattice nodes [r0, r0 + n) of the
// group (node index relative to the group's first).  S [rows, V], Z and dZ [rows, H] are chunk buffers of
// n rounded up to a multiple of 128 rows.  have_scores: S and Z already hold what launch_fwd_f32_gemm left for these nodes.
// Lattice tiles [tile0, tile1) hold all of the nodes.
hipError_t launch_fwd_f32_gemm(const Problem& pr, const SampleTable& st, const LatticeState& ls, int s0, int s1,
                               long long r0, long long n, float* S, float* Z, hipStream_t stream);
hipError_t launch_bwd_f32_gemm(const Problem& pr, const SampleTable& st, const LatticeState& ls, const GradOut& go,
                               int s0, int s1, int tile0, int tile1, long long r0, long long n, bool have_scores, float* S, float* Z,
                               float* dZ, hipStream_t stream);

// ---- lattice (alpha, beta, loss) ------------------------------------------------------------
// wide != 0: the sweep accumulates in fp64 (alpha, beta, ln P still stored as fp32); used by the fp32 path
hipError_t launch_lattice(const SampleTable& st, const LatticeState& ls, int s0, int s1, int u_max, int wide,
                          float* loss, hipStream_t stream);

// After the lattice pass of a group: flags[tile] = 1 for tiles [tile0, tile1) with a node whose posterior
// ln gamma = alpha + beta - ln P is at least log_floor, their ids in ascending order in active[tile0 ...] and their
// number in *n_active.
hipError_t launch_select_tiles(const SampleTable& st, const LatticeState& ls, int s0, int s1, int tile0, int tile1,
                               float log_floor, int* flags, int* active, int* n_active, hipStream_t stream);
// The tiles a backward launch works on: null active = tiles [tile0, tile1) one by one; else entry cbase + i of the
// group's list active[group_tile0 ...], for i below *n_active - cbase (workgroups beyond that return at once).
// Where a listed tile's 64 rows lie in the chunk buffers: in slot i (slot_tile0 < 0: the backward pass fills the
// buffers itself, densely), or in slot tile - slot_tile0 (kept scores: the forward pass has filled the buffers
// tile by tile before the list existed).
struct ActiveTiles {
    const int* active;
    const int* n_active;
    int group_tile0;
    int cbase;
    int slot_tile0;
};
constexpr ActiveTiles EVERY_TILE{nullptr, nullptr, 0, 0, -1};

// ---- bf16 MFMA path -------------------------------------------------------------------------
// Wpack: W_out^T in fragments [V/32][H/16], Wq: W_out in fragments [V/16][H/32] (launch_prepare).
// scores on MFMA -> online log-softmax -> lse, emissions   (tiles [tile0,tile1)).  part: scratch for partial statistics where
// a small launch splits the vocabulary over workgroups; these count their arrivals in the emission sums of the tiles, which are
// zero before the launch (launch_prepare)
hipError_t launch_fwd_bf16(const Problem& pr, const void* Wpack, const SampleTable& st, const LatticeState& ls, int tile0,
                           int tile1, void* part, size_t part_bytes, hipStream_t stream);
// scores recomputed -> dh and z (bf16) into the chunk buffers
hipError_t launch_bwd_scores_bf16(const Problem& pr, const void* Wpack, const SampleTable& st, const LatticeState& ls, int tile0,
                                  int tile1, void* dH, void* Z, const ActiveTiles& at, hipStream_t stream);
// The forward launch that also keeps the joint rows (Z) and the scores (kept, in the dH buffer: fp16 differences to the running
// maxima kept_max [tiles][V/64][64]) of tiles [tile0,tile1), and the launch that turns the kept scores into dh (bf16, in
// place) once alpha and beta are known.  part: as for launch_fwd_bf16, of part_bytes (0: never split).
hipError_t launch_fwd_keep_bf16(const Problem& pr, const void* Wpack, const SampleTable& st, const LatticeState& ls, int tile0,
                                int tile1, void* kept, void* Z, float* kept_max, void* part, size_t part_bytes, hipStream_t stream);
hipError_t launch_kept_to_dh_bf16(const Problem& pr, const SampleTable& st, const LatticeState& ls, int tile0, int tile1,
                                  void* kept, const float* kept_max, const ActiveTiles& at, hipStream_t stream);
// dz = dH W^T, times the tanh derivative, reduced over the tile's u resp. t, added to d_enc, d_pred
hipError_t launch_gemm_dz_bf16(const Problem& pr, const void* Wq, const SampleTable& st, int tile0, int tile1, const void* dH,
                               float* d_enc, float* d_pred, const ActiveTiles& at, hipStream_t stream);
// launch_gemm_dz_bf16 and launch_gemm_dw_bf16 in one launch, for plans whose one_grid is set
hipError_t launch_gemm_dz_dw_bf16(const Problem& pr, const void* Wq, const SampleTable& st, int tile0, int tile1, const void* Z,
                                  const void* dH, float* d_enc, float* d_pred, int splits, int first, float* slots, float* db,
                                  const ActiveTiles& at, hipStream_t stream);
// Shape of a sample's lattice tiles (64 rows each): 8 frames x 8 label positions, or 16 x 4 where that covers the
// sample's T x (U + 1) lattice with at least 3 % fewer tiles (the padding rows of partly filled tiles cost as
// much as real ones; a 16 x 4 tile adds to 20 rows of d_enc / d_pred instead of 16, which costs about 2 %).
// Returns the label positions per tile, 8 or 4; a tile then has 64 / that many frames, and row r of a tile is
// frame r / uw, label position r % uw.
__host__ __device__ inline int tile_label_width(int T, int U) {
    const long long a = (long long)((T + 7) / 8) * ((U + 8) / 8), b = (long long)((T + 15) / 16) * ((U + 4) / 4);
    return b * 33 < a * 32 ? 4 : 8;
}
__host__ __device__ inline long long sample_tiles(int T, int U) {
    const int uw = tile_label_width(T, U), th = 64 / uw;
    return (long long)((T + th - 1) / th) * ((U + uw) / uw);
}
// Elements a row takes in the two bf16 chunk buffers Z [rows, H] and dH [rows, V] (a block of 32 rows is 4 KiB longer than its
// data; layout: device_common.h)
__host__ __device__ inline int chunk_pitch(int n) { return n + 64; }

// Split-K GEMM Z^T dH over one chunk's rows: every (split, tile) workgroup adds its 256x256 partial
// product to its own slot (`first` != 0: overwrites it), db += column sums of dH.  `splits` and the
// slot buffer size follow dw_split_choice / dw_slot_bytes (plan.h).
// With at.active set the chunk holds only min(rows, 64 * (*at.n_active - at.cbase)) rows (read on the device).
hipError_t launch_gemm_dw_bf16(int H, int V, long long rows, int splits, int first, const void* Z,
                               const void* dH, float* slots, float* db, const ActiveTiles& at, hipStream_t stream);
// dW = (accumulate ? dW : 0) + sum of the slots over the splits
hipError_t launch_dw_reduce(int H, int V, int splits, const float* slots, float* dW, int accumulate,
                            hipStream_t stream);

// ---- input projections of the joint network (Eq. 4) and their backward -----------------------
// Row r of a [B*period, D] array is real data iff there is no mask (len == nullptr) or
// (r % period) < len[r / period] + extra; other rows are read as zero.
struct RowMask {
    const int* len;   // device, [B]
    int period;       // T_max, or U_max + 1
    int extra;        // 0 for frames (t < T_len), 1 for label positions (u <= U_len)
};
// One of the two maps, out = h W (+ bias), with what its backward pass reads and writes.  h [rows,D] and W [D,H] in the input dtype, padded rows of h
// may hold anything; out [rows,H] in the input dtype; d_out fp32 [rows,H], zero in padded rows; d_in fp32 [rows,D].
struct ProjSide {
    const void* h;
    long long rows;
    int D;
    RowMask mask;            // of the rows (length tables on the device: read by the backward launch only)
    const void* W;
    const float* bias;       // or null
    void* out;
    const float* d_out;
    float* d_in;
    float* dW;               // fp32 [D,H], added to
    float* db;               // += column sums of d_out, or null
};
// out of both maps; with `clear` dW of both and db of the first are cleared besides
hipError_t launch_proj_forward(int bf16, const ProjSide (&s)[2], int H, bool clear, hipStream_t stream);
// d_in = d_out W^T, dW += h^T d_out over the real rows, db += column sums of d_out
hipError_t launch_proj_backward(int bf16, const ProjSide (&s)[2], int H, hipStream_t stream);
// C[m,n] (+)= sum_k A(m,k) B(k,n) (+ bias[n]) in fp32 precision (operands as three bf16 parts), any M, N, K.  An operand
// is k-slow (element (i,k) at p[k*ld + i]) or k-contiguous (at p[i*ld + k]); combinations: A contiguous with
// either B, or both slow.  Rows of an operand's source array outside its mask read as zero.  atomic: C is
// added to with float atomics (required for splits > 1).  gemm_f32_edge_fits: the 16-byte alignment the
// kernel's loads need (extents along the contiguous index: K resp. M for A, K resp. N for B).
bool gemm_f32_edge_fits(const void* A, long long lda, const void* B, long long ldb, long long a_contig_extent,
                        long long b_contig_extent);
// k_splits_f32: the splits of a sum over K rows.
int k_splits_f32(long long M, long long N, long long K);
hipError_t launch_gemm_f32_masked(int a_kslow, int b_kslow, const float* A, long long lda, const RowMask& ma,
                                  const float* B, long long ldb, const RowMask& mb, float* C, long long ldc,
                                  const float* bias, int atomic, long long M, long long N, long long K, int splits,
                                  hipStream_t stream);
// out[c] += sum_r x[r,c]   (x fp32 [rows,cols])
hipError_t launch_col_sum(const float* x, long long rows, int cols, float* out, hipStream_t stream);

}  // namespace rnnt
