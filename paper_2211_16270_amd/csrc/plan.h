// Host-side scheduler: packs the samples of a call into groups and backward chunks and lays
// out the workspace.  Pure C++ (no HIP), so it is unit-testable without a GPU.
//
// The paper recovers parallelism lost by sample-wise processing by running several loop
// iterations of Algorithm 1 at once, as many as a memory limit allows (Section 4.1.2, Eq. 11).
// Here the same idea is a packing problem: samples are cut into lattice tiles of 64 nodes (8 frames x 8 label positions, or 16 x 4), the tiles of
// all samples of a *group* are processed by one launch, and a group holds as many samples as
// its per-node state (5 floats per lattice node) fits the workspace.  The backward pass walks a
// group in *chunks* of tiles whose bf16 score-gradient buffers fit the rest of the workspace.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <vector>

#include "../../include/rnnt_joint_loss.h"

// (this header is also read by a host compiler)
#ifdef __HIPCC__
#define RNNT_HOST_DEVICE __host__ __device__
#else
#define RNNT_HOST_DEVICE
#endif

namespace rnnt {

constexpr int TILE_ROWS = 64;    // lattice tile: 8 frames x 8 label positions or 16 x 4 (kernels.h: tile_label_width)
constexpr int GEMM_TILE = 128;   // row granularity of the backward GEMMs (two lattice tiles)
constexpr size_t WS_ALIGN = 256;

struct Group {
    int s0, s1;          // samples [s0, s1)
    int tile0, tile1;    // global tile range
    long long rows;      // lattice nodes of the group
    int u_max;           // largest U_len in the group
};

struct Chunk {
    int group;
    int tile0, tile1;    // global tile range, inside the group's range
    // fp32 GEMM form: lattice nodes [row0, row0 + rows) of the group instead, in tiles [tile0, tile1).  [s0, s1): the samples that are swept together, when all
    // chunks with this s0 have their scores: whole samples that one chunk holds, one that takes several, or all of the group (plan.cpp: F32Chunks)
    long long row0 = 0, rows = 0;
    int s0 = 0, s1 = 0;
};

struct Plan {
    int B = 0;
    bool bf16 = false;
    bool f32_gemm = false;              // fp32 only: H, V multiples of 4 from 64 on, the steps run as fp32 GEMMs over chunks
    bool keep = false;                  // bf16 only: forward keeps the scores, one backward chunk per group
    bool stage = false;                 // bf16 only: d_enc, d_pred leave as bf16; fp32 sums of one group in the workspace
    long long stage_samples = 0;        // samples a group may hold then
    std::vector<int> tile_off;          // [B+1] cumulative tile counts
    std::vector<long long> row_off;     // [B+1] cumulative lattice nodes
    std::vector<Group> groups;
    std::vector<Chunk> chunks;
    std::vector<Chunk> group_chunks;    // fp32 GEMM form, lat_buffers = 2: full chunks, for calls whose sweeps run on a stream of their own
    long long rows_total = 0, tiles_total = 0;
    long long group_rows_cap = 0;       // lattice nodes a group may hold
    int lat_buffers = 1;                // 2: the lattice arrays hold two groups (group g uses half g % 2)
    long long chunk_rows = 0;           // rows (multiple of GEMM_TILE) of the chunk buffers (fp32 GEMM form: lattice nodes)
    // workspace layout (byte offsets)
    size_t off_T = 0, off_U = 0, off_weight = 0, off_tile_off = 0, off_row_off = 0, off_lnP = 0, off_shift = 0, off_tile_sample = 0;
    size_t off_tile_esum = 0;          // bf16: per-tile emission sums (float per tile)
    int skip_log2 = 0;                 // > 0: tiles whose posteriors all lie below 2^-skip_log2 stay out of the backward pass
    size_t off_n_active = 0;           // skip_log2 > 0: per group the number of tiles that stay (their list lies in the
                                       // tile_esum array, over the entries of the same tiles)
    size_t off_wpack = 0, off_wq = 0;
    size_t off_lse = 0, off_em = 0, off_alpha = 0, off_beta = 0;
    size_t off_dh = 0, off_z = 0, off_kept_max = 0;
    size_t off_dz32 = 0;                // fp32 GEMM form: dZ [chunk_rows, H]; off_dh, off_z hold S and Z as fp32
    size_t off_stage_enc = 0, off_stage_pred = 0;   // fp32 [stage_samples, T_max, H], [stage_samples, U_max+1, H]
    size_t off_dwslots = 0;             // bf16: per-workgroup partial sums of the dW GEMM
    bool one_grid = false;              // bf16: the dz and dW GEMMs run as one grid (one_grid_shape)
    int dw_splits = 0;                  // bf16: K splits of the dW GEMM (dw_split_choice, dw_split_one_grid)
    size_t lattice_bytes = 0, chunk_bytes = 0, total_bytes = 0;
    size_t min_bytes = 0;               // smallest workable workspace
};

// A score gradient dh = gamma * softmax - posteriors is at most the node's posterior gamma in magnitude, and a
// magnitude below 2^-134 (half the smallest bfloat16 denormal) rounds to zero as bf16: with gamma < 2^-135 at every
// node of a tile, every operand the tile would feed into the backward GEMMs is exactly zero.
constexpr int ZERO_IN_BF16_LOG2 = 135;

// Shapes the fp32 GEMM form covers: rows of 16-byte pieces, and wide enough for 128 x 128 tiles to pay.
inline bool f32_gemm_shape(int H, int V) { return H % 4 == 0 && V % 4 == 0 && H >= 64 && V >= 64; }

// dW GEMM geometry: 256x256 output tiles (the last hidden one of 128 where H is not a multiple of 256).  Every (split, tile) workgroup
// owns a 256 KiB slot of partial sums in the workspace.  The slots have room for dw_split_count splits less, for H > 640, a packed
// copy of W_out: the room of the copy for the dz GEMM, which so takes nothing from what a workspace of a given size can hold.  A call
// uses at most dw_splits_max of them.
constexpr int DW_TILE = 256;
inline int dw_tiles(int H, int V) { return ((H + DW_TILE - 1) / DW_TILE) * (V / DW_TILE); }
inline int dw_split_count(int H, int V) {
    const int t = dw_tiles(H, V);
    return ((256 + t - 1) / t + 7) / 8 * 8;
}
inline size_t dw_slot_bytes(int H, int V) {
    return (size_t)dw_tiles(H, V) * dw_split_count(H, V) * DW_TILE * DW_TILE * 4 - (H > 640 ? (size_t)H * V * 2 : 0);
}
inline int dw_splits_max(int H, int V) {
    return (int)(dw_slot_bytes(H, V) / ((size_t)dw_tiles(H, V) * DW_TILE * DW_TILE * 4));
}

// How many workgroups of the dz GEMM share the vocabulary of one set of rows (1, 2 or 4): the fewest rounds of the chip, a workgroup costing
// its share of the blocks and `fixed` blocks' time for its start and end.
inline long long split_cost(int workgroups, int vs, int slots, int nvb, int fixed) {
    return ((long long)workgroups * vs + slots - 1) / slots * (fixed + nvb / vs);
}
inline int vocabulary_split(int workgroups, int slots, int nvb, int fixed = 8) {
    int best = 1;
    long long best_cost = 0;
    for (int vs = 1; vs <= 4; vs *= 2) {
        const long long cost = split_cost(workgroups, vs, slots, nvb, fixed);
        if (vs == 1 || cost * 10 < best_cost * 9) {
            best = vs;
            best_cost = cost;
        }
    }
    return best;
}

// Score kernels: how many workgroups share the vocabulary of one set of rows.  Statistics (forward pass) are formed per segment of the vocabulary and
// folded in order, so that a result does not depend on the number of workgroups; a part is a run of whole segments, of up to one more than another's.
// Eight segments from V = 2048 on, where a fold per 256 entries and more is nothing; else four.  The backward pass forms no statistics: its parts are
// runs of whole pairs of blocks.
// (A segment is a whole number of pairs of blocks: kept scores leave in pairs, as differences to one maximum.)
RNNT_HOST_DEVICE inline int score_segments(int V) { return V >= 2048 && V % 512 == 0 ? 8 : 4; }
// first block (of 32 entries) of part y of `parts`; statistics: parts of whole segments
RNNT_HOST_DEVICE inline int score_part_begin(int y, int parts, int V, bool statistics) {
    const int nvb = V / 32, units = statistics ? score_segments(V) : nvb / 2;
    return units * y / parts * (nvb / units);
}
// The fewest rounds of the chip, a workgroup costing the blocks of the longest part and `fixed` blocks' time for its start and end; every part has a
// multiple of `multiple` blocks.  Up to eight parts instead of 1, 2 or 4, a call: H = 640, V = 8192 one sample of 60 x 10 205 -> 152 us, of 250 x 50
// 506 -> 454; H = 1024, V = 4096 one of 60 x 10 174 -> 139, 16 of up to 50 x 10 380 -> 346, eight of 100 x 20 623 -> 581; losses alone 16 of 50 x 10,
// H = 640, V = 4096 90.5 -> 76.1 (H = 512, where the number of parts stays: 68.8 -> 69.5, eight segments to fold instead of four).
struct ScoreSplit {
    int parts;
    long long cost;
};
inline ScoreSplit score_split(int workgroups, int slots, int V, bool statistics, int multiple = 2, int fixed = 8) {
    ScoreSplit best{1, 0};
    for (int p = 1; p <= 8; ++p) {
        int longest = 0;
        bool whole = true;
        for (int y = 0; y < p; ++y) {
            const int n = score_part_begin(y + 1, p, V, statistics) - score_part_begin(y, p, V, statistics);
            longest = std::max(longest, n);
            whole = whole && n > 0 && n % multiple == 0;
        }
        if (!whole) continue;
        const long long cost = ((long long)workgroups * p + slots - 1) / slots * (fixed + longest);
        if (p == 1 || cost * 10 < best.cost * 9) best = ScoreSplit{p, cost};
    }
    return best;
}

// K splits for chunks of `rows` rows: the least of (longest chain of workgroups on one of the 32 compute units of an XCD) x (stages of 32
// rows, and about 8 for start and end) + the slots' traffic, in units of a stage of a whole tile (about 0.5 us; a slot written
// once and read once costs a fifth of that when the whole chip moves them).  Half tiles cost half and run two to a gap.
// Against a multiple of 8 for every shape: H = 1024, V = 4096, 8800 rows 402 -> 394 us a call (4 splits, not 8), H = 640, V = 4096 60.1 -> 58.0 ms
// (6 splits with the half tiles, not 8 with whole ones; both relative to the same start).
inline int dw_split_choice(int H, int V, long long rows) {
    const int fm = H / DW_TILE, hm = (H + DW_TILE - 1) / DW_TILE - fm, nt = V / DW_TILE;
    const double stages = (double)rows / 32.0;
    int best = 1;
    double best_cost = 0.0;
    for (int s = 1; s <= dw_splits_max(H, V); ++s) {
        const int f8 = (s * fm * nt + 7) / 8, h8 = (s * hm * nt + 7) / 8;
        const int gaps = f8 % 32 ? 2 * (32 - f8 % 32) : 0;
        const int rest = h8 > gaps ? (h8 - gaps + 31) / 32 : 0;
        const double rounds = (f8 + 31) / 32 + 0.5 * rest;
        const double cost = rounds * (stages / s + 8.0) + 0.2 * s * nt * (fm + 0.5 * hm);
        if (s == 1 || cost < best_cost) {
            best = s;
            best_cost = cost;
        }
    }
    return best;
}

// dz GEMM of a chunk of lattice tiles: 4 of them x `edge` hidden columns (256; 128 for the rest, or for all) and one of vs parts of the
// vocabulary per workgroup.  Alone on the chip: whole tiles (the half one counts half), or, in a launch of one round, half tiles alone where they
// fill the chip better: twice the workgroups of about half the cost each, so that a small launch need not split the vocabulary, which runs the
// epilogue and its atomics once per part (one utterance of 250 x 50, H = 512, V = 1024: a call 175.7 -> 165 us).  Past one
// round the half tiles' poorer ratio of LDS reads to MFMAs shows (288 of them, H = 1024, V = 4096, against 144 whole ones: 394 -> 407 us a
// call).  About 16 stages' time for start and epilogue.
struct DzForm {
    int edge, vs;
};
// Waves of a dz workgroup of its own launch.  Four and two workgroups per compute unit: one's start and epilogue (a quarter of the time at V = 1024) stand beside
// the other's MFMAs, for half as much again of W_out's way from the L2 to LDS; a long vocabulary has little of the one and much of the other.  A call with
// eight -> four, 64 samples of 500 x 100: H = 256 V = 1024 5.70 -> 5.53 ms, H = 384 V = 768 6.46 -> 6.23, H = 512 V = 512 5.49 -> 5.26, V = 1024 9.45 -> 9.26,
// V = 2048 (with the line further up) 16.42 -> 16.42, H = 1024 V = 1024 18.4 -> 18.15; 1024 of up to 1000 x 200, H = 512, V = 1024 314.6 -> 310.2; H = 128
// V = 1024 2130 -> 2145 us, H = 1024 V = 4096 11.1 -> 11.6.
inline int dz_waves(int H, int V) { return H >= 256 && V <= 1024 ? 4 : 8; }
inline DzForm dz_alone(int H, int V, long long tiles) {
    const int m_tiles = (int)((tiles + 3) / 4), stages = V / 32;
    const int whole = (m_tiles * H + 255) / 256, halves = m_tiles * (H / 128);
    const int vs_w = vocabulary_split(whole, 256, stages, 16), vs_h = vocabulary_split(halves, 256, stages, 16);
    const long long cost_w = 2 * split_cost(whole, vs_w, 256, stages, 16), cost_h = split_cost(halves, vs_h, 256, stages, 16);
    return halves <= 256 && cost_h * 10 < cost_w * 9 ? DzForm{128, vs_h} : DzForm{256, vs_w};
}

// The two GEMMs of a call whose backward pass is one chunk run as one grid, dW's workgroups first: there neither fills the chip to the end,
// and what one leaves idle the other takes.  Two launches -> one grid, V = 1024, a call: H = 512 one utterance of 20 x 4 80 -> 71 us, of 250 x 50
// 172 -> 157, of 500 x 100 445 -> 411, 32 samples 1042 -> 1010; H = 256 one of 250 x 50 134 -> 120.
// Their forms are those whose last workgroup ends first when each is taken by the first of the 256 compute units that is free (a
// workgroup fills one).  Costs in stages of a whole dz tile (32 entries, about 0.45 us): dz 16 for start and epilogue, a half tile 0.6 of a
// whole one (the 144 against 288 above); dW 8 for start and end and 1.15 per 32 rows; its slots, written once and read once by the whole
// chip, a fifth of a stage each.
// Not in larger calls (one of H = 512, V = 8192 lost 1 %, one of 64 samples of 500 x 100 with kept scores, H = 640, 1.5 %; others gained 0 to
// 4 %): there the ends matter less than that all workgroups of a chunk read the same rows at a time.
constexpr long long ONE_GRID_MAX = 4096;      // workgroups
inline long long dz_workgroups(int H, int V, long long tiles, DzForm f) { return (tiles + 3) / 4 * ((H + f.edge - 1) / f.edge) * f.vs; }
// (whole hidden tiles and a half one: their mean, with dz's half at 0.9.  With 0.6 the rule takes whole ones at H = 384 where half tiles alone are
// better, one sample of 400 x 80 313 against 304 us; with 1.0 the reverse at H = 640, 32 samples 1421 against 1386.)
inline double tile_mean(int H, double half) { return (H / 256 + (H % 256 ? half : 0.0)) / ((H + 255) / 256); }
inline double dz_cost(int H, int V, DzForm f) { return (16.0 + V / 32 / f.vs) * (f.edge == 128 || H == 128 ? 0.6 : tile_mean(H, 0.9)); }
inline double dw_cost(int H, long long tiles, int splits) { return (1.15 * tiles * (TILE_ROWS / 32) / splits + 8.0) * tile_mean(H, 0.6); }
inline bool one_grid_shape(int H, int V, long long tiles) {
    return dz_workgroups(H, V, tiles, DzForm{256, 1}) + (long long)dw_tiles(H, V) * dw_split_choice(H, V, tiles * TILE_ROWS) <= ONE_GRID_MAX;
}
// When the last of n workgroups of cost c ends that follow nw of cost cw.
inline double one_grid_end(long long nw, double cw, long long n, double c) {
    const long long full = nw / 256, r = nw % 256;
    const double ta = full * cw, tb = r ? ta + cw : ta;      // 256 - r units are free from ta on, r from tb on
    for (double k = std::max(1.0, std::floor((n * c + r * cw) / (256.0 * c)) - 1.0);; k += 1.0) {
        // in order of time: a unit of the first kind ends its k-th workgroup, then one of the second kind its (in_b + 1)-th
        const double at_a = ta + k * c, in_b = std::floor(std::max(0.0, at_a - tb) / c), at_b = tb + (in_b + 1.0) * c;
        if ((256 - r) * (long long)k + r * (long long)in_b >= n) return std::max(at_a, tb);
        if (at_b < at_a + c && (256 - r) * (long long)k + r * (long long)(in_b + 1.0) >= n) return at_b;
    }
}
inline double dz_dw_end(int H, int V, long long tiles, int splits, DzForm f) {
    return one_grid_end((long long)dw_tiles(H, V) * splits, dw_cost(H, tiles, splits), dz_workgroups(H, V, tiles, f), dz_cost(H, V, f));
}
// (a split of the vocabulary repeats epilogue and atomics: only where it saves a tenth)
inline DzForm dz_one_grid(int H, int V, long long tiles, int splits) {
    DzForm best{256, 1};
    double best_end = dz_dw_end(H, V, tiles, splits, best);
    for (int vs = 1; vs <= 4; vs *= 2)
        for (int edge = 256; edge >= 128; edge -= 128) {
            const DzForm f{edge, vs};
            if (vs > 1 && dz_workgroups(H, V, tiles, f) > 1024) continue;
            const double end = dz_dw_end(H, V, tiles, splits, f);
            if (end < (vs > best.vs ? 0.9 : 1.0) * best_end) {
                best = f;
                best_end = end;
            }
        }
    return best;
}
inline int dw_split_one_grid(int H, int V, long long tiles) {
    int best = 1;
    double best_cost = 0.0;
    for (int s = 1, most = dw_splits_max(H, V); s <= most; s += s < 4 ? 1 : s / 4) {
        const double slots = 0.2 * s * (V / DW_TILE) * (H / DW_TILE + (H % DW_TILE ? 0.5 : 0.0));
        const double cost = dz_dw_end(H, V, tiles, s, dz_one_grid(H, V, tiles, s)) + slots;
        if (s == 1 || cost < best_cost) {
            best = s;
            best_cost = cost;
        }
    }
    return best;
}

// Argument checks shared by every entry point (no pointers to data arrays here).
rnnt_status check_desc(const rnnt_desc* d);
rnnt_status check_lengths(const rnnt_desc* d, const int32_t* T_len, const int32_t* U_len);

// Builds the plan for a workspace of `workspace_bytes` (0 = default trade-off).  If the size
// is below the smallest workable one, plan.total_bytes = plan.min_bytes > workspace_bytes and
// the group/chunk lists are those of the smallest plan.
// two_lattice_buffers: room for the lattice state of two groups at a time (for calls that run a group's lattice
// sweep on a second stream while the previous group's backward pass is still reading its own state).  grads: false for calls that form
// losses alone (the workspace is the same).
void build_plan(const rnnt_desc& d, const int32_t* T_len, const int32_t* U_len,
                size_t workspace_bytes, Plan& plan, bool two_lattice_buffers = false, bool grads = true);

}  // namespace rnnt
