// Host scheduler and workspace layout (see plan.h).  No HIP in this file.
#include "plan.h"

#include "kernels.h"

#include <algorithm>
#include <cmath>

namespace rnnt {

static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

rnnt_status check_desc(const rnnt_desc* d) {
    if (!d) return RNNT_ERR_NULL;
    if (d->B < 1 || d->T_max < 1 || d->U_max < 0 || d->H < 1 || d->V < 2) return RNNT_ERR_SHAPE;
    if (d->blank < 0 || d->blank >= d->V) return RNNT_ERR_SHAPE;
    if (d->accumulate_params != 0 && d->accumulate_params != 1) return RNNT_ERR_SHAPE;
    if (d->keep_scores != 0 && d->keep_scores != 1) return RNNT_ERR_SHAPE;
    if (d->keep_scores && d->dtype != RNNT_BF16) return RNNT_ERR_UNSUPPORTED;
    if (d->input_grads_bf16 != 0 && d->input_grads_bf16 != 1) return RNNT_ERR_SHAPE;
    if (d->input_grads_bf16 && d->dtype != RNNT_BF16) return RNNT_ERR_UNSUPPORTED;
    if (d->dtype != RNNT_F32 && d->dtype != RNNT_BF16) return RNNT_ERR_UNSUPPORTED;
    if (d->skip_below_log2 < -1 || d->skip_below_log2 > 126) return RNNT_ERR_SHAPE;
    if (d->skip_below_log2 > 0 && d->dtype != RNNT_BF16)
        return RNNT_ERR_UNSUPPORTED;                            // the bf16 backward kernels take a tile list
    if (d->U_max > 1023) return RNNT_ERR_UNSUPPORTED;           // one lattice thread per label position
    if ((long long)d->T_max * (d->U_max + 1) > (1LL << 30)) return RNNT_ERR_UNSUPPORTED;
    if (d->dtype == RNNT_BF16) {
        if (d->H % 128 != 0 || d->H > 1024) return RNNT_ERR_UNSUPPORTED;
        if (d->V % 256 != 0) return RNNT_ERR_UNSUPPORTED;
    } else {
        if (d->H > 4096 || d->V > 16384) return RNNT_ERR_UNSUPPORTED;
    }
    return RNNT_OK;
}

rnnt_status check_lengths(const rnnt_desc* d, const int32_t* T_len, const int32_t* U_len) {
    if (!T_len || !U_len) return RNNT_ERR_NULL;
    for (int b = 0; b < d->B; ++b) {
        if (T_len[b] < 1 || T_len[b] > d->T_max) return RNNT_ERR_LENGTH;
        if (U_len[b] < 0 || U_len[b] > d->U_max) return RNNT_ERR_LENGTH;
    }
    return RNNT_OK;
}

namespace {

// Fills every offset for the given capacities and returns the total size.
size_t lay_out(const rnnt_desc& d, Plan& p, long long lat_cap, long long chunk_rows, long long stage_samples) {
    const size_t B = (size_t)d.B;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes, WS_ALIGN); return at; };
    p.off_T = take(B * 4);
    p.off_U = take(B * 4);
    p.off_weight = take(B * 4);
    p.off_tile_off = take((B + 1) * 4);
    p.off_row_off = take((B + 1) * 8);
    p.off_lnP = take(B * 4);
    p.off_shift = take(B * 4);
    p.off_tile_sample = take((size_t)p.tiles_total * 4);
    p.off_tile_esum = take(p.bf16 ? (size_t)p.tiles_total * 4 : 0);
    // the list of tiles that take part in the backward pass is written over the emission sums of the same tiles
    // (the lattice pass has consumed them by then): only the per-group counts need room of their own
    p.off_n_active = take(p.skip_log2 ? B * 4 : 0);
    p.off_wpack = take(p.bf16 ? (size_t)d.H * d.V * 2 : 0);
    p.off_wq = take(p.bf16 ? (size_t)d.H * d.V * 2 : 0);
    p.off_dwslots = take(p.bf16 ? dw_slot_bytes(d.H, d.V) : 0);
    size_t lat0 = o;
    // lat_buffers = 2: consecutive groups alternate between two halves of each array, so that one group's
    // lattice sweep can run while its neighbour's state is still in use
    const size_t lat_elems = (size_t)lat_cap * (size_t)p.lat_buffers;
    p.off_lse = take(lat_elems * 4);
    p.off_em = take(align_up(lat_elems * 4, WS_ALIGN) * 2);
    p.off_alpha = take(lat_elems * 4);
    p.off_beta = take(lat_elems * 4);
    p.lattice_bytes = o - lat0;
    size_t ch0 = o;
    if (p.bf16) {
        p.off_dh = take((size_t)chunk_rows * chunk_pitch(d.V) * 2);
        p.off_z = take((size_t)chunk_rows * chunk_pitch(d.H) * 2);
        p.off_kept_max = take(p.keep ? (size_t)chunk_rows * (d.V / 64) * 4 : 0);
    } else if (p.f32_gemm) {
        p.off_dh = take((size_t)chunk_rows * d.V * 4);
        p.off_z = take((size_t)chunk_rows * d.H * 4);
        p.off_dz32 = take((size_t)chunk_rows * d.H * 4);
        p.off_kept_max = o;
    } else {
        p.off_dh = p.off_z = p.off_kept_max = o;
    }
    p.chunk_bytes = o - ch0;
    p.off_stage_enc = take((size_t)stage_samples * d.T_max * d.H * 4);
    p.off_stage_pred = take((size_t)stage_samples * (d.U_max + 1) * d.H * 4);
    p.stage_samples = stage_samples;
    p.group_rows_cap = lat_cap;
    p.chunk_rows = (p.bf16 || p.f32_gemm) ? chunk_rows : 0;
    p.total_bytes = o;
    return o;
}

// fp32 GEMM form: the chunks of a group, ranges of lattice nodes that fit the chunk buffers, in one of two orders.  Chunks of whole samples are swept as they
// come, and their scores computed once; but a sweep takes as long for a few samples as for all of them, and the chunks are more.  Full chunks need one
// sweep a group, and all their scores but the last chunk's twice.  64 samples of 500 x 100, one order -> the other: H = V = 64 in the default workspace 7.3 ms
// -> 9.1, in a sixteenth of it 24.6 -> 14.4; H = V = 256 18.1 -> 21.8, 55.8 -> 41.9; 16 of them, H = 1024, V = 4096, 99.6 -> 127.1, and in a quarter
// 134.3 -> 133.4.
struct F32Chunks {
    const rnnt_desc& d;
    const int32_t *T_len, *U_len;
    const Plan& p;
    int gi;
    long long chunk_rows;

    // nodes [row0, row0 + rows) of the group, out of samples [s0, s1): the blocks of frames they touch
    Chunk range(int s0, int s1, long long row0, long long rows) const {
        const long long base = p.row_off[p.groups[gi].s0];
        auto block = [&](long long row, int after) {
            const int s = (int)(std::upper_bound(p.row_off.begin(), p.row_off.end(), base + row) - p.row_off.begin()) - 1;
            const int W = U_len[s] + 1, uw = tile_label_width(T_len[s], U_len[s]), th = TILE_ROWS / uw, across = (W + uw - 1) / uw;
            return p.tile_off[s] + (int)((base + row - p.row_off[s]) / W / th + after) * across;
        };
        Chunk c{gi, block(row0, 0), block(row0 + rows - 1, 1)};
        c.row0 = row0;
        c.rows = rows;
        c.s0 = s0;
        c.s1 = s1;
        return c;
    }
    // samples [s0, s1) in chunks of `per` nodes
    void cut(int s0, int s1, long long per, std::vector<Chunk>& out) const {
        const long long base = p.row_off[p.groups[gi].s0], end = p.row_off[s1] - base;
        for (long long r0 = p.row_off[s0] - base; r0 < end; r0 += per) out.push_back(range(s0, s1, r0, std::min(per, end - r0)));
    }
    // As many whole samples as a chunk holds, or one that takes several chunks (of equal size).
    std::vector<Chunk> of_samples() const {
        const Group& g = p.groups[gi];
        std::vector<Chunk> out;
        for (int s0 = g.s0, s1; s0 < g.s1; s0 = s1) {
            s1 = s0 + 1;
            while (s1 < g.s1 && p.row_off[s1 + 1] - p.row_off[s0] <= chunk_rows) ++s1;
            const long long rows = p.row_off[s1] - p.row_off[s0], n = (rows + chunk_rows - 1) / chunk_rows;
            cut(s0, s1, (long long)align_up((size_t)((rows + n - 1) / n), GEMM_TILE), out);
        }
        return out;
    }
    // Full chunks, wherever samples end.
    std::vector<Chunk> of_nodes() const {
        std::vector<Chunk> out;
        cut(p.groups[gi].s0, p.groups[gi].s1, chunk_rows, out);
        return out;
    }
    // What an order costs beyond the other, in microseconds.  Fitted to both orders of 91 calls, 16 to 200 samples of 40 x 8 to 1000 x 200, H x V from 64 x 64
    // to 1024 x 4096, default workspaces to 1/24 of them: the order that is then chosen was the slower one in six of them, by at most 2.3 %; of
    // 40 calls of random sizes and workspaces in one that was seen, two samples of 580 x 175, H = 368, V = 520 (3.66 ms, the other order 3.47).
    double cost(const std::vector<Chunk>& chunks) const {
        const double H = d.H, V = d.V;
        // a chunk: its launches, and its GEMMs' last, partly empty round
        double us = (double)chunks.size() * (75.0 + 0.04 * (H + V));
        // a node's scores, computed again: Z (a workgroup a node), the GEMM, and the bytes of both
        const double again = 0.5e-3 + 2.0 * H * std::max(V, 128.0) / 250e6 + (8.0 * H + 4.0 * V) / 2.4e6;
        for (size_t i = 0; i < chunks.size(); ++i) {
            const Chunk& c = chunks[i];
            if (i + 1 < chunks.size() && chunks[i + 1].s0 == c.s0) {
                us += 25.0 + (double)c.rows * again;
                continue;
            }
            // the sweep of the chunk's samples: a step of the longest one's; more wavefronts than SIMDs take turns
            int steps = 0, waves = 0;
            for (int s = c.s0; s < c.s1; ++s) {
                steps = std::max(steps, T_len[s] + U_len[s]);
                waves = std::max(waves, (U_len[s] + 64) / 64);
            }
            const double step = d.T_max + d.U_max >= 128 ? 0.28 + 0.045 * waves : 0.075;
            us += 7.0 + steps * step * std::max(1.0, 2.0 * (c.s1 - c.s0) * waves / 1024.0);
        }
        return us;
    }
};

}  // namespace

void build_plan(const rnnt_desc& d, const int32_t* T_len, const int32_t* U_len,
                size_t workspace_bytes, Plan& p, bool two_lattice_buffers, bool grads) {
    const int B = d.B;
    p.B = B;
    p.lat_buffers = two_lattice_buffers ? 2 : 1;
    const long long lat_row_bytes = 20LL * p.lat_buffers;    // workspace bytes per lattice node a group may hold
    p.bf16 = (d.dtype == RNNT_BF16);
    p.keep = p.bf16 && d.keep_scores;
    p.stage = p.bf16 && d.input_grads_bf16;
    // 0: on the bf16 paths, tiles whose score gradients are all zero as bf16 values are left out
    // (ZERO_IN_BF16_LOG2); -1: no tile is ever left out
    p.skip_log2 = d.skip_below_log2 > 0 ? d.skip_below_log2
                  : (d.skip_below_log2 == 0 && p.bf16) ? ZERO_IN_BF16_LOG2 : 0;
    p.f32_gemm = !p.bf16 && f32_gemm_shape(d.H, d.V);
    const bool chunked = p.bf16 || p.f32_gemm;
    const size_t stage_per_sample = ((size_t)d.T_max + d.U_max + 1) * d.H * 4;
    p.tile_off.assign(B + 1, 0);
    p.row_off.assign(B + 1, 0);
    long long max_rows = 0, max_tile_rows = 0;
    for (int b = 0; b < B; ++b) {
        long long rows = (long long)T_len[b] * (U_len[b] + 1);
        long long tiles = sample_tiles(T_len[b], U_len[b]);
        p.row_off[b + 1] = p.row_off[b] + rows;
        p.tile_off[b + 1] = (int)(p.tile_off[b] + tiles);
        max_rows = std::max(max_rows, rows);
        max_tile_rows = std::max(max_tile_rows, (long long)align_up((size_t)tiles * TILE_ROWS, GEMM_TILE));
    }
    p.rows_total = p.row_off[B];
    p.tiles_total = p.tile_off[B];
    // the most rows a chunk can hold: tile rows (bf16), lattice nodes (fp32 GEMM form)
    const long long all_tile_rows =
        (long long)align_up((size_t)(p.bf16 ? p.tiles_total * TILE_ROWS : p.rows_total), GEMM_TILE);
    const size_t crb = p.f32_gemm ? (size_t)4 * d.V + (size_t)8 * d.H
                       : !p.bf16  ? 0
                                  : (size_t)2 * chunk_pitch(d.V) + (size_t)2 * chunk_pitch(d.H) +
                                        (p.keep ? (size_t)(d.V / 64) * 4 : 0);
    // With kept scores a group's backward pass is one chunk: the chunk buffers hold whole samples.
    const long long chunk_floor = p.keep ? max_tile_rows : GEMM_TILE;

    // smallest workable plan: one (largest) sample per group, one GEMM tile of rows per chunk
    Plan tmp = p;
    p.min_bytes = lay_out(d, tmp, max_rows, chunked ? chunk_floor : 0, p.stage ? 1 : 0);

    // the default plan; a caller that passes exactly the size it was told gets exactly this plan back
    const long long lat_default = std::min(p.rows_total, std::max(max_rows, (256LL << 20) / lat_row_bytes));
    long long chunk_default = 0;
    if (chunked) {
        // 832 MiB: 768 MiB of rows at H = 512, V = 1024 plus the padding of their row pitch
        // kept scores: 8 GiB, so that a group still fills the GPU when a row takes 10 KB
        const unsigned long long budget = p.keep ? (8ULL << 30) : (832ULL << 20);
        long long by_bytes = (long long)(budget / crb) / GEMM_TILE * GEMM_TILE;
        // fp32: up to 2 GiB where the longest sample needs them, so that its scores are computed once (H = 1024, V = 4096, four samples of up to 500 x 100,
        // 45 k nodes each where 832 MiB hold 35 k: 30.9 -> 26.3 ms a call).  (2 GiB for every call would give 1 to 12 % more.)
        if (p.f32_gemm)
            by_bytes = std::max(by_bytes, std::min((long long)align_up((size_t)max_rows, GEMM_TILE), (long long)((2ULL << 30) / crb) / GEMM_TILE * GEMM_TILE));
        chunk_default = std::min(all_tile_rows, std::max<long long>(chunk_floor, by_bytes));
    }
    // fp32 sums of d_enc, d_pred for the samples of a group: 256 MiB by default
    const long long stage_default =
        !p.stage ? 0 : std::min<long long>(B, std::max<long long>(1, (long long)((256ULL << 20) / stage_per_sample)));
    Plan dflt = p;
    const size_t default_bytes = lay_out(d, dflt, lat_default, chunk_default, stage_default);

    long long lat_cap, chunk_rows, stage_samples;
    if (workspace_bytes == 0 || workspace_bytes == default_bytes) {
        lat_cap = lat_default;
        chunk_rows = chunk_default;
        stage_samples = stage_default;
    } else if (workspace_bytes < p.min_bytes) {
        lat_cap = max_rows;
        chunk_rows = chunked ? chunk_floor : 0;
        stage_samples = p.stage ? 1 : 0;
    } else {
        // the fixed part and the alignment slack come off first
        Plan probe = p;
        size_t fixed = lay_out(d, probe, 0, 0, 0) + 10 * WS_ALIGN;
        size_t avail = workspace_bytes > fixed ? workspace_bytes - fixed : 0;
        // an eighth of the rest (at most the default) for the fp32 sums of a group
        stage_samples = !p.stage ? 0
                                 : std::min<long long>(stage_default,
                                                       std::max<long long>(1, (long long)(avail / 8 / stage_per_sample)));
        const size_t stage_bytes = (size_t)stage_samples * stage_per_sample;
        avail = avail > stage_bytes ? avail - stage_bytes : 0;
        if (!chunked) {
            lat_cap = std::min<long long>(p.rows_total, std::max<long long>(max_rows, (long long)(avail / lat_row_bytes)));
            chunk_rows = 0;
        } else {
            long long lat_quarter = (long long)(avail / 4 / lat_row_bytes);
            lat_cap = std::min(p.rows_total, std::max(max_rows, lat_quarter));
            size_t lat_bytes = (size_t)lat_cap * lat_row_bytes;
            size_t rest = avail > lat_bytes ? avail - lat_bytes : 0;
            chunk_rows = (long long)(rest / crb) / GEMM_TILE * GEMM_TILE;
            chunk_rows = std::min(all_tile_rows, std::max<long long>(chunk_floor, chunk_rows));
            // what the chunk buffers do not need goes to the lattice
            size_t chunk_bytes = (size_t)chunk_rows * crb;
            if (avail > chunk_bytes) {
                long long more = (long long)((avail - chunk_bytes) / lat_row_bytes);
                lat_cap = std::min(p.rows_total, std::max(lat_cap, more));
            }
        }
        // never below the minimum, never above the given size
        Plan t2 = p;
        while (lay_out(d, t2, lat_cap, chunk_rows, stage_samples) > workspace_bytes) {
            if (chunk_rows > chunk_floor) chunk_rows -= GEMM_TILE;
            else if (lat_cap > max_rows) lat_cap = std::max(max_rows, lat_cap - 4096);
            else if (stage_samples > 1) --stage_samples;
            else break;
        }
    }
    // the kernels index a group's lattice state with 32-bit integers (a sample alone has at most 2^30 nodes)
    lat_cap = std::min<long long>(lat_cap, 2147483647LL);
    lay_out(d, p, lat_cap, chunk_rows, stage_samples);
    if (workspace_bytes != 0 && workspace_bytes < p.min_bytes) p.total_bytes = p.min_bytes;

    // groups: consecutive samples while the lattice state fits
    p.groups.clear();
    p.chunks.clear();
    p.group_chunks.clear();
    int s = 0;
    while (s < B) {
        Group g{};
        g.s0 = s;
        g.rows = 0;
        g.u_max = 0;
        while (s < B) {
            long long rows = p.row_off[s + 1] - p.row_off[s];
            if (g.rows > 0 && g.rows + rows > lat_cap) break;
            if (p.stage && s - g.s0 >= stage_samples) break;
            if (p.keep && g.rows > 0 &&
                (long long)align_up((size_t)(p.tile_off[s + 1] - p.tile_off[g.s0]) * TILE_ROWS, GEMM_TILE) > chunk_rows)
                break;
            g.rows += rows;
            g.u_max = std::max(g.u_max, (int)U_len[s]);
            ++s;
        }
        g.s1 = s;
        g.tile0 = p.tile_off[g.s0];
        g.tile1 = p.tile_off[g.s1];
        p.groups.push_back(g);
    }
    // backward chunks of at most chunk_rows rows: a group that fits one chunk is one chunk; a larger one is cut
    // into chunks of a whole number of 256 tiles where the chunk buffers hold at least four times that (the last chunk
    // takes the rest), else into equal parts of an even number of tiles
    if (p.bf16 && !p.keep) {
        const long long cap_tiles = chunk_rows / TILE_ROWS;
        for (int gi = 0; gi < (int)p.groups.size(); ++gi) {
            const Group& g = p.groups[gi];
            long long n = g.tile1 - g.tile0;
            long long nch = (n + cap_tiles - 1) / cap_tiles;
            long long per = (n + nch - 1) / nch;
            per = std::min(cap_tiles, (per + 1) / 2 * 2);
            // chunks of whole multiples of 256 tiles: the dz GEMM takes 4 tiles x 256 hidden columns per workgroup, so 256 tiles are
            // one round of the chip at H = 1024, and half a one at H = 512 (B=64, T<=500, U<=100, H=1024, V=4096: 5 rounds instead of
            // 5.3 per chunk, -12 %, measured when dz took a tile per workgroup); the other kernels take two or four tiles
            // per workgroup and split the vocabulary where that fills their rounds better (vocabulary_split)
            if (cap_tiles >= 1024 && n > cap_tiles) per = cap_tiles / 256 * 256;
            for (long long t = g.tile0; t < g.tile1; t += per) {
                Chunk c{gi, (int)t, (int)std::min<long long>(g.tile1, t + per)};
                p.chunks.push_back(c);
            }
        }
    } else if (p.f32_gemm) {
        for (int gi = 0; gi < (int)p.groups.size(); ++gi) {
            const F32Chunks c{d, T_len, U_len, p, gi, chunk_rows};
            std::vector<Chunk> chunks = c.of_nodes();
            if (p.lat_buffers == 2) p.group_chunks.insert(p.group_chunks.end(), chunks.begin(), chunks.end());
            if (grads) {                              // (losses alone: no score is needed again)
                std::vector<Chunk> samples = c.of_samples();
                if (c.cost(samples) <= c.cost(chunks)) chunks.swap(samples);
            }
            p.chunks.insert(p.chunks.end(), chunks.begin(), chunks.end());
        }
    } else {
        for (int gi = 0; gi < (int)p.groups.size(); ++gi)
            p.chunks.push_back(Chunk{gi, p.groups[gi].tile0, p.groups[gi].tile1});
    }
    if (p.bf16) {
        p.one_grid = p.chunks.size() == 1 && one_grid_shape(d.H, d.V, p.tiles_total);
        p.dw_splits = p.one_grid ? dw_split_one_grid(d.H, d.V, p.tiles_total) : dw_split_choice(d.H, d.V, chunk_rows);
    }
}

}  // namespace rnnt
