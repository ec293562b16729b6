// Forward/backward variables of the transducer lattice (f^W_2) and the loss (f^W_3) in log space.
//
// blockIdx.y = 0 sweeps alpha from (0,0), blockIdx.y = 1 beta from (T-1,U), one anti-diagonal per step; the lattice arrays lie in
// that order (kernels.h: lattice_index).  A lane owns a label position; the value of the neighbouring frame is its own
// previous result, that of the neighbouring column the next lane's.
//
// Every alignment emits exactly T blanks and U labels, so adding a constant c to every emission
// log-probability shifts ln P by c*(T+U) and leaves all posteriors unchanged.  c is chosen per
// sample (minus the mean of the larger of the two emission log-probabilities over the lattice)
// so that alpha and beta stay near zero instead of growing to thousands, which keeps fp32
// resolution for the posteriors of long utterances.  The fp32 path's long sweeps (k_lattice_f64)
// accumulate in fp64 and take c = -ln P / (T+U) from a first sweep.
#include "device_common.h"
#include "scaled.h"

namespace rnnt {

constexpr int LAT_MAX_T = 1024; // threads per workgroup (label positions 0..U <= 1023)

// This thread's share (i = first, first + stride, ...) of the sum over the lattice of the larger emission of a node: from the per-tile sums
// the bf16 forward kernels leave behind (a few hundred numbers), else from the emissions.  The sweep cannot start before
// this sum is known, and a workgroup has few threads for the size of a lattice: LAT_SUM_DEPTH independent loads are in
// flight per thread, so that few memory latencies are exposed.
constexpr int LAT_SUM_DEPTH = 24;
__device__ __forceinline__ float emission_sum_partial(const SampleTable& st, const LatticeState& ls, int s, const float2* __restrict__ em,
                                                      int n, int first, int stride) {
    float acc[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    auto add_all = [&](int end, auto&& value) {
        for (int i0 = first; i0 < end; i0 += LAT_SUM_DEPTH * stride) {
            float v[LAT_SUM_DEPTH];
#pragma unroll
            for (int j = 0; j < LAT_SUM_DEPTH; ++j) {
                const int i = i0 + j * stride;
                v[j] = value(i < end ? i : first);
            }
#pragma unroll
            for (int j = 0; j < LAT_SUM_DEPTH; ++j) acc[j & 7] += i0 + j * stride < end ? v[j] : 0.0f;
        }
    };
    if (ls.tile_esum != nullptr) {
        const float* __restrict__ esum = ls.tile_esum + st.tile_off[s];
        add_all(st.tile_off[s + 1] - st.tile_off[s], [&](int i) { return esum[i]; });
    } else {
        add_all(n, [&](int i) { const float2 e = em[i]; return fmaxf(fmaxf(e.x, e.y), OFFSET_FLOOR); });
    }
    return ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
}
// The sample's offset c, in every thread.  Formed by as many wavefronts as the sample has blocks of 64 columns, so that it does not depend on
// which other samples share the launch, and is the same in both workgroups of a sample.
__device__ __forceinline__ float emission_offset(const SampleTable& st, const LatticeState& ls, int s, const float2* __restrict__ em, int n,
                                                 float* red) {
    const int waves = (st.U[s] + 64) >> 6;
    float acc = 0.0f;
    if ((int)threadIdx.x < 64 * waves) acc = wave_sum(emission_sum_partial(st, ls, s, em, n, (int)threadIdx.x, 64 * waves));
    if (blockDim.x > 64) {
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
        __syncthreads();
        acc = 0.0f;
        for (int w = 0; w < waves; ++w) acc += red[w];
    }
    return -acc / (float)n;
}

// ---- sweep in fp32.  A wavefront owns 64 label positions; with more of them a workgroup has as many wavefronts as it takes,
// each a block of steps behind the one that holds the columns below, whose last column's values come through LDS.  One barrier per
// block (none with a single wavefront).
//
// What bounds it: the issue of a wavefront's instructions and the dependent chain of a step, shift - difference - exp2 - add -
// log2 - add (values are kept as logarithms to base 2, so nothing is scaled on the way).  Emissions are loaded (BLOCKS - 1) LW_B steps
// ahead into registers, one 8-byte load per step and lane, whole lines (the arrays lie by anti-diagonals); about half of them are in flight at a time,
// since the compiler does not count the store of each step in its waits.  No lane is masked but in the store: what lies outside the lattice is a finite value that never reaches a lane inside (before its first frame
// a column holds LW_NONE, which absorbs whatever is added; past its last frame and past the last column nothing flows back).
//
// Measured against the sweep it replaces (one anti-diagonal per step over row-major arrays, a barrier per step above 64 label positions): 250 x 50,
// one sample 43 -> 25 us; 500 x 100, 16 samples 191 -> 56 us; 1000 x 200, 113 samples 660 -> 119 us.  The error of ln gamma against 64 bits (where
// gamma is not negligible, root mean square over 24 to 256 samples a shape, 45 x 8 to 1000 x 200) is 0.77 of what it was for the scores of a random network
// and 0.96 for scores six times as large, geometric means over 14 batches each.
constexpr int LW_B = 8;                   // steps per block
constexpr float LW_NONE = -1e30f;         // ln 0

// Value of lane l-1; lane 0 gets `first`.
__device__ __forceinline__ float lane_from_below(float v, float first) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(first), __float_as_int(v), 0x138 /* wave_shr:1 */, 0xf, 0xf, false));
}

// Value of lane l+1 (lane 63: any).
__device__ __forceinline__ float lane_from_above(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130 /* wave_shl:1 */, 0xf, 0xf, true));
}

// Returns (STORE = false, alpha, the lane with v = U) ln P with the offset c.
// BLOCKS (even): blocks in registers, the current one and those ahead of it.
template <bool BETA, bool MANY, bool STORE, int BLOCKS>
__device__ __forceinline__ float lattice_sweep(const SampleTable& st, const LatticeState& ls, int s, float c, float* __restrict__ loss,
                                               float (*edge)[2][LW_B]) {
    const int lane = threadIdx.x & 63, wave = MANY ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
    const int waves = MANY ? (int)(blockDim.x >> 6) : 1;
    const int T = st.T[s], U = st.U[s], W = U + 1, n = T * W;
    const long long base = st.row_off[s] - ls.row_base;
    const float2* __restrict__ em = ls.em + base;
    float* out = (BETA ? ls.beta : ls.alpha) + base;
    // (in scalar registers: the store below is written as text)
    const unsigned long long out_bits = (unsigned long long)out;
    const unsigned long long out_s = ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(out_bits >> 32)) << 32) |
                                     (unsigned)__builtin_amdgcn_readfirstlane((int)out_bits);
    const float c2 = c * LOG2E_F;
    const int nsteps = T + U;
    const int v = 64 * wave + lane;               // column in sweep order: label position v (alpha), U - v (beta)
    const unsigned T_act = v < W ? (unsigned)T : 0u;
    const int v_off = BETA ? U - v : v;

    // Memory position of column 0 (its label position 0) on the diagonals of block b, diagonal LW_B b + j in lane j.
    auto block_base = [&](int b) {
        int k = LW_B * b + (lane & (LW_B - 1));
        k = k < 0 ? 0 : k < nsteps ? k : nsteps - 1;
        const int K = BETA ? nsteps - 1 - k : k;
        return diagonal_offset(T, W, K) - (K >= T ? K - T + 1 : 0);
    };
    // Node of this lane at step j of a block (clamped into the sample: lanes without a node read some other one's emissions)
    auto node = [&](int bases, int j) {
        const unsigned i = (unsigned)(__builtin_amdgcn_readlane(bases, j) + v_off);
        return i < (unsigned)(n - 1) ? i : (unsigned)(n - 1);
    };
    float2 e[BLOCKS][LW_B];
    unsigned at[BLOCKS][LW_B];
    auto load = [&](auto slot_tag, int bases, auto j_tag) {
        constexpr int slot = decltype(slot_tag)::value, j = decltype(j_tag)::value;
        at[slot][j] = node(bases, j);
        e[slot][j] = em[at[slot][j]];
    };
    static_for<0, BLOCKS - 1>([&](auto q) {
        const int bases = block_base(decltype(q)::value - wave);
        static_for<0, LW_B>([&](auto j) { load(q, bases, j); });
    });
    // A node's value is kept as the larger of its two ways, m, and what the other one adds, l in [0, 1]; what leaves for the next step is
    // m + (l + emission): one rounding at the size of the values per step instead of two.  pb: to this lane's column, py: to the
    // next one's.  alpha adds the emissions of the node that is left; beta those of the node that is entered, py the next lane's.
    float pb = LW_NONE, py = LW_NONE, ey_here = 0.0f;
    if constexpr (BETA) ey_here = fmaf(e[0][0].y, LOG2E_F, c2);
    if (v == 0) pb = BETA ? fmaf(e[0][0].x, LOG2E_F, c2) : 0.0f;
    const int nblk = (nsteps + LW_B - 1) / LW_B, total = nblk + waves - 1;
    float fin = 0.0f;
    float carry = LW_NONE;                        // last column of the wavefront below, at the step before the block
    for (int i0 = 0; i0 < total; i0 += BLOCKS) {
        static_for<0, BLOCKS>([&](auto q_tag) {
            constexpr int q = decltype(q_tag)::value;
            const int i = i0 + q, b = i - wave;
            float below = LW_NONE;                            // lane j: the last column of the wavefront below at step j
            f32x4 above[LW_B / 4];                            // this lane's values
            if (MANY && wave > 0) below = edge[wave - 1][(q + 1) & 1][lane & (LW_B - 1)];
            const int bases_ahead = block_base(b + BLOCKS - 1);
            static_for<0, LW_B>([&](auto j_tag) {
                constexpr int j = decltype(j_tag)::value;
                const int k = LW_B * b + j;
                float first = LW_NONE;
                if (MANY) {
                    first = j == 0 ? carry : __int_as_float(__builtin_amdgcn_readlane(__float_as_int(below), j - 1));
                    if (BETA) first += ey_here;
                }
                const float x = pb, y = lane_from_below(py, first), m = fmaxf(x, y);
                // (the argument of the logarithm lies in [1, 2]: no range fix-up is needed)
                const float l = __builtin_amdgcn_logf(1.0f + __builtin_amdgcn_exp2f(-fabsf(x - y))), val = m + l;
                const float2 ev = !BETA ? e[q][j] : j + 1 < LW_B ? e[q][(j + 1) % LW_B] : e[(q + 1) % BLOCKS][0];
                const float eb = fmaf(ev.x, LOG2E_F, c2), ey = fmaf(ev.y, LOG2E_F, c2);
                pb = m + (l + eb);
                py = m + (l + (BETA ? lane_from_above(ey) : ey));
                ey_here = ey;
                if (MANY) above[j / 4][j % 4] = BETA ? val : py;
                if constexpr (!STORE) fin = k == nsteps - 1 ? pb : fin;
                const unsigned long long inside = __builtin_amdgcn_ballot_w64((unsigned)(k - v) < T_act);
                // (as text: a branch around a store costs as much as the step's arithmetic)
                if constexpr (STORE)
                    asm volatile("s_mov_b64 exec, %3\n\tglobal_store_dword %0, %1, %2\n\ts_mov_b64 exec, -1" ::"v"(at[q][j] * 4u), "v"(val * LN2_F),
                                 "s"(out_s), "s"(inside));
                load(std::integral_constant<int, (q + BLOCKS - 1) % BLOCKS>{}, bases_ahead, j_tag);
                __builtin_amdgcn_sched_barrier(0);
            });
            if (MANY) {
                if (wave > 0) carry = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(below), LW_B - 1));
                if (wave + 1 < waves && lane == 63)
#pragma unroll
                    for (int h = 0; h < LW_B / 4; ++h) *reinterpret_cast<f32x4*>(&edge[wave][q & 1][4 * h]) = above[h];
                __syncthreads();
            }
        });
    }
    if constexpr (!STORE) return fin * LN2_F;
    if (!BETA && v == U) {
        // alpha[T-1,U] and the final blank
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const double lnP2 = *(volatile const float*)(out + (n - 1)) / (double)LN2_F + fma((double)em[n - 1].x, (double)LOG2E_F, (double)c2);
        // (the offset as it was added, T + U times, and the emissions as they were scaled: neither one's rounding stays in the loss)
        const double lnP_true = (lnP2 - (double)c2 * (T + U)) / LOG2E_F;
        const bool none = no_alignment(lnP_true);
        ls.lnP[s] = none ? RNNT_NEG_INF : (float)(lnP2 * LN2_F);
        ls.shift[s] = c2 * LN2_F;
        loss[s] = none ? -RNNT_NEG_INF : (float)-lnP_true;
    }
    return 0.0f;
}

template <int MAX_WAVES>
__global__ __launch_bounds__(64 * MAX_WAVES) void k_lattice_wave(SampleTable st, LatticeState ls, int s0, float* __restrict__ loss) {
    __shared__ float red[MAX_WAVES];
    __shared__ __align__(16) float edge[MAX_WAVES][2][LW_B];
    // (no wavefront has left an edge for the first block: nothing flows in)
    if (MAX_WAVES > 1 && threadIdx.x < MAX_WAVES * LW_B) edge[threadIdx.x / LW_B][1][threadIdx.x % LW_B] = LW_NONE;
    const int s = s0 + blockIdx.x;
    const float c = emission_offset(st, ls, s, ls.em + (st.row_off[s] - ls.row_base), st.T[s] * (st.U[s] + 1), red);
    constexpr int BLOCKS = MAX_WAVES > 8 ? 2 : 4;     // (registers)
    if (blockIdx.y == 0) lattice_sweep<false, (MAX_WAVES > 1), true, BLOCKS>(st, ls, s, c, loss, edge);
    else lattice_sweep<true, (MAX_WAVES > 1), true, BLOCKS>(st, ls, s, c, loss, edge);
}

// ---- sweep in fp64 (fp32 path, 128 steps or more): the recursion accumulates in fp64 and alpha, beta are rounded to fp32 once, when stored (a
// sweep of T+U dependent fp32 log-add-exps loses about sqrt(T+U) half-ulps of values of the order of 100, 2e-4 relative in
// the posteriors of a 500 x 100 lattice).  The same wavefronts, blocks and loads as the fp32 sweep.  A value is m 2^k: a step multiplies the two ways
// by their emissions, brings them to the larger k and adds, so the dependent chain holds no exponential and no logarithm; those of the emissions and of
// what is stored stand beside it.  k is a whole number in fp64, so no emission is too small for it (EMISSION_FLOOR included).
// What bounds it: issue, about 115 instructions a step.  One thread per label position, a barrier per step and the recursion in logarithms before: 16 samples
// of 120 x 24 135 -> 49 us, four of 500 x 100 503 -> 219, one of 300 x 600 977 -> 712.  A step's functions are good to the last places of fp64 (scaled.h);
// with exponentials good to 1e-11 the same three took 47, 212 and 686.
constexpr double LW_NONE_K = -1e280;      // 0 = 2^LW_NONE_K (absorbs whatever is added)

__device__ __forceinline__ double from_words(int lo, int hi) { return __hiloint2double(hi, lo); }
__device__ __forceinline__ double lane_from_below(double v, double first) {
    return from_words(__builtin_amdgcn_update_dpp(__double2loint(first), __double2loint(v), 0x138, 0xf, 0xf, false),
                      __builtin_amdgcn_update_dpp(__double2hiint(first), __double2hiint(v), 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ double lane_value(double v, int lane) {
    return from_words(__builtin_amdgcn_readlane(__double2loint(v), lane), __builtin_amdgcn_readlane(__double2hiint(v), lane));
}

template <bool BETA, bool MANY, int BLOCKS>
__device__ __forceinline__ void lattice_sweep_f64(const SampleTable& st, const LatticeState& ls, int s, float c, float* __restrict__ loss,
                                                  Scaled (*edge)[2][LW_B]) {
    const int lane = threadIdx.x & 63, wave = MANY ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
    const int waves = MANY ? (int)(blockDim.x >> 6) : 1;
    const int T = st.T[s], U = st.U[s], W = U + 1, n = T * W;
    const long long base = st.row_off[s] - ls.row_base;
    const float2* __restrict__ em = ls.em + base;
    float* __restrict__ out = (BETA ? ls.beta : ls.alpha) + base;
    const double cd = (double)c;
    const int nsteps = T + U;
    const int v = 64 * wave + lane;               // column in sweep order: label position v (alpha), U - v (beta)
    const unsigned T_act = v < W ? (unsigned)T : 0u;
    const int v_off = BETA ? U - v : v;

    // (as in the fp32 sweep)
    auto block_base = [&](int b) {
        int k = LW_B * b + (lane & (LW_B - 1));
        k = k < 0 ? 0 : k < nsteps ? k : nsteps - 1;
        const int K = BETA ? nsteps - 1 - k : k;
        return diagonal_offset(T, W, K) - (K >= T ? K - T + 1 : 0);
    };
    auto node = [&](int bases, int j) {
        const unsigned i = (unsigned)(__builtin_amdgcn_readlane(bases, j) + v_off);
        return i < (unsigned)(n - 1) ? i : (unsigned)(n - 1);
    };
    float2 e[BLOCKS][LW_B];
    unsigned at[BLOCKS][LW_B];
    auto load = [&](auto slot_tag, int bases, auto j_tag) {
        constexpr int slot = decltype(slot_tag)::value, j = decltype(j_tag)::value;
        at[slot][j] = node(bases, j);
        e[slot][j] = em[at[slot][j]];
    };
    static_for<0, BLOCKS - 1>([&](auto q) {
        const int bases = block_base(decltype(q)::value - wave);
        static_for<0, LW_B>([&](auto j) { load(q, bases, j); });
    });
    const Scaled none{1.0, LW_NONE_K};
    // What leaves a node for the next step, to this lane's column and to the next one's: alpha with the node's own emissions, beta without any (those of
    // the node that is entered are taken there).
    Scaled to_own = none, to_next = none, fin = none;
    if (v == 0) to_own = Scaled{1.0, 0.0};
    const int nblk = (nsteps + LW_B - 1) / LW_B, total = nblk + waves - 1;
    Scaled carry = none;                          // last column of the wavefront below, at the step before the block
    for (int i0 = 0; i0 < total; i0 += BLOCKS) {
        static_for<0, BLOCKS>([&](auto q_tag) {
            constexpr int q = decltype(q_tag)::value;
            const int i = i0 + q, b = i - wave;
            Scaled below = none;                              // lane j: the last column of the wavefront below at step j
            if (MANY && wave > 0) below = edge[wave - 1][(q + 1) & 1][lane & (LW_B - 1)];
            const int bases_ahead = block_base(b + BLOCKS - 1);
            static_for<0, LW_B>([&](auto j_tag) {
                constexpr int j = decltype(j_tag)::value;
                const int k = LW_B * b + j;
                Scaled first = none;
                if (MANY) first = j == 0 ? carry : Scaled{lane_value(below.m, j - 1), lane_value(below.k, j - 1)};
                Scaled x = to_own, y{lane_from_below(to_next.m, first.m), lane_from_below(to_next.k, first.k)};
                const Scaled eb = scaled_exp((double)e[q][j].x + cd), ey = scaled_exp((double)e[q][j].y + cd);
                if constexpr (BETA) {
                    x = times(x, eb);
                    y = times(y, ey);
                }
                Scaled val = plus(x, y);
                if constexpr (j == LW_B - 1) {                // (the mantissa of a value stays within 2^(2 LW_B) of 1)
                    int up;
                    const double m = mantissa(val.m, up);
                    val = Scaled{m, val.k + up};
                }
                to_own = BETA ? val : times(val, eb);
                to_next = BETA ? val : times(val, ey);
                if (!BETA) {
                    const bool end = k == nsteps - 1;
                    fin.m = end ? to_own.m : fin.m;
                    fin.k = end ? to_own.k : fin.k;
                }
                if (MANY && wave + 1 < waves && lane == 63) edge[wave][q & 1][j] = to_next;
                if ((unsigned)(k - v) < T_act) out[at[q][j]] = (float)scaled_log(val);
                load(std::integral_constant<int, (q + BLOCKS - 1) % BLOCKS>{}, bases_ahead, j_tag);
                __builtin_amdgcn_sched_barrier(0);
            });
            if (MANY) {
                if (wave > 0) carry = Scaled{lane_value(below.m, LW_B - 1), lane_value(below.k, LW_B - 1)};
                __syncthreads();
            }
        });
    }
    if (!BETA && v == U) {
        const double lnP_off = scaled_log(fin), lnP_true = lnP_off - cd * (double)(T + U);
        const bool none_possible = no_alignment(lnP_true);
        ls.lnP[s] = none_possible ? RNNT_NEG_INF : (float)lnP_off;
        ls.shift[s] = c;
        loss[s] = none_possible ? -RNNT_NEG_INF : (float)-lnP_true;
    }
}

template <int MAX_WAVES>
__global__ __launch_bounds__(64 * MAX_WAVES) void k_lattice_f64(SampleTable st, LatticeState ls, int s0, float* __restrict__ loss) {
    constexpr bool MANY = MAX_WAVES > 1;
    // A step takes long enough that loads eight steps ahead suffice, in the first sweep, too (four blocks there: four samples of 500 x 100 606 -> 610 us a
    // call).  Sixteen wavefronts leave 128 registers each; 25 of them are spilled, and the sweep still takes less time than the one it replaces.
    constexpr int BLOCKS = 2;
    __shared__ float red[MAX_WAVES];
    __shared__ __align__(16) float edge32[MAX_WAVES][2][LW_B];
    __shared__ __align__(16) Scaled edge[MAX_WAVES][2][LW_B];
    __shared__ float c_better;
    if (threadIdx.x < MAX_WAVES * LW_B) {
        edge32[threadIdx.x / LW_B][1][threadIdx.x % LW_B] = LW_NONE;
        edge[threadIdx.x / LW_B][1][threadIdx.x % LW_B] = Scaled{1.0, LW_NONE_K};
    }
    const int s = s0 + blockIdx.x, T = st.T[s], U = st.U[s];
    const float c_mean = emission_offset(st, ls, s, ls.em + (st.row_off[s] - ls.row_base), T * (U + 1), red);
    // alpha and beta are still stored as fp32, so their magnitude where the posteriors
    // are not negligible decides the accuracy.  With c = -ln P / (T+U) the offset ln P is zero and alpha, beta
    // stay near zero along the alignments that carry the probability, whatever the emissions look like (flat
    // scores, where the number of alignments adds hundreds to ln P, or peaked ones).  ln P is not known
    // beforehand: both workgroups of the sample first run the fp32 alpha sweep without storing anything (the same arithmetic in
    // both, hence the same c; any c near it would do), then the sweep proper.
    const double lnP_off = lattice_sweep<false, MANY, false, BLOCKS>(st, ls, s, c_mean, nullptr, edge32), steps = T + U;
    if ((int)threadIdx.x == U) c_better = no_alignment(lnP_off - c_mean * steps) ? c_mean : (float)(c_mean - lnP_off / steps);
    __syncthreads();
    if (blockIdx.y == 0) lattice_sweep_f64<false, MANY, BLOCKS>(st, ls, s, c_better, loss, edge);
    else lattice_sweep_f64<true, MANY, BLOCKS>(st, ls, s, c_better, loss, edge);
}

hipError_t launch_lattice(const SampleTable& st, const LatticeState& ls, int s0, int s1, int u_max, int wide,
                          float* loss, hipStream_t stream) {
    if (s1 <= s0) return hipSuccess;
    const int waves = (u_max + 64) / 64;
    if (64 * waves > LAT_MAX_T) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(s1 - s0), 2), threads(64 * waves);
    if (wide && waves == 1) k_lattice_f64<1><<<grid, threads, 0, stream>>>(st, ls, s0, loss);
    else if (wide && waves <= 8) k_lattice_f64<8><<<grid, threads, 0, stream>>>(st, ls, s0, loss);
    else if (wide) k_lattice_f64<16><<<grid, threads, 0, stream>>>(st, ls, s0, loss);
    else if (waves == 1) k_lattice_wave<1><<<grid, threads, 0, stream>>>(st, ls, s0, loss);
    else if (waves <= 8) k_lattice_wave<8><<<grid, threads, 0, stream>>>(st, ls, s0, loss);
    else k_lattice_wave<16><<<grid, threads, 0, stream>>>(st, ls, s0, loss);
    return hipGetLastError();
}

}  // namespace rnnt
