"""CPU-only tests of the C-ABI library: it loads, exports what the header declares, rejects bad
arguments before touching a GPU, and its scheduler packs samples as promised."""
import ctypes
import os
import re

import numpy as np
import pytest

from paper_2211_16270_amd import binding as Bd
from paper_2211_16270_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "rnnt_joint_loss.h")
HEADERS = [HEADER, os.path.join(ROOT, "include", "rnnt_joint_loss_debug.h")]
GOLD = os.path.join(ROOT, "tests", "golden")


def test_library_exports_every_declared_symbol():
    text = "".join(open(h).read() for h in HEADERS)
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    declared = set(re.findall(r"\b(rnnt_[a-z_0-9]+)\s*\(", text))
    assert declared == set(Bd.EXPORTS), declared ^ set(Bd.EXPORTS)
    L = Bd.lib()
    for name in declared:
        assert hasattr(L, name), name
    assert L.rnnt_status_string(0) == b"ok"
    for code in range(1, 8):
        assert len(L.rnnt_status_string(code)) > 3


def test_no_hip_error_is_reported_before_one_happened():
    assert Bd.lib().rnnt_last_hip_error() == b""
    assert Bd.lib().rnnt_debug_mfma_loop(None, None, 1, 1, None) == 1   # null pointers are refused on the host
    assert Bd.lib().rnnt_debug_mfma_loop(ctypes.c_void_p(256), ctypes.c_void_p(256), 0, 1, None) == 2
    assert Bd.lib().rnnt_debug_mfma_loop(ctypes.c_void_p(256), ctypes.c_void_p(256), 1, 2000000, None) == 2
    assert Bd.lib().rnnt_debug_mfma_loop_fp8(None, None, 1, 1, None) == 1
    assert Bd.lib().rnnt_debug_mfma_loop_fp8(ctypes.c_void_p(256), ctypes.c_void_p(256), 1, 0, None) == 2


def test_struct_layouts_match_the_header():
    assert ctypes.sizeof(Bd.RnntDesc) == 44
    assert ctypes.sizeof(Bd.RnntPlanInfo) == 8 * 3 + 4 * 2 + 8 * 2 + 8 * 3


def _tiles(T, U):
    """64-row lattice tiles per sample: 8 frames x 8 label positions, or 16 x 4 where that needs 3 % fewer."""
    T, U = np.asarray(T, dtype=np.int64), np.asarray(U, dtype=np.int64)
    a, b = ((T + 7) // 8) * ((U + 8) // 8), ((T + 15) // 16) * ((U + 4) // 4)
    return np.where(b * 33 < a * 32, b, a)


def _lens(name):
    wl = synth.WORKLOADS[name]
    T, U, _ = synth.draw_lengths_labels(wl)
    dt = Bd.RNNT_BF16 if wl.dtype == "bf16" else Bd.RNNT_F32
    return wl, Bd.make_desc(wl.B, wl.T_max, wl.U_max, wl.H, wl.V, 0, dt), T, U


def test_argument_checks_happen_on_the_host():
    wl, desc, T, U = _lens("C2")
    L = Bd.lib()
    dummy = ctypes.c_void_p(0x1000)

    def call(d, Tl, Ul, ws=dummy, ws_bytes=1 << 30, enc=dummy):
        Tl = np.ascontiguousarray(Tl, dtype=np.int32)
        Ul = np.ascontiguousarray(Ul, dtype=np.int32)
        return L.rnnt_joint_loss_fwd_bwd(ctypes.byref(d), enc, dummy, dummy, dummy, dummy, Bd._ip(Tl), Bd._ip(Ul),
                                         dummy, dummy, dummy, dummy, dummy, ws, ws_bytes, None)

    assert call(desc, T, U, enc=None) == 1                       # RNNT_ERR_NULL
    bad = Bd.make_desc(wl.B, wl.T_max, wl.U_max, wl.H, wl.V, wl.V, Bd.RNNT_BF16)
    assert call(bad, T, U) == 2                                  # blank out of range
    T2 = T.copy(); T2[3] = wl.T_max + 1
    assert call(desc, T2, U) == 3
    T2[3] = 0
    assert call(desc, T2, U) == 3
    U2 = U.copy(); U2[0] = -1
    assert call(desc, T, U2) == 3
    assert call(desc, T, U, ws=None) == 5
    assert call(desc, T, U, ws=ctypes.c_void_p(0x1010)) == 5     # misaligned
    assert call(desc, T, U, ws_bytes=4096) == 5                  # too small
    odd = Bd.make_desc(wl.B, wl.T_max, wl.U_max, 500, wl.V, 0, Bd.RNNT_BF16)
    assert call(odd, T, U) == 6                                  # H not supported by the MFMA path
    assert call(desc, T, U, enc=ctypes.c_void_p(0x1004)) == 6    # the kernels need 16-byte aligned arrays
    assert Bd.rnnt_joint_loss_workspace_bytes(bad, T, U) == 0


def test_sample_weights_are_checked_on_the_host():
    wl, desc, T, U = _lens("C2")
    L = Bd.lib()
    dummy = ctypes.c_void_p(0x1000)

    def call(w, ws=dummy):
        w = None if w is None else np.ascontiguousarray(w, dtype=np.float32)
        wp = None if w is None else w.ctypes.data_as(ctypes.POINTER(ctypes.c_float))
        return L.rnnt_joint_loss_fwd_bwd_weighted(ctypes.byref(desc), dummy, dummy, dummy, dummy, dummy, Bd._ip(T),
                                                  Bd._ip(U), wp, dummy, dummy, dummy, dummy, dummy, ws, 1 << 30, None)

    w = np.ones(wl.B, dtype=np.float32)
    for bad in (-0.5, np.nan, np.inf):
        w2 = w.copy(); w2[7] = bad
        assert call(w2) == 8                                     # RNNT_ERR_WEIGHT, before the workspace is looked at
    assert call(w, ws=None) == 5                                 # valid weights: the next check (workspace) fails
    assert call(None, ws=None) == 5                              # no weights = the unweighted call
    assert Bd.lib().rnnt_status_string(8).decode().startswith("a sample weight")


def test_label_validation():
    wl, desc, T, U = _lens("C2")
    _, _, lab = synth.draw_lengths_labels(wl)
    assert Bd.rnnt_validate_labels_host(desc, lab, U) == 0
    lab2 = lab.copy(); lab2[5, U[5] - 1] = wl.V
    assert Bd.rnnt_validate_labels_host(desc, lab2, U) == 4
    lab2[5, U[5] - 1] = 3; lab2[5, wl.U_max - 1] = -9 if U[5] < wl.U_max else 3   # beyond U_len: ignored
    assert Bd.rnnt_validate_labels_host(desc, lab2, U) == 0


def test_parallel_iterations_rule_matches_the_worked_values():
    with open(os.path.join(GOLD, "eq11_parallel_iterations.txt")) as f:
        rows = [l.split() for l in f if l.strip() and not l.startswith("#")]
    for T, U, V, _, pi in rows:
        assert Bd.rnnt_parallel_iterations(int(T), int(U), int(V)) == int(pi)
    assert Bd.rnnt_parallel_iterations(0, 1, 1) == 0


@pytest.mark.parametrize("name", ["C1", "C2", "C3", "C4", "C5"])
def test_default_plan_properties(name):
    wl, desc, T, U = _lens(name)
    n = Bd.rnnt_joint_loss_workspace_bytes(desc, T, U, 0)
    # 256 MiB lattice state + 832 MiB chunk buffers + tables, packed weights and the dW partial sums
    assert 0 < n <= (1088 << 20) + (160 << 20)
    st, info, groups = Bd.rnnt_joint_loss_plan(desc, T, U, n)
    assert st == 0
    rows = T.astype(np.int64) * (U.astype(np.int64) + 1)
    assert info["rows_total"] == rows.sum()
    assert info["rows_padded"] == wl.B * wl.T_max * (wl.U_max + 1)
    tiles = _tiles(T, U)
    assert info["tiles_total"] == tiles.sum()
    assert info["workspace_bytes"] <= n
    # every sample in exactly one group, groups are consecutive, each fits the lattice capacity
    assert groups.min() == 0 and groups.max() == info["n_groups"] - 1
    assert np.all(np.diff(groups) >= 0)
    for g in range(info["n_groups"]):
        assert rows[groups == g].sum() <= info["group_rows_cap"]
    assert info["lattice_bytes"] >= 20 * info["group_rows_cap"]
    if wl.dtype == "bf16":
        assert info["chunk_rows"] % 128 == 0 and info["chunk_rows"] >= 128
        assert info["chunk_bytes"] >= info["chunk_rows"] * (2 * wl.V + 2 * wl.H)


def test_backward_chunks_are_whole_rounds_of_256_tiles_when_a_group_needs_several():
    # four tiles x 256 hidden columns per workgroup of the dz GEMM and 256 compute units: at H = 1024 a multiple of 256 tiles leaves no
    # partly filled last round
    for name in ("C3", "C4"):
        wl, desc, T, U = _lens(name)
        st, info, groups = Bd.rnnt_joint_loss_plan(desc, T, U, 0)
        assert st == 0
        cap = info["chunk_rows"] // 64
        assert cap >= 1024
        per = cap // 256 * 256
        tiles = _tiles(T, U)
        want = 0
        for g in range(info["n_groups"]):
            n = int(tiles[groups == g].sum())
            want += -(-n // per) if n > cap else 1
        assert info["n_chunks"] == want, name


def test_fp32_shapes_with_gemm_tiles_get_chunk_buffers():
    T = np.array([30, 17, 25], dtype=np.int32); U = np.array([7, 0, 11], dtype=np.int32)
    rows = int((T.astype(np.int64) * (U + 1)).sum())
    for H, V, gemm in [(128, 256, True), (256, 128, True), (96, 200, True), (128, 202, False), (60, 256, False)]:
        desc = Bd.make_desc(3, 30, 11, H, V, 0, Bd.RNNT_F32)
        st, info, _ = Bd.rnnt_joint_loss_plan(desc, T, U, 0)
        assert st == 0
        if gemm:
            # S [rows, V], Z and dZ [rows, H] in fp32, rows = the call's lattice nodes rounded up to 128
            assert info["chunk_rows"] == -(-rows // 128) * 128
            assert info["chunk_bytes"] >= info["chunk_rows"] * (4 * V + 8 * H)
            nmin = Bd.rnnt_joint_loss_workspace_bytes(desc, T, U, 1)
            st, small, groups = Bd.rnnt_joint_loss_plan(desc, T, U, nmin)
            assert st == 0 and small["chunk_rows"] == 128 and small["n_groups"] == 2
            # chunks are ranges of 128 lattice nodes of a group
            per_sample = T.astype(np.int64) * (U + 1)
            assert small["n_chunks"] == sum(-(-int(per_sample[groups == g].sum()) // 128) for g in range(2))
            assert info["n_chunks"] == info["n_groups"] == 1
        else:
            assert info["chunk_rows"] == 0 and info["chunk_bytes"] == 0


def test_workspace_does_not_grow_with_batch_size_once_capped():
    # memory "almost independent of batch size" (Section 5.2): doubling B leaves the default plan's size
    wl = synth.WORKLOADS["C4"]
    T, U, _ = synth.draw_lengths_labels(wl)
    d1 = Bd.make_desc(512, wl.T_max, wl.U_max, wl.H, wl.V, 0, Bd.RNNT_BF16)
    d2 = Bd.make_desc(1024, wl.T_max, wl.U_max, wl.H, wl.V, 0, Bd.RNNT_BF16)
    n1 = Bd.rnnt_joint_loss_workspace_bytes(d1, T[:512], U[:512], 0)
    n2 = Bd.rnnt_joint_loss_workspace_bytes(d2, T, U, 0)
    assert abs(n2 - n1) <= 8 * 1024 * 1024      # only the per-sample and per-tile index tables grow


def test_budgets_shrink_the_plan_and_a_too_small_budget_is_reported():
    wl, desc, T, U = _lens("C4")
    big = Bd.rnnt_joint_loss_workspace_bytes(desc, T, U, 0)
    small_budget = 96 << 20
    n = Bd.rnnt_joint_loss_workspace_bytes(desc, T, U, small_budget)
    assert 0 < n <= small_budget < big
    st, info, groups = Bd.rnnt_joint_loss_plan(desc, T, U, n)
    st0, info0, _ = Bd.rnnt_joint_loss_plan(desc, T, U, big)
    assert st == 0 and st0 == 0
    assert info["n_groups"] > info0["n_groups"] and info["n_chunks"] > info0["n_chunks"]
    rows = T.astype(np.int64) * (U.astype(np.int64) + 1)
    for g in range(info["n_groups"]):
        assert rows[groups == g].sum() <= info["group_rows_cap"]
    # the largest sample still fits: it is processed alone, the backward walks it in row chunks
    assert info["group_rows_cap"] >= rows.max()
    tiny = Bd.rnnt_joint_loss_workspace_bytes(desc, T, U, 1 << 20)
    assert tiny > (1 << 20)
    st, _, _ = Bd.rnnt_joint_loss_plan(desc, T, U, 1 << 20)
    assert st == 5
    st, info_min, _ = Bd.rnnt_joint_loss_plan(desc, T, U, tiny)
    assert st == 0 and info_min["chunk_rows"] == 128 and info_min["group_rows_cap"] == rows.max()


def test_keep_scores_plan_has_one_backward_chunk_per_group_of_whole_samples():
    wl, desc, T, U = _lens("C2")
    keep = Bd.make_desc(wl.B, wl.T_max, wl.U_max, wl.H, wl.V, 0, Bd.RNNT_BF16, keep_scores=1)
    st, info, groups = Bd.rnnt_joint_loss_plan(keep, T, U, 0)
    assert st == 0 and info["n_chunks"] == info["n_groups"] == 1 and (groups == 0).all()
    # the chunk buffers hold every tile row of the call: dH, Z and the running maxima
    per_row = 2 * (wl.V + 64) + 2 * (wl.H + 64) + 4 * (wl.V // 64)
    slack = 128 * 2 * (wl.V + 64) + 3 * 256          # dH ends on a multiple of 256 rows; alignment of the three
    assert info["chunk_rows"] * per_row <= info["chunk_bytes"] < info["chunk_rows"] * per_row + slack
    assert info["chunk_rows"] >= info["tiles_total"] * 64
    # smallest plan: the chunk buffers still hold the largest sample, one sample or more per group
    nmin = Bd.rnnt_joint_loss_workspace_bytes(keep, T, U, 1)
    st, small, groups = Bd.rnnt_joint_loss_plan(keep, T, U, nmin)
    assert st == 0 and small["n_chunks"] == small["n_groups"] > 1
    tiles = _tiles(T, U)
    assert small["chunk_rows"] >= int(tiles.max()) * 64
    for g in range(small["n_groups"]):
        assert int(tiles[groups == g].sum()) * 64 <= small["chunk_rows"]
    assert np.all(np.diff(groups) >= 0)
    st, _, _ = Bd.rnnt_joint_loss_plan(keep, T, U, nmin - 256)
    assert st == 5
    # a budget in between gives groups in between
    st, mid, _ = Bd.rnnt_joint_loss_plan(keep, T, U, (nmin + info["workspace_bytes"]) // 2)
    assert st == 0 and 1 <= mid["n_groups"] < small["n_groups"] and mid["workspace_bytes"] <= (nmin + info["workspace_bytes"]) // 2
    # only the bf16 path has the mode, and the flag is 0 or 1
    assert Bd.rnnt_joint_loss_workspace_bytes(Bd.make_desc(2, 8, 3, 16, 8, 0, Bd.RNNT_F32, keep_scores=1), [8, 8], [3, 3]) == 0
    assert Bd.rnnt_joint_loss_workspace_bytes(
        Bd.make_desc(wl.B, wl.T_max, wl.U_max, wl.H, wl.V, 0, Bd.RNNT_BF16, keep_scores=2), T, U) == 0


def test_bf16_input_gradients_add_a_bounded_staging_area_and_cap_the_group_size():
    wl, desc, T, U = _lens("C4")
    half = Bd.make_desc(wl.B, wl.T_max, wl.U_max, wl.H, wl.V, 0, Bd.RNNT_BF16, input_grads_bf16=1)
    n0 = Bd.rnnt_joint_loss_workspace_bytes(desc, T, U, 0)
    n1 = Bd.rnnt_joint_loss_workspace_bytes(half, T, U, 0)
    per_sample = (wl.T_max + wl.U_max + 1) * wl.H * 4
    cap = (256 << 20) // per_sample
    assert 0 < n1 - n0 <= (256 << 20) + 512 and n1 - n0 >= cap * per_sample
    st, info, groups = Bd.rnnt_joint_loss_plan(half, T, U, n1)
    assert st == 0 and np.bincount(groups).max() <= cap
    # the outputs shrink by more than the workspace grows
    assert (n1 - n0) < wl.B * per_sample // 2
    # smallest plan: one sample per group
    nmin = Bd.rnnt_joint_loss_workspace_bytes(half, T[:8], U[:8], 1)
    h8 = Bd.make_desc(8, wl.T_max, wl.U_max, wl.H, wl.V, 0, Bd.RNNT_BF16, input_grads_bf16=1)
    nmin = Bd.rnnt_joint_loss_workspace_bytes(h8, T[:8], U[:8], 1)
    st, info, groups = Bd.rnnt_joint_loss_plan(h8, T[:8], U[:8], nmin)
    assert st == 0 and info["n_groups"] == 8
    # bf16 only; not for the projected entry point, whose d_enc / d_pred are internal
    assert Bd.rnnt_joint_loss_workspace_bytes(Bd.make_desc(2, 8, 3, 16, 8, 0, Bd.RNNT_F32, input_grads_bf16=1), [8, 8], [3, 3]) == 0
    assert Bd.rnnt_joint_proj_workspace_bytes(half, 512, 512, T, U, 0) == 0


def test_random_plans_keep_their_promises():
    # seeded random shapes, lengths, options and budgets: every sample is in exactly one group, groups are runs of
    # consecutive samples, a plan never exceeds the workspace it was made for, the size the library asks for is
    # accepted, and the options' extra limits hold (kept scores: a group's tile rows fit the chunk buffers;
    # bfloat16 input gradients: groups no larger than the staging area was sized for)
    rng = np.random.default_rng(20240)
    for case in range(150):
        bf16 = bool(rng.integers(0, 4))
        B = int(rng.integers(1, 40))
        T_max, U_max = int(rng.integers(1, 300)), int(rng.integers(0, 120))
        if bf16:
            H, V = int(rng.choice([128, 256, 512, 640, 768, 1024])), int(rng.choice([256, 512, 1024, 4096]))
            opts = dict(keep_scores=int(rng.integers(0, 2)), input_grads_bf16=int(rng.integers(0, 2)))
        else:
            H, V, opts = int(rng.integers(1, 200)), int(rng.integers(2, 300)), {}
        T = rng.integers(1, T_max + 1, size=B).astype(np.int32)
        U = rng.integers(0, U_max + 1, size=B).astype(np.int32)
        desc = Bd.make_desc(B, T_max, U_max, H, V, 0, Bd.RNNT_BF16 if bf16 else Bd.RNNT_F32, **opts)
        n_default = Bd.rnnt_joint_loss_workspace_bytes(desc, T, U, 0)
        n_min = Bd.rnnt_joint_loss_workspace_bytes(desc, T, U, 1)
        assert 0 < n_min <= n_default, (case, n_min, n_default)
        tiles = _tiles(T, U)
        rows = T.astype(np.int64) * (U + 1)
        for budget in (n_default, n_min, int(rng.integers(n_min, n_default + 1)), n_default + int(rng.integers(1, 1 << 24))):
            st, info, groups = Bd.rnnt_joint_loss_plan(desc, T, U, budget)
            what = (case, opts, budget, info)
            assert st == 0, what
            assert info["workspace_bytes"] <= budget, what
            assert groups.min() == 0 and np.all(np.diff(groups) >= 0) and np.all(np.diff(groups) <= 1), what
            assert groups.max() + 1 == info["n_groups"] and info["n_chunks"] >= info["n_groups"], what
            assert info["rows_total"] == rows.sum() and info["tiles_total"] == tiles.sum(), what
            for g in range(info["n_groups"]):
                m = groups == g
                assert rows[m].sum() <= info["group_rows_cap"] or m.sum() == 1, what
                if opts.get("keep_scores"):
                    assert tiles[m].sum() * 64 <= info["chunk_rows"], what
            if opts.get("keep_scores"):
                assert info["n_chunks"] == info["n_groups"], what
            if bf16:
                assert info["chunk_rows"] % 128 == 0 and info["chunk_rows"] >= 128, what
        assert Bd.rnnt_joint_loss_plan(desc, T, U, n_min - 256)[0] == 5, case


def test_tile_shape_per_sample():
    # 8 x 8 tiles, or 16 x 4 where that covers the lattice with at least 3 % fewer tiles
    desc = Bd.make_desc(5, 40, 20, 128, 256, 0, Bd.RNNT_BF16)
    T = np.array([16, 8, 32, 40, 33], dtype=np.int32)
    U = np.array([3, 7, 11, 20, 8], dtype=np.int32)
    st, info, _ = Bd.rnnt_joint_loss_plan(desc, T, U, 0)
    # 16 x 4: 1 (against 2); 8 x 8: 1; 16 x 4: 2 * 3 = 6 (against 4 * 2 = 8); 8 x 8: 5 * 3 = 15 (16 x 4: 3 * 6 = 18);
    # 33 x 9: 8 x 8 gives 5 * 2 = 10, 16 x 4 gives 3 * 3 = 9
    assert st == 0 and info["tiles_total"] == 1 + 1 + 6 + 15 + 9
    assert info["tiles_total"] == int(_tiles(T, U).sum())


def test_projected_entry_point_checks_and_workspace():
    wl, desc, T, U = _lens("C2")
    L = Bd.lib()
    dummy = ctypes.c_void_p(0x1000)
    Tl, Ul = np.ascontiguousarray(T, dtype=np.int32), np.ascontiguousarray(U, dtype=np.int32)

    def call(H_A, H_L, hA=dummy, ws_bytes=1 << 32, d=desc):
        return L.rnnt_joint_proj_loss_fwd_bwd(ctypes.byref(d), H_A, H_L, hA, dummy, dummy, dummy, dummy, dummy, dummy,
                                              dummy, Bd._ip(Tl), Bd._ip(Ul), *([dummy] * 8), dummy, ws_bytes, None)

    assert call(512, 512, hA=None) == 1                # RNNT_ERR_NULL
    assert call(0, 512) == 2                           # RNNT_ERR_SHAPE
    assert call(200, 512) == 6                         # bf16 needs multiples of 128
    assert call(8192, 512) == 6
    inner = Bd.rnnt_joint_loss_workspace_bytes(desc, T, U, 0)
    n = Bd.rnnt_joint_proj_workspace_bytes(desc, 512, 256, T, U, 0)
    # in front of the inner workspace: enc, pred in the input dtype and d_enc, d_pred in fp32
    rows_a, rows_l = wl.B * wl.T_max, wl.B * (wl.U_max + 1)
    extra = (rows_a + rows_l) * wl.H * (2 + 4)
    assert inner + extra <= n <= inner + extra + 4 * 256
    assert call(512, 256, ws_bytes=extra) == 5         # RNNT_ERR_WORKSPACE: nothing left for the inner path
    assert call(512, 256, ws_bytes=extra + 4096) == 5  # less than the smallest inner plan
    assert Bd.rnnt_joint_proj_workspace_bytes(desc, 100, 256, T, U, 0) == 0


def test_group_of_samples_never_exceeds_32_bit_lattice_indices():
    # 4096 samples of 1000 x 1024 nodes are 4.2e9 lattice nodes; with a workspace that could hold them all the
    # planner still cuts groups below 2^31 nodes (the kernels index a group's lattice state with 32-bit integers)
    B = 4096
    desc = Bd.make_desc(B, 1000, 1023, 512, 1024, 0, Bd.RNNT_BF16)
    T, U = np.full(B, 1000, dtype=np.int32), np.full(B, 1023, dtype=np.int32)
    st, info, groups = Bd.rnnt_joint_loss_plan(desc, T, U, 200 << 30)
    assert st == 0 and info["rows_total"] == B * 1000 * 1024 > 2 ** 31
    assert info["group_rows_cap"] <= 2 ** 31 - 1 and info["n_groups"] >= 2
    counts = np.bincount(groups)
    assert counts.max() * 1000 * 1024 <= 2 ** 31 - 1


def test_plan_handle_holds_the_schedule_of_the_plan_query():
    # no GPU needed: the handle falls back to ordinary host memory for its tables
    wl = synth.WORKLOADS["C4"]
    T, U, _ = synth.draw_lengths_labels(wl)
    desc = Bd.make_desc(wl.B, wl.T_max, wl.U_max, wl.H, wl.V, 0, Bd.RNNT_BF16)
    st, info, _ = Bd.rnnt_joint_loss_plan(desc, T, U, 0)
    assert st == 0
    h = Bd.PlanHandle(desc, T, U)
    assert h.workspace_bytes == info["workspace_bytes"] == Bd.rnnt_joint_loss_workspace_bytes(desc, T, U, 0)
    assert h.describe() == info
    h.close()
    # room for the lattice state of two groups: each group at most half as large, same lattice bytes
    h2 = Bd.PlanHandle(desc, T, U, overlap_lattice=True)
    d2 = h2.describe()
    assert d2["lattice_bytes"] <= info["lattice_bytes"] + 4096
    assert d2["group_rows_cap"] * 2 <= info["group_rows_cap"] + 2
    assert d2["n_groups"] >= 2 * info["n_groups"] - 1 and d2["rows_total"] == info["rows_total"]
    h2.close()
    # bad arguments are refused when the handle is made
    bad = Bd.make_desc(wl.B, wl.T_max, wl.U_max, 500, wl.V, 0, Bd.RNNT_BF16)
    with pytest.raises(Bd.RnntError):
        Bd.PlanHandle(bad, T, U)
    with pytest.raises(Bd.RnntError):
        Bd.PlanHandle(desc, T + 1000, U)
    assert Bd.lib().rnnt_plan_workspace_bytes(None) == 0
    Bd.lib().rnnt_plan_destroy(None)


def _smallest_workspace_promised(T, U, H, V, keep, g16, T_max, U_max):
    """What the smallest bf16 workspace may take: the tables, one packed copy of W_out and up to H = 640 a second one, slots of the
    dW GEMM for about one 256 x 256 tile per compute unit in whole eighths, the largest sample's lattice state, one chunk."""
    al = lambda n, a=256: -(-n // a) * a
    B, tiles = len(T), _tiles(T, U)
    rows = (T.astype(np.int64) * (U + 1)).max()
    chunk = al(int(tiles.max()) * 64, 128) if keep else 128
    dw = -(-H // 256) * (V // 256)
    splits = al(-(-256 // dw), 8)
    n = 6 * al(4 * B) + al(4 * (B + 1)) + al(8 * (B + 1)) + 2 * al(4 * int(tiles.sum())) + (2 if H <= 640 else 1) * al(2 * H * V)
    n += dw * splits * (1 << 18) + 5 * al(4 * int(rows)) + al(al(chunk) * 2 * (V + 64)) + al(chunk * 2 * (H + 64))
    n += al(chunk * (V // 64) * 4) if keep else 0
    return n + (al(4 * T_max * H) + al(4 * (U_max + 1) * H) if g16 else 0)


@pytest.mark.parametrize("H", [128, 256, 512, 640, 768, 896, 1024])
@pytest.mark.parametrize("V", [256, 1024, 4096, 8192])
def test_smallest_workspace_keeps_its_bound(H, V):
    g = np.random.default_rng(H + V)
    for T_max, U_max, B in ((1, 0, 1), (40, 9, 3), (700, 120, 1), (3000, 300, 2)):
        T, U = g.integers(1, T_max + 1, B).astype(np.int32), g.integers(0, U_max + 1, B).astype(np.int32)
        for keep, g16 in ((0, 0), (1, 0), (0, 1)):
            desc = Bd.make_desc(B, T_max, U_max, H, V, 0, Bd.RNNT_BF16, keep_scores=keep, input_grads_bf16=g16)
            need = Bd.rnnt_joint_loss_workspace_bytes(desc, T, U, 1)
            assert need <= _smallest_workspace_promised(T, U, H, V, keep, g16, T_max, U_max), (T_max, U_max, keep, g16)
            st, info, _ = Bd.rnnt_joint_loss_plan(desc, T, U, need)
            assert st == 0 and info["workspace_bytes"] <= need


def test_long_samples_that_just_fit_the_static_workspace():
    # 128 MiB, the largest sample for which the bound above holds: 20 bytes per lattice node beside tables, weights and slots
    for H, V in ((768, 256), (896, 512), (1024, 1024), (1024, 256)):
        U = 1000
        fits = lambda t: _smallest_workspace_promised(np.array([t]), np.array([U]), H, V, 0, 0, t, U) <= 128 << 20
        T = max(t for t in range(1000, 5000) if fits(t))
        assert not fits(T + 1)
        desc = Bd.make_desc(1, T, U, H, V, 0, Bd.RNNT_BF16)
        st, _, _ = Bd.rnnt_joint_loss_plan(desc, np.array([T], np.int32), np.array([U], np.int32), 128 << 20)
        assert st == 0, (H, V, T)


def test_end_of_one_grid_of_two_kinds_of_workgroups_against_a_schedule(tmp_path):
    # the closed form that chooses the splits of the two backward GEMMs, against placing every workgroup on the first free unit
    import shutil
    import subprocess
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host compiler")
    src = tmp_path / "end.cpp"
    src.write_text('#include "%s"\n' % os.path.join(ROOT, "paper_2211_16270_amd", "csrc", "plan.h") + """
#include <cstdio>
#include <functional>
#include <queue>
#include <random>
int main() {
    std::mt19937 g(7);
    int bad = 0;
    for (int i = 0; i < 4000; ++i) {
        const long long nw = 1 + g() % 700, n = 1 + g() % 1500;
        const double cw = 1 + g() % 60 + 0.25 * (g() % 4), c = 1 + g() % 60 + 0.5 * (g() % 2);
        std::priority_queue<double, std::vector<double>, std::greater<double>> unit;
        for (int u = 0; u < 256; ++u) unit.push(0.0);
        double end = 0.0;
        for (long long j = 0; j < nw + n; ++j) {
            const double t = unit.top() + (j < nw ? cw : c);
            unit.pop();
            unit.push(t);
            end = std::max(end, t);
        }
        if (std::abs(end - rnnt::one_grid_end(nw, cw, n, c)) > 1e-6) ++bad;
    }
    std::printf("%d\\n", bad);
}
""")
    subprocess.run([gxx, "-O1", "-std=c++17", "-o", str(tmp_path / "end"), str(src)], check=True)
    assert subprocess.run([str(tmp_path / "end")], check=True, capture_output=True, text=True).stdout.strip() == "0"


def test_counter_summaries_name_kernels_the_library_has():
    # bench.py looks bytes per launch up by kernel name: a summary may not outlive the kernels it was taken with
    import glob
    have = {Bd.rnnt_profile_kernel_name(i) for i in range(Bd.rnnt_profile_kernel_count())}
    files = glob.glob(os.path.join(ROOT, "profiles", "hbm_traffic_*.txt"))
    assert files
    for f in files:
        names = {line.split()[0] for line in open(f) if line.strip() and not line.startswith("#")}
        assert names and names <= have, (os.path.basename(f), names - have)


def test_parts_of_the_vocabulary_are_runs_of_whole_segments(tmp_path):
    # every vocabulary the score kernels take, every number of parts the rule may choose: the parts follow each other, cover the vocabulary, hold
    # whole segments (statistics) or pairs of blocks, and where scores are kept a multiple of four blocks
    import shutil
    import subprocess
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host compiler")
    src = tmp_path / "parts.cpp"
    src.write_text('#include "%s"\n' % os.path.join(ROOT, "paper_2211_16270_amd", "csrc", "plan.h") + """
#include <cstdio>
int main() {
    int bad = 0, most = 0;
    for (int V = 256; V <= 16384; V += 256)
        for (int statistics = 0; statistics < 2; ++statistics)
            for (int multiple = 2; multiple <= (statistics ? 4 : 2); multiple += 2)
                for (int slots = 256; slots <= 512; slots += 256)
                    for (int n = 1; n <= 520; ++n) {
                        const int p = rnnt::score_split(n, slots, V, statistics, multiple).parts, seg = V / 32 / rnnt::score_segments(V);
                        most = std::max(most, p);
                        if (seg % 2) ++bad;
                        if (rnnt::score_part_begin(0, p, V, statistics) != 0 || rnnt::score_part_begin(p, p, V, statistics) != V / 32) ++bad;
                        for (int y = 0; y < p; ++y) {
                            const int b = rnnt::score_part_begin(y, p, V, statistics), e = rnnt::score_part_begin(y + 1, p, V, statistics);
                            if (e <= b || (e - b) % multiple || (statistics && b % seg)) ++bad;
                        }
                    }
    std::printf("%d %d\\n", bad, most);
}
""")
    exe = tmp_path / "parts"
    subprocess.run([gxx, "-std=c++17", "-O1", "-o", str(exe), str(src)], check=True, capture_output=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout
    assert out.split() == ["0", "8"]


def test_numbers_of_the_fp64_sweep_keep_64_bits(tmp_path):
    # the sweep's exponentials and logarithm against 80-bit arithmetic, with h = 2^-53 (a rounding).  An emission: log2 e and the product with it, h |x| each;
    # the polynomial, 2.8 h and 1.5 h for its last steps: h (2 |x| + 4.5).  The logarithm: a sum, ln 2 and the last step, h |x| each; sqrt 2 twice, the
    # polynomial and a step, 7.5 h.  1200 equal emissions, whose errors all have one sign: an emission and a product each.
    import shutil
    import subprocess
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host compiler")
    src = tmp_path / "scaled.cpp"
    src.write_text('#include "%s"\n' % os.path.join(ROOT, "paper_2211_16270_amd", "csrc", "scaled.h") + """
#include <cstdio>
using namespace rnnt;
int main() {
    const double eps = 1.1102230246251565e-16;
    double one = 0, log_ = 0, chain = 0, sum = 0;
    for (int i = -40000; i <= 4000; ++i) {
        const double x = i * 1.0009765625e-3;
        const Scaled e = scaled_exp(x);
        one = std::max(one, (double)(std::abs(logl((long double)e.m) + (long double)e.k * logl(2.0L) - x) / (eps * (4.5 + 2 * std::abs(x)))));
        const double v = scaled_log(e);
        log_ = std::max(log_, (double)(std::abs(logl((long double)e.m) + (long double)e.k * logl(2.0L) - v) / (eps * (7.5 + 3 * std::abs(x)))));
    }
    for (int i = 0; i < 400; ++i) {
        const double x = -8 + 0.0203125 * i;
        Scaled v{1.0, 0.0};
        const Scaled e = scaled_exp(x);
        for (int n = 1; n <= 1200; ++n) {
            v = times(v, e);
            if (n % 8 == 0) { int up; const double m = mantissa(v.m, up); v = Scaled{m, v.k + up}; }
        }
        chain = std::max(chain, (double)(std::abs((long double)scaled_log(v) - 1200.0L * x) / (eps * (1200 * (5.5 + 2 * std::abs(x)) + 7.5 + 3 * 1200 * std::abs(x)))));
        const Scaled a = scaled_exp(x), b = scaled_exp(-3.0 - 0.31 * x);
        const long double want = logl(expl((long double)x) + expl((long double)(-3.0 - 0.31 * x)));
        sum = std::max(sum, (double)(std::abs((long double)scaled_log(plus(a, b)) - want) / (eps * (4.5 + 2 * std::abs(x) + 7.5 + 3 * std::abs(x) + 4.5 + 2 * std::abs(-3.0 - 0.31 * x)))));
    }
    const Scaled floor_ = scaled_exp(-1e30), none{1.0, -1e280};
    const bool edge = floor_.m == 1.0 && scaled_log(plus(floor_, none)) == scaled_log(floor_) && scaled_log(plus(scaled_exp(-700.0), floor_)) + 700 < 1e-12;
    std::printf("%d %d %d %d %d\\n", one <= 1, log_ <= 1, chain <= 1, sum <= 1, edge);
    std::fprintf(stderr, "%g %g %g %g\\n", one, log_, chain, sum);
}
""".replace("\\\\n", "\\n"))
    exe = tmp_path / "scaled"
    subprocess.run([gxx, "-std=c++17", "-O1", "-ffp-contract=off", "-Wno-unknown-pragmas", "-o", str(exe), str(src)], check=True, capture_output=True)
    run = subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60)
    assert run.stdout.split() == ["1"] * 5, run.stderr


def _f32_chunk_counts(T_len, U_len, groups, chunk_rows):
    """chunks of whole samples (one that takes several: of equal size), full chunks wherever samples end"""
    rows = T_len.astype(np.int64) * (U_len + 1)
    up = lambda x, k: -(-int(x) // k)
    samples = nodes = 0
    for g in np.unique(groups):
        r = rows[groups == g]
        nodes += up(r.sum(), chunk_rows)
        s = 0
        while s < len(r):
            e = s + 1
            while e < len(r) and r[s:e + 1].sum() <= chunk_rows:
                e += 1
            n = r[s:e].sum()
            samples += up(n, up(up(n, up(n, chunk_rows)), 128) * 128)
            s = e
    return samples, nodes


@pytest.mark.parametrize("B,T,U,H,V,parts", [
    # (part of the default workspace, whole samples) where both orders were timed, ms: (1, 7.3 : 9.1), (4, 11.0 : 10.7), (16, 24.6 : 14.4)
    (64, 500, 100, 64, 64, ((1, True), (4, False), (16, False))),
    # (1, 18.1 : 21.8), (4, 34.5 : 26.0), (16, 55.8 : 41.9)
    (64, 500, 100, 256, 256, ((1, True), (4, False), (16, False))),
    # (1, 33.3 : 37.9), (4, 55.7 : 46.6), (16, 88.9 : 82.3)
    (64, 500, 100, 128, 1024, ((1, True), (4, False), (16, False))),
    # (1, 100.0 : 119.6), (4, 175.9 : 117.2)
    (200, 1000, 200, 64, 64, ((1, True), (4, False))),
    # (4, 13.6 : 15.4), (16, 31.3 : 24.5)
    (64, 200, 40, 512, 1024, ((4, True), (16, False))),
    # (1, 99.6 : 127.1)
    (16, 500, 100, 1024, 4096, ((1, True),)),
])
def test_f32_samples_are_swept_with_their_chunk_only_where_that_is_faster(B, T, U, H, V, parts):
    g = np.random.default_rng([2211, B, T, U])
    T_len, U_len = g.integers(int(.9 * T), T + 1, size=B).astype(np.int32), g.integers(int(.9 * U), U + 1, size=B).astype(np.int32)
    desc = Bd.make_desc(B, T, U, H, V, 0, Bd.RNNT_F32)
    full = Bd.rnnt_joint_loss_workspace_bytes(desc, T_len, U_len)
    for part, whole in parts:
        n = Bd.rnnt_joint_loss_workspace_bytes(desc, T_len, U_len, full // part)
        st, info, groups = Bd.rnnt_joint_loss_plan(desc, T_len, U_len, n)
        samples, nodes = _f32_chunk_counts(T_len, U_len, groups, info["chunk_rows"])
        assert st == 0 and info["n_chunks"] == (samples if whole else nodes), (part, info, samples, nodes)


def test_f32_chunks_cover_their_group_in_either_order(tmp_path):
    # random batches and chunk sizes: every node of a group in one chunk, in order; what is swept together covers the group, too; the tiles of a chunk hold
    # all of its nodes, and the first and the last of them some
    import shutil
    import subprocess
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host compiler")
    src = tmp_path / "chunks.cpp"
    src.write_text('#include "%s"\n' % os.path.join(ROOT, "paper_2211_16270_amd", "csrc", "plan.cpp") + """
#include <cstdio>
#include <random>
using namespace rnnt;
int main() {
    std::mt19937 g(11);
    int bad = 0, several = 0, whole = 0, losses = 0;
    for (int i = 0; i < 3000; ++i) {
        const int B = 1 + g() % 9, T = 1 + g() % 90, U = g() % 40, H = 64 << (g() % 5), V = 64 << (g() % 7);
        std::vector<int32_t> Tl(B), Ul(B);
        for (int b = 0; b < B; ++b) { Tl[b] = 1 + g() % T; Ul[b] = g() % (U + 1); }
        rnnt_desc d{};
        d.B = B; d.T_max = T; d.U_max = U; d.H = H; d.V = V; d.dtype = RNNT_F32;
        Plan p;
        build_plan(d, Tl.data(), Ul.data(), 1, p);
        const size_t given = p.min_bytes + g() % (1 << (14 + g() % 12));
        build_plan(d, Tl.data(), Ul.data(), given, p);
        Plan l;
        build_plan(d, Tl.data(), Ul.data(), given, l, false, false);
        Plan two;                                     // sweeps on a stream of their own: full chunks
        build_plan(d, Tl.data(), Ul.data(), given + (1 << 20), two, true);
        size_t full = 0;
        for (int gi = 0; gi < (int)two.groups.size(); ++gi) {
            const std::vector<Chunk> nodes = F32Chunks{d, Tl.data(), Ul.data(), two, gi, two.chunk_rows}.of_nodes();
            for (size_t k = 0; k < nodes.size(); ++k, ++full)
                if (full >= two.group_chunks.size() || two.group_chunks[full].row0 != nodes[k].row0 || two.group_chunks[full].group != gi) ++bad;
        }
        if (full != two.group_chunks.size() || !p.group_chunks.empty()) ++bad;
        for (int gi = 0; gi < (int)p.groups.size(); ++gi) {
            const Group& gr = p.groups[gi];
            const F32Chunks f{d, Tl.data(), Ul.data(), p, gi, p.chunk_rows};
            std::vector<Chunk> taken, taken_l;
            for (const Chunk& c : p.chunks) if (c.group == gi) taken.push_back(c);
            for (const Chunk& c : l.chunks) if (c.group == gi) taken_l.push_back(c);
            const std::vector<Chunk> samples = f.of_samples(), nodes = f.of_nodes();
            const bool s = f.cost(samples) <= f.cost(nodes);
            const std::vector<Chunk>& want = s ? samples : nodes;
            if (taken.size() != want.size() || taken[0].s1 != want[0].s1) ++bad;
            if (taken_l.size() != nodes.size()) ++losses;
            if (samples.size() > 1) ++(s ? whole : several);
            for (const std::vector<Chunk>& cs : {samples, nodes}) {
                long long at = 0;
                int swept = gr.s0;
                for (size_t k = 0; k < cs.size(); ++k) {
                    const Chunk& c = cs[k];
                    if (c.row0 != at || c.rows < 1 || c.rows > p.chunk_rows || c.s0 != swept) ++bad;
                    if (k + 1 < cs.size() ? cs[k + 1].s0 != c.s0 : true) swept = c.s1;
                    at += c.rows;
                    int lo = 1 << 30, hi = -1;
                    for (int s2 = c.s0; s2 < c.s1; ++s2) {
                        const int W = Ul[s2] + 1, uw = tile_label_width(Tl[s2], Ul[s2]), th = 64 / uw, across = (W + uw - 1) / uw;
                        for (long long r = 0; r < (long long)Tl[s2] * W; ++r) {
                            const long long n = p.row_off[s2] - p.row_off[gr.s0] + r;
                            if (n < c.row0 || n >= c.row0 + c.rows) continue;
                            const int tile = p.tile_off[s2] + (int)(r / W) / th * across + (int)(r % W) / uw;
                            lo = std::min(lo, tile); hi = std::max(hi, tile);
                        }
                    }
                    if (lo < c.tile0 || hi >= c.tile1 || c.tile0 < gr.tile0 || c.tile1 > gr.tile1) ++bad;
                }
                if (at != gr.rows || swept != gr.s1) ++bad;
            }
        }
    }
    std::printf("%d %d %d %d\\n", bad, losses, several > 100, whole > 100);
}
""")
    exe = tmp_path / "chunks"
    subprocess.run([gxx, "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-w", "-o", str(exe), str(src)], check=True,
                   capture_output=True)
    assert subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=100).stdout.split() == ["0", "0", "1", "1"]


def test_vocabulary_parts_as_the_gpu_tests_expect_them(tmp_path):
    # the rule as the tests of the score kernels repeat it, to name the parts they run
    import shutil
    import subprocess
    from tests.test_gpu_parity import _vocabulary_parts
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host compiler")
    src = tmp_path / "rule.cpp"
    src.write_text('#include "%s"\n' % os.path.join(ROOT, "paper_2211_16270_amd", "csrc", "plan.h") + """
#include <cstdio>
int main() {
    for (int V : {256, 768, 2048, 2304, 4096, 8192})
        for (int n = 1; n <= 300; ++n)
            for (int slots : {256, 512})
                std::printf("%d %d %d\\n", rnnt::score_split(n, slots, V, true).parts, rnnt::score_split(n, slots, V, false).parts,
                            rnnt::score_split(n, slots, V, true, 4).parts);
}
""")
    exe = tmp_path / "rule"
    subprocess.run([gxx, "-std=c++17", "-O1", "-o", str(exe), str(src)], check=True, capture_output=True)
    out = [tuple(map(int, l.split())) for l in subprocess.run([str(exe)], check=True, capture_output=True, text=True, timeout=60).stdout.splitlines()]
    assert out == [(_vocabulary_parts(V, 2 * n, True, slots=slots), _vocabulary_parts(V, 2 * n, False, slots=slots),
                    _vocabulary_parts(V, 2 * n, True, 4, slots)) for V in (256, 768, 2048, 2304, 4096, 8192) for n in range(1, 301)
                   for slots in (256, 512)]
