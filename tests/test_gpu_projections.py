"""GPU parity of the path with the joint network's input projections inside (Eq. 4 complete,
Algorithm 1 line 9), through the C ABI, against the float64 checker."""
import numpy as np
import pytest

from oracle import rnnt_oracle as O
from paper_2211_16270_amd import binding as Bd
from paper_2211_16270_amd import synth
from tests.gpu_util import TOL, rel_grad_err, rel_loss_err

pytestmark = pytest.mark.gpu

PGRADS = ("d_hA", "d_hL", "dW_A", "db_Z", "dW_L", "dW_out", "db_out")


def _say(*a):
    print(*a, flush=True)


def run_gpu_proj(batch, proj, budget_bytes=0, accumulate_into=None, keep_scores=0):
    import torch
    wl = batch.wl
    dev = Bd.to_device(batch)
    devp = Bd.proj_to_device(proj, wl.dtype)
    dt = Bd.RNNT_BF16 if wl.dtype == "bf16" else Bd.RNNT_F32
    out = Bd.run_proj_fwd_bwd(dev, devp, batch.B, wl.T_max, wl.U_max, wl.H, wl.V, wl.blank, dt,
                              budget_bytes=budget_bytes, accumulate_into=accumulate_into, keep_scores=keep_scores)
    torch.cuda.synchronize()
    return {k: out[k].float().cpu().numpy() for k in ("loss",) + PGRADS}


def run_oracle_proj(batch, proj):
    f = lambda x: np.asarray(x, dtype=np.float64)
    return O.rnnt_joint_proj_loss(f(proj.hA), f(proj.hL), f(proj.W_A), f(proj.b_Z), f(proj.W_L), f(batch.W_out),
                                  f(batch.b_out), batch.labels, batch.T_len, batch.U_len, batch.wl.blank)


def check(got, ref, dtype, batch, what):
    tol = TOL[dtype]
    el = rel_loss_err(got["loss"].astype(np.float64), ref["loss"])
    errs = {k: rel_grad_err(got[k].astype(np.float64), ref[k]) for k in PGRADS}
    _say(what, "loss", el, {k: float("%.2e" % v) for k, v in errs.items()})
    assert np.all(np.isfinite(got["loss"])) and el <= tol["loss"], (what, el)
    for k in PGRADS:
        assert np.all(np.isfinite(got[k])), (what, k)
        assert errs[k] <= tol["grad"], (what, k, errs[k])
    for b in range(batch.B):
        assert np.all(got["d_hA"][b, batch.T_len[b]:] == 0.0)
        assert np.all(got["d_hL"][b, batch.U_len[b] + 1:] == 0.0)


def test_f32_projected_path_ragged_lengths():
    wl = synth.custom_workload("pf32", B=3, T_max=9, U_max=4, H=24, V=11, dtype="f32", index=131,
                               t_rule="uniform", t_lo=1, u_rule="uniform", u_lo=0)
    batch = synth.make_batch(wl)
    proj = synth.make_proj_inputs(batch, H_A=20, H_L=12)
    check(run_gpu_proj(batch, proj), run_oracle_proj(batch, proj), "f32", batch, "f32 ragged")


@pytest.mark.parametrize("H,V,H_A,H_L", [(256, 128, 132, 200), (24, 11, 10, 7), (128, 256, 516, 4)])
def test_f32_projected_path_tile_gemms_with_edges_and_the_fallback(H, V, H_A, H_L):
    # widths that are multiples of 4 run the projections as tile GEMMs (ragged tiles, masked padded rows),
    # others as one thread per output element; (256, 128) and (128, 256) also take the GEMM form of the joint path
    wl = synth.custom_workload("pf32b", B=4, T_max=37, U_max=11, H=H, V=V, dtype="f32", index=133,
                               t_rule="uniform", t_lo=5, u_rule="uniform", u_lo=0)
    batch = synth.make_batch(wl)
    proj = synth.make_proj_inputs(batch, H_A=H_A, H_L=H_L)
    check(run_gpu_proj(batch, proj), run_oracle_proj(batch, proj), "f32", batch, f"f32 {H},{V},{H_A},{H_L}")


@pytest.mark.parametrize("value", [np.inf, -np.inf, 3.4e38])
def test_f32_projected_path_with_an_encoding_beyond_the_largest_bf16(value):
    # the frame's activations are +-1; only the gradient of the weights that the infinite value meets has no value (inf times 0)
    wl = synth.custom_workload("pinf32", B=4, T_max=37, U_max=11, H=256, V=128, dtype="f32", index=133,
                               t_rule="uniform", t_lo=5, u_rule="uniform", u_lo=0)
    batch = synth.make_batch(wl)
    proj = synth.make_proj_inputs(batch, H_A=132, H_L=200)
    proj.hA[1, 2, 5] = value
    if np.isfinite(value):
        proj.W_A[5] = np.copysign(0.9, proj.W_A[5])       # (no product overflows)
    with np.errstate(all="ignore"):
        got, ref = run_gpu_proj(batch, proj), run_oracle_proj(batch, proj)
    if np.isinf(value):
        assert np.all(np.isnan(got["dW_A"][5])) and np.all(np.isnan(ref["dW_A"][5]))
        got["dW_A"][5] = ref["dW_A"][5] = 0.0
    check(got, ref, "f32", batch, f"encoding {value}")


def test_f32_identity_projection_equals_the_unprojected_entry_point():
    import torch
    batch = synth.make_batch("C1")
    wl = batch.wl
    fill = lambda x: np.nan_to_num(x, nan=0.0)
    proj = synth.ProjInputs(hA=batch.enc, hL=batch.pred, W_A=np.eye(wl.H, dtype=np.float32),
                            b_Z=np.zeros(wl.H, dtype=np.float32), W_L=np.eye(wl.H, dtype=np.float32))
    got = run_gpu_proj(batch, proj)
    dev = Bd.to_device(batch)
    base = Bd.run_fwd_bwd(dev, batch.B, wl.T_max, wl.U_max, wl.H, wl.V, wl.blank, Bd.RNNT_F32)
    torch.cuda.synchronize()
    np.testing.assert_allclose(got["loss"], base["loss"].cpu().numpy(), rtol=1e-6)
    np.testing.assert_allclose(got["d_hA"], base["d_enc"].cpu().numpy(), atol=1e-6)
    np.testing.assert_allclose(got["d_hL"], base["d_pred"].cpu().numpy(), atol=1e-6)
    np.testing.assert_allclose(got["db_Z"], fill(base["d_enc"].cpu().numpy()).sum(axis=(0, 1)), atol=1e-5)


@pytest.mark.parametrize("H_A,H_L", [(128, 128), (384, 256)])
def test_bf16_projected_path_small(H_A, H_L):
    wl = synth.custom_workload("pbf16", B=4, T_max=37, U_max=11, H=256, V=512, dtype="bf16", index=132,
                               t_rule="uniform", t_lo=5, u_rule="uniform", u_lo=0)
    batch = synth.make_batch(wl)
    proj = synth.make_proj_inputs(batch, H_A=H_A, H_L=H_L)
    ref = run_oracle_proj(batch, proj)
    check(run_gpu_proj(batch, proj), ref, "bf16", batch, f"bf16 small {H_A},{H_L}")
    check(run_gpu_proj(batch, proj, keep_scores=1), ref, "bf16", batch, f"bf16 small {H_A},{H_L}, kept scores")


def test_bf16_projected_path_bench_workload_subbatch_and_accumulate():
    import torch
    ids = [0, 7, 19]
    batch = synth.make_batch("C2", sample_ids=ids)
    proj = synth.make_proj_inputs(batch, H_A=512, H_L=512)
    ref = run_oracle_proj(batch, proj)
    got = run_gpu_proj(batch, proj)
    check(got, ref, "bf16", batch, "C2 sub-batch")
    # accumulate_params: a second call adds to all five parameter gradients
    wl = batch.wl
    acc = {k: torch.from_numpy(got[k].copy()).cuda() for k in ("dW_A", "db_Z", "dW_L", "dW_out", "db_out")}
    got2 = run_gpu_proj(batch, proj, accumulate_into=acc)
    for k in ("dW_A", "db_Z", "dW_L", "dW_out", "db_out"):
        e = rel_grad_err(got2[k].astype(np.float64), 2.0 * ref[k])
        assert e <= TOL["bf16"]["grad"], (k, e)


@pytest.mark.parametrize("B,T_max,U_max,H,H_A,H_L", [
    (1, 1, 0, 128, 128, 128),       # one row a side
    (2, 64, 127, 128, 128, 256),    # whole tiles and K-steps
    (37, 29, 6, 384, 256, 640),     # several splits of the rows, padded rows (NaN) among them and at the end of a split
    (3, 341, 2, 256, 128, 128),     # a split ends inside a K-step
])
def test_bf16_projections_at_the_edges_of_tiles_and_splits(B, T_max, U_max, H, H_A, H_L):
    wl = synth.custom_workload("pedge", B=B, T_max=T_max, U_max=U_max, H=H, V=256, dtype="bf16", index=134,
                               t_rule="uniform", t_lo=max(1, T_max // 2), u_rule="uniform", u_lo=U_max // 2)
    batch = synth.make_batch(wl)
    proj = synth.make_proj_inputs(batch, H_A=H_A, H_L=H_L)
    check(run_gpu_proj(batch, proj), run_oracle_proj(batch, proj), "bf16", batch, f"bf16 {B}x{T_max}x{U_max} {H},{H_A},{H_L}")


@pytest.mark.parametrize("one_sign", [False, True])
@pytest.mark.parametrize("B,D", [(64, 1024), (128, 512), (16, 128)])
def test_bf16_weight_gradients_of_many_rows_keep_their_precision(B, D, one_sign):
    # Identity maps: d_hA is d_enc as it goes into dW_A's product, and the entry point without projections gives d_enc itself for db_Z, so what is left is
    # the error of the sums alone.  n rows a split (the kernels' rule), S splits; a rounded addition is off by at most u = 2^-24 / sqrt(3) of the
    # sum so far (root mean square), which over terms of random sign leaves u sqrt(n / 32 + S / 2) of the result (16 rows an addition: the matrix
    # instruction's k, and the threads of a column of db_Z), over terms of one sign u sqrt(n / (48 S) + S / 3).
    import torch
    T, U, V, rows = 1000, 1, 256, B * 1000
    g = torch.Generator(device="cuda").manual_seed(3)
    normal = lambda *s, to=torch.bfloat16: torch.empty(*s, dtype=to, device="cuda").normal_(generator=g)
    out = lambda *s: torch.empty(*s, device="cuda")
    T_len, U_len = np.full(B, T, np.int32), np.full(B, U, np.int32)
    desc = Bd.make_desc(B, T, U, D, V, 0, Bd.RNNT_BF16)
    hA, hL, eye = normal(B, T, D), normal(B, U + 1, D), torch.eye(D, dtype=torch.bfloat16, device="cuda")
    if one_sign:
        hA = hA.abs()
    W, b = normal(D, V) * D ** -0.5, normal(V, to=torch.float32) * 0.1
    labels = torch.randint(1, V, (B, U), device="cuda", dtype=torch.int32, generator=g)
    loss, d_hA, d_hL, dW_A, db_Z, dW_L, dW, db = out(B), out(B, T, D), out(B, U + 1, D), out(D, D), out(D), out(D, D), out(D, V), out(V)
    _say("many rows", B, D, one_sign)
    ws = Bd.Workspace(Bd.rnnt_joint_proj_workspace_bytes(desc, D, D, T_len, U_len))
    assert Bd.rnnt_joint_proj_loss_fwd_bwd(desc, D, D, hA, hL, eye, torch.zeros(D, device="cuda"), eye, W, b, labels, T_len, U_len, loss,
                                           d_hA, d_hL, dW_A, db_Z, dW_L, dW, db, ws.buf) == 0
    d_enc, d_pred = out(B, T, D), out(B, U + 1, D)
    ws = Bd.Workspace(Bd.rnnt_joint_loss_workspace_bytes(desc, T_len, U_len))
    assert Bd.rnnt_joint_loss_fwd_bwd(desc, hA, hL, W, b, labels, T_len, U_len, loss, d_enc, d_pred, dW, db, ws.buf) == 0
    ref_W, ref_b = torch.zeros(D, D, dtype=torch.float64, device="cuda"), torch.zeros(D, dtype=torch.float64, device="cuda")
    for x, y, z in zip(hA.view(-1, D).split(16000), d_hA.view(-1, D).split(16000), d_enc.view(-1, D).split(16000)):
        ref_W += x.double().t().contiguous() @ y.double()
        ref_b += z.double().sum(0)
    fill, low, high = rows * (D // 128) ** 2 / 256, 4 * rows ** 0.5, 2 * rows ** (2 / 3)
    n = max(256, fill if fill ** 2 <= 2 * low ** 2 else max(low, min(fill / 2, high)))
    u, S = 2.0 ** -24 / 3 ** 0.5, -(-rows // n)
    err = lambda a, r: float((a.double() - r).norm() / r.norm())
    either, one = u * (n / 32 + S / 2) ** 0.5, u * (n / (48 * S) + S / 3) ** 0.5
    e_W, e_b = err(dW_A, ref_W), err(db_Z, ref_b)
    _say("many rows", D, rows, "dW_A", e_W, "db_Z", e_b, "bounds", either, one)
    assert e_W <= (one if one_sign else either) and e_b <= either
