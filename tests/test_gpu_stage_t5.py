"""GPU parity of the encoder-decoder (T5-style) stage against the per-sequence float64 oracle:
RMSNorm, gated-GELU MLP, bidirectional / causal / cross attention, two token streams, on a DP plan
with a per-micro-batch overhead (padding in both streams, NaN planted in it) and on single-sample
micro-batches.  fp32 runs the generic kernels, bf16 the matrix-core kernels."""
import numpy as np
import pytest
import torch

from oracle import stage as ost
from paper_2311_10418_amd import binding as ds
from paper_2311_10418_amd import workload as wl
from helpers import check, check_seqs, params_to_dev, run_t5_stage, seqs_from_stream, stream_from_seqs, tdtype, to_np, zero_grads_like

pytestmark = pytest.mark.gpu

CFG = dict(d_model=256, n_heads=4, d_ff=512, n_layers=2, n_dec_layers=2)
SPEC = dict(rule="count", count=24, mu=4.2, sigma=0.8, lo=8, hi=300, tgt_mu=3.0, tgt_sigma=0.9, tgt_lo=1, tgt_hi=150)


def _case(bf16):
    lens, tgts = wl.draw_lengths(SPEC, seed=2)
    ep = wl.draw_params(wl.T5_ENC_KEYS, CFG["n_layers"], CFG["d_model"], CFG["d_ff"], seed=2, tag=6, bf16=bf16, std=0.05)
    dp = wl.draw_params(wl.T5_DEC_KEYS, CFG["n_dec_layers"], CFG["d_model"], CFG["d_ff"], seed=2, tag=7, bf16=bf16, std=0.05)
    ex = wl.draw_rows(lens, CFG["d_model"], seed=2, tag=3, bf16=bf16)
    dx = wl.draw_rows(tgts, CFG["d_model"], seed=2, tag=8, bf16=bf16)
    ddy = wl.draw_rows(tgts, CFG["d_model"], seed=2, tag=5, bf16=bf16)
    return lens, tgts, ep, dp, ex, dx, ddy


@pytest.mark.parametrize("dtype_code", [ds.DS_DTYPE_F32, ds.DS_DTYPE_BF16])
def test_t5_stage_matches_oracle(dtype_code):
    bf16 = dtype_code == ds.DS_DTYPE_BF16
    tol = 2e-2 if bf16 else 1e-4
    lens, tgts, ep, dp, ex, dx, ddy = _case(bf16)
    r_outs, r_denc, r_ddec, r_eg, r_dg = ost.t5_stage_fwd_bwd(ex, dx, ddy, ep, dp, CFG["n_heads"])
    cm = ds.make_cost_model(kind=ds.DS_COST_POLY_T5, fixed=1_500_000)
    layouts = [("dp_overhead", ds.dp_plan(lens, cm, 2048, 4, lengths_tgt=tgts)),
               ("singletons", ds.ds_layout_from_cuts(lens, list(range(len(lens) + 1)), lengths_tgt=tgts))]
    assert layouts[0][1].total_rows > layouts[0][1].total_tokens          # the plan really pads
    for name, lo in layouts:
        got = run_t5_stage(lo, CFG, ep, dp, ex, dx, ddy, dtype_code)
        # every sample on its own, every weight-gradient tensor; normwise and elementwise (helpers.check)
        errs = {"dec_out": check_seqs(got["outs"], r_outs, tol, name + " dec_out"),
                "d_enc_in": check_seqs(got["d_enc"], r_denc, tol, name + " d_enc_in"),
                "d_dec_in": check_seqs(got["d_dec"], r_ddec, tol, name + " d_dec_in")}
        for tag, gg, rr in (("enc", got["eg"], r_eg), ("dec", got["dg"], r_dg)):
            for li, layer in enumerate(rr):
                for k, v in layer.items():
                    errs["%s%d.%s" % (tag, li, k)] = check(gg[li][k], v, tol, "%s %s%d.%s" % (name, tag, li, k))
        worst = max(errs, key=errs.get)
        print(name, "worst", worst, "%.3e" % errs[worst])
        for p in got["pads"]:
            assert p.size == 0 or np.all(p == 0), name


@pytest.mark.parametrize("dtype_code", [ds.DS_DTYPE_F32, ds.DS_DTYPE_BF16])
def test_decoder_gradient_returned_in_place(dtype_code):
    """One decoder layer without padding rows, grad_in_tgt is grad_out: every decoder gradient is the oracle's."""
    bf16, tol = dtype_code == ds.DS_DTYPE_BF16, 2e-2 if dtype_code == ds.DS_DTYPE_BF16 else 1e-4
    lens, tgts, ep, dp, ex, dx, ddy = _case(bf16)
    ep, dp, d = ep[:1], dp[:1], CFG["d_model"]
    _, _, r_dy, _, r_dg = ost.t5_stage_fwd_bwd(ex, dx, ddy, ep, dp, CFG["n_heads"])
    lo = ds.ds_layout_from_cuts(lens, list(range(len(lens) + 1)), lengths_tgt=tgts)
    assert lo.total_rows_tgt == int(tgts.sum())
    dt = tdtype(dtype_code)
    we, wd = params_to_dev(ep, dt), params_to_dev(dp, dt)
    ge, gd = zero_grads_like(we), zero_grads_like(wd)
    x, y, grad = stream_from_seqs(ex, lo, d, dt), stream_from_seqs(dx, lo, d, dt, which=1), stream_from_seqs(ddy, lo, d, dt, which=1)
    stage = ds.Stage(ds.DS_MODEL_T5, dtype_code, 1, d, CFG["n_heads"], CFG["d_ff"], max_rows=lo.total_rows, max_seqs=lo.n_seq,
                     n_dec_layers=1, max_rows_tgt=lo.total_rows_tgt)
    ds.stage_fwd_bwd(stage, lo, we, x, grad, torch.empty_like(y), torch.empty_like(x), ge, weights_dec=wd, grads_dec=gd, act_in_tgt=y,
                     grad_in_tgt=grad)
    torch.cuda.synchronize()
    check_seqs(seqs_from_stream(grad, lo, which=1)[0], r_dy, tol, "grad_in_tgt")
    for k, v in r_dg[0].items():
        check(to_np(gd[0][k]), v, tol, k)
    stage.close()


@pytest.mark.parametrize("dtype_code", [ds.DS_DTYPE_F32, ds.DS_DTYPE_BF16])
def test_decoder_outputs_as_their_own_gradient(dtype_code):
    """grad_out is act_out, with padding rows: the backward pass starts from this call's outputs."""
    bf16, tol = dtype_code == ds.DS_DTYPE_BF16, 2e-2 if dtype_code == ds.DS_DTYPE_BF16 else 1e-4
    lens, tgts, ep, dp, ex, dx, ddy = _case(bf16)
    d, dt = CFG["d_model"], tdtype(dtype_code)
    outs = ost.t5_stage_fwd_bwd(ex, dx, ddy, ep, dp, CFG["n_heads"])[0]
    _, _, r_dy, _, r_dg = ost.t5_stage_fwd_bwd(ex, dx, [wl.to_bf16_grid(o) if bf16 else o for o in outs], ep, dp, CFG["n_heads"])
    lo = ds.dp_plan(lens, ds.make_cost_model(kind=ds.DS_COST_POLY_T5, fixed=1_500_000), 2048, 4, lengths_tgt=tgts)
    assert lo.total_rows_tgt > int(tgts.sum())
    we, wd = params_to_dev(ep, dt), params_to_dev(dp, dt)
    ge, gd = zero_grads_like(we), zero_grads_like(wd)
    x, y = stream_from_seqs(ex, lo, d, dt), stream_from_seqs(dx, lo, d, dt, which=1)
    out, dy = torch.full_like(y, float("nan")), torch.empty_like(y)
    stage = ds.Stage(ds.DS_MODEL_T5, dtype_code, CFG["n_layers"], d, CFG["n_heads"], CFG["d_ff"], max_rows=lo.total_rows,
                     max_seqs=lo.n_seq, n_dec_layers=CFG["n_dec_layers"], max_rows_tgt=lo.total_rows_tgt)
    ds.stage_fwd_bwd(stage, lo, we, x, out, out, torch.empty_like(x), ge, weights_dec=wd, grads_dec=gd, act_in_tgt=y, grad_in_tgt=dy)
    torch.cuda.synchronize()
    check_seqs(seqs_from_stream(out, lo, which=1)[0], outs, tol, "act_out")
    check_seqs(seqs_from_stream(dy, lo, which=1)[0], r_dy, tol, "grad_in_tgt")
    for layer, ref in zip(gd, r_dg):
        for k, v in ref.items():
            check(to_np(layer[k]), v, tol, k)
    stage.close()


@pytest.mark.parametrize("dtype_code", [ds.DS_DTYPE_F32, ds.DS_DTYPE_BF16])
def test_decoder_parameters_that_share_a_gradient(dtype_code):
    """w_g, w_u and (of the same shape here) w_ckv; w_co, w_cq and w_o; the gains of the norms: summed in one buffer each."""
    bf16, tol = dtype_code == ds.DS_DTYPE_BF16, 2e-2 if dtype_code == ds.DS_DTYPE_BF16 else 1e-4
    lens, tgts, ep, dp, ex, dx, ddy = _case(bf16)
    ep, dp, d, dt = ep[:1], dp[:1], CFG["d_model"], tdtype(dtype_code)
    assert CFG["d_ff"] == 2 * d
    ref = ost.t5_stage_fwd_bwd(ex, dx, ddy, ep, dp, CFG["n_heads"])[4][0]
    lo = ds.ds_layout_from_cuts(lens, list(range(len(lens) + 1)), lengths_tgt=tgts)
    we, wd = params_to_dev(ep, dt), params_to_dev(dp, dt)
    ge, gd = zero_grads_like(we), zero_grads_like(wd)[0]
    shared = [("w_g", "w_u", "w_ckv"), ("w_co", "w_cq", "w_o"), ("ln2_g", "lnc_g", "ln1_g")]
    for names in shared:
        for k in names[1:]:
            gd[k] = gd[names[0]]
    x, y, dy = stream_from_seqs(ex, lo, d, dt), stream_from_seqs(dx, lo, d, dt, which=1), stream_from_seqs(ddy, lo, d, dt, which=1)
    stage = ds.Stage(ds.DS_MODEL_T5, dtype_code, 1, d, CFG["n_heads"], CFG["d_ff"], max_rows=lo.total_rows, max_seqs=lo.n_seq,
                     n_dec_layers=1, max_rows_tgt=lo.total_rows_tgt)
    ds.stage_fwd_bwd(stage, lo, we, x, dy, torch.empty_like(y), torch.empty_like(x), ge, weights_dec=wd, grads_dec=[gd], act_in_tgt=y,
                     grad_in_tgt=torch.empty_like(y), accumulate=True)
    torch.cuda.synchronize()
    for names in shared:
        check(to_np(gd[names[0]]), sum(ref[k] for k in names), tol, " + ".join(names))
    for k in ("w_2", "w_qkv"):
        check(to_np(gd[k]), ref[k], tol, k)
    stage.close()
