"""Performance cases: the work a user of this framework has it do, through its public entry points.

`listed()` names the cases, `draw(rng)` gives more of the same ranges, `prepare` makes what a program holds before the
call (inputs, weights, plan, stage), `run` makes one pass, `work` says what the pass cannot do without, `tolerance` how
far another correct implementation at the same precision may be off, and `exact` gives the outputs in 64 bits.

Kinds of case
  gpt        one stage_fwd_bwd call of a decoder-only stage over a planned global batch (forward, backward, all gradients)
  t5         the same for an encoder-decoder stage
  iteration  a pipeline stage that runs its micro-batches one after the other, one call each, gradients accumulated,
             the weights promised unchanged after the first call
  attention  ds_attention_fwd and / or ds_attention_bwd over variable-length sequences
  mlp        the projections of an MLP block through ds_gemm_ws: up (GELU), down (+ residual), both weight gradients, both
             input gradients
  norm       ds_norm_fwd and ds_norm_bwd
  pack       ds_pack and ds_unpack of a batch
  plan       dp_plan of a global batch (host only)

Sequence lengths are the log-normal draws of paper_2311_10418_amd/workload.py; values are N(0, 1) activations and
gradients and N(0, 0.02) weights, as there.
"""
import math

import numpy as np
import torch

from paper_2311_10418_amd import binding as ds
from paper_2311_10418_amd import workload as wl

DEV = "cuda"


# ------------------------------------------------------------------------------------ the cases
def listed():
    return [
        # the small fp32 configuration (64 sequences, 2 layers): what somebody runs first, and the fp32 path
        dict(name="gpt_256_f32", kind="gpt", dtype="f32", layers=2, d=256, heads=4, ff=1024, rule="count", count=64,
             mu=4.5, sigma=0.8, lo=8, hi=512, len_seed=0, fixed=0, cap=4096, stages=4, recompute=0),
        # a global batch of 65 536 tokens through two layers of the d = 2048 decoder stage, the everyday training call
        dict(name="gpt_2048_bf16", kind="gpt", dtype="bf16", layers=2, d=2048, heads=16, ff=8192, rule="tokens",
             tokens=65536, mu=5.5, sigma=1.0, lo=16, hi=2048, len_seed=0, fixed=0, cap=16384, stages=4, recompute=0),
        # one layer of the largest workload: 131 072 tokens with a long tail, d = 4096
        dict(name="gpt_4096_longtail_bf16", kind="gpt", dtype="bf16", layers=1, d=4096, heads=32, ff=16384,
             rule="tokens_bimodal", tokens=131072, p_short=0.7, mu=4.5, sigma=0.7, mu2=7.5, sigma2=0.5, lo=16, hi=8192,
             len_seed=0, fixed=0, cap=32768, stages=8, recompute=0),
        # one encoder and one decoder layer over 65 536 input tokens
        dict(name="t5_1024_bf16", kind="t5", dtype="bf16", layers=1, dec_layers=1, d=1024, heads=16, ff=2816,
             tokens=65536, mu=5.3, sigma=1.0, lo=8, hi=2048, tgt_mu=3.5, tgt_sigma=1.0, tgt_lo=1, tgt_hi=512, len_seed=0,
             fixed=0, cap=16384, stages=4),
        # a pipeline stage between its sends and receives: micro-batches of up to 2048 padded tokens, one call each
        dict(name="iteration_2048_bf16", kind="iteration", dtype="bf16", layers=2, d=2048, heads=16, ff=8192, tokens=8192,
             mu=5.5, sigma=1.0, lo=16, hi=2048, len_seed=0, fixed=2000000, cap=2048, stages=4),
        # the smallest call: one short micro-batch of a small bf16 stage; launches and latency count
        dict(name="gpt_256_bf16_short", kind="gpt", dtype="bf16", layers=2, d=256, heads=4, ff=1024, rule="count", count=5,
             mu=4.0, sigma=0.6, lo=8, hi=128, len_seed=1, fixed=2000000, cap=4096, stages=4, recompute=0),
        # attention of the d = 2048 decoder stage alone: causal, head size 128, forward and backward
        dict(name="attention_causal_128", kind="attention", dtype="bf16", heads=16, hd=128, causal=True, cross=False,
             fwd=True, bwd=True, tokens=65536, mu=5.5, sigma=1.0, lo=16, hi=2048, len_seed=0),
        # attention of the encoder: unmasked, head size 64, forward (the backward is in the whole-stage case)
        dict(name="attention_full_64_fwd", kind="attention", dtype="bf16", heads=16, hd=64, causal=False, cross=False,
             fwd=True, bwd=False, tokens=65536, mu=5.3, sigma=1.0, lo=8, hi=2048, len_seed=0),
        # the MLP projections of a mid-sized micro-batch (ragged row count) as a caller of the building blocks runs them
        dict(name="mlp_1024_bf16", kind="mlp", dtype="bf16", rows=4173, d=1024, ff=4096),
        # LayerNorm forward and backward of the widest model
        dict(name="norm_4096_bf16", kind="norm", dtype="bf16", rows=32771, d=4096, rms=False),
        # moving a batch into the padded stream and back, once per iteration each
        dict(name="pack_2048_bf16", kind="pack", dtype="bf16", d=2048, tokens=65536, mu=5.5, sigma=1.0, lo=16, hi=2048,
             len_seed=0, fixed=2000000, cap=16384, stages=4),
        # planning one global batch of the long-tail workload, with a fixed cost per micro-batch so that batching pays
        dict(name="plan_longtail", kind="plan", rule="tokens_bimodal", tokens=131072, p_short=0.7, mu=4.5, sigma=0.7,
             mu2=7.5, sigma2=0.5, lo=16, hi=8192, len_seed=0, fixed=2000000, cap=32768, stages=8),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _model(rng, dtype, widths):
    d = rng.choice(widths)
    hd = rng.choice([32, 64] if dtype == "f32" else [64, 128])
    while d % hd or d // hd < 2:
        hd = rng.choice([32, 64] if dtype == "f32" else [64, 128])
    return d, d // hd, d * rng.choice([2, 4] if dtype == "f32" else [3, 4])


def draw(rng):
    kind = rng.choice(["gpt", "gpt", "gpt_f32", "t5", "iteration", "iteration", "attention", "attention_f32", "mlp", "norm",
                       "pack", "plan"])
    seed = rng.randrange(1 << 20)
    mu, sigma = rng.uniform(4.0, 6.0), rng.uniform(0.5, 1.1)
    hi = rng.choice([512, 1024, 2048])
    lens = dict(mu=mu, sigma=sigma, lo=rng.choice([1, 8, 16]), hi=hi, len_seed=seed)
    fixed = rng.choice([0, 500000, 2000000])
    if kind == "gpt":
        d, heads, ff = _model(rng, "bf16", [256, 512, 768, 1024, 1536, 2048])
        return dict(kind="gpt", dtype="bf16", layers=rng.choice([1, 2]), d=d, heads=heads, ff=ff, rule="tokens",
                    tokens=_log(rng, 256, 65536), fixed=fixed, cap=rng.choice([4096, 16384]), stages=4,
                    recompute=rng.choice([0, 0, 0, 1]), **lens)
    if kind == "gpt_f32":
        d, heads, ff = _model(rng, "f32", [128, 192, 256, 384, 512])
        return dict(kind="gpt", dtype="f32", layers=rng.choice([1, 2]), d=d, heads=heads, ff=ff, rule="tokens",
                    tokens=_log(rng, 256, 12288), fixed=fixed, cap=4096, stages=4, recompute=rng.choice([0, 0, 0, 1]), **lens)
    if kind == "t5":
        d, heads, ff = _model(rng, "bf16", [256, 512, 1024])
        return dict(kind="t5", dtype="bf16", layers=1, dec_layers=1, d=d, heads=heads, ff=ff, tokens=_log(rng, 1024, 65536),
                    tgt_mu=rng.uniform(2.5, 4.5), tgt_sigma=1.0, tgt_lo=1, tgt_hi=512, fixed=fixed, cap=16384, stages=4, **lens)
    if kind == "iteration":
        d, heads, ff = _model(rng, "bf16", [512, 768, 1024, 1536, 2048])
        return dict(kind="iteration", dtype="bf16", layers=rng.choice([1, 2]), d=d, heads=heads, ff=ff,
                    tokens=_log(rng, 2048, 12288), fixed=max(fixed, 500000), cap=rng.choice([2048, 4096]), stages=4, **lens)
    if kind == "attention":
        hd = rng.choice([64, 128])
        cross = rng.random() < 0.3
        bwd = rng.random() < 0.6
        return dict(kind="attention", dtype="bf16", heads=rng.choice([4, 8, 12, 16]), hd=hd, causal=not cross and rng.random() < 0.6,
                    cross=cross, fwd=not bwd or rng.random() < 0.5, bwd=bwd, tokens=_log(rng, 512, 65536), **lens)
    if kind == "attention_f32":
        bwd = rng.random() < 0.5
        return dict(kind="attention", dtype="f32", heads=rng.choice([2, 4, 8]), hd=rng.choice([32, 64, 96, 128]),
                    causal=rng.random() < 0.6, cross=False, fwd=not bwd or rng.random() < 0.5, bwd=bwd,
                    tokens=_log(rng, 512, 8192), **lens)
    if kind == "mlp":
        d = rng.choice([256, 512, 768, 1024, 1536, 2048])
        return dict(kind="mlp", dtype="bf16", rows=_log(rng, 64, 32768), d=d, ff=d * rng.choice([3, 4]))
    if kind == "norm":
        return dict(kind="norm", dtype=rng.choice(["bf16", "bf16", "f32"]), rows=_log(rng, 64, 65536),
                    d=rng.choice([256, 512, 768, 1024, 1536, 2048, 3072, 4096]), rms=rng.random() < 0.5)
    if kind == "pack":
        return dict(kind="pack", dtype=rng.choice(["bf16", "f32"]), d=rng.choice([256, 768, 1024, 2048]),
                    tokens=_log(rng, 512, 65536), fixed=max(fixed, 500000), cap=16384, stages=4, **lens)
    return dict(kind="plan", rule="tokens", tokens=_log(rng, 4096, 24576), fixed=max(fixed, 500000),
                cap=rng.choice([16384, 32768]), stages=rng.choice([4, 8]), **lens)


# ------------------------------------------------------------------------------------ lengths and plans
def _lengths(case, seed=None):
    spec = {k: case[k] for k in ("mu", "sigma", "lo", "hi", "count", "tokens", "p_short", "mu2", "sigma2", "tgt_mu",
                                 "tgt_sigma", "tgt_lo", "tgt_hi") if k in case}
    spec["rule"] = case.get("rule", "tokens")
    return wl.draw_lengths(spec, case["len_seed"] if seed is None else seed)


def _plan(case, lens, tgts=None):
    cm = ds.make_cost_model(kind=ds.DS_COST_POLY_GPT if tgts is None else ds.DS_COST_POLY_T5, fixed=case["fixed"])
    return ds.dp_plan(lens, cm, max(case["cap"], int(lens.max())), case["stages"], lengths_tgt=tgts)


def _layouts(case):
    """The micro-batches of a plan, each as a layout of its own (kind "iteration")."""
    lens, _ = _lengths(case)
    plan = _plan(case, lens)
    cuts = plan.cuts
    return [ds.ds_layout_from_cuts(lens[plan.perm[a:b]], [0, int(b - a)]) for a, b in zip(cuts[:-1], cuts[1:])]


# ------------------------------------------------------------------------------------ inputs
def _gen(seed, tag=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 1000003 + tag)
    return g


def _randn(g, *shape, dtype, scale=1.0, shift=0.0):
    """Drawn in fp32, rounded once to the storage type."""
    return torch.randn(*shape, device=DEV, generator=g).mul_(scale).add_(shift).to(dtype)


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


_CODE = {"bf16": ds.DS_DTYPE_BF16, "f32": ds.DS_DTYPE_F32}


def _weights(g, keys, n, d, ff, dtype):
    shapes = {"w_qkv": (d, 3 * d), "b_qkv": (3 * d,), "w_1": (d, ff), "b_1": (ff,), "w_2": (ff, d), "w_g": (d, ff),
              "w_u": (d, ff), "w_ckv": (d, 2 * d), "w_o": (d, d), "w_cq": (d, d), "w_co": (d, d)}
    return [{k: _randn(g, *shapes.get(k, (d,)), dtype=dtype, scale=0.02,
                       shift=1.0 if k.startswith("ln") and k.endswith("_g") else 0.0) for k in keys} for _ in range(n)]


def _grads(weights):
    return [{k: torch.zeros(v.shape, dtype=torch.float32, device=DEV) for k, v in layer.items()} for layer in weights]


def _model_inputs(case, seed, rows, rows_tgt=0):
    g, dt, d = _gen(seed), _dtype(case), case["d"]
    st = {}
    if rows_tgt:
        st["w"] = _weights(g, ds.T5_ENC_KEYS, case["layers"], d, case["ff"], dt)
        st["wd"] = _weights(g, ds.T5_DEC_KEYS, case["dec_layers"], d, case["ff"], dt)
        st["y"] = _randn(g, rows_tgt, d, dtype=dt)
    else:
        st["w"] = _weights(g, ds.GPT_KEYS, case["layers"], d, case["ff"], dt)
    st["x"] = _randn(g, rows, d, dtype=dt)
    st["dy"] = _randn(g, rows_tgt or rows, d, dtype=dt)
    return st


def _i32(a):
    return torch.as_tensor(np.asarray(a), dtype=torch.int32, device=DEV)


def _attention_inputs(case, seed):
    lens, _ = _lengths(case)
    q_len = np.maximum(lens // 6, 1) if case["cross"] else lens
    g, dt, D = _gen(seed), _dtype(case), case["heads"] * case["hd"]
    Tq, Tk = int(q_len.sum()), int(lens.sum())
    st = {"q_len": q_len, "k_len": lens, "Tq": Tq, "Tk": Tk, "D": D}
    if case["cross"]:
        st["q"] = _randn(g, Tq, D, dtype=dt)
        st["kv"] = _randn(g, Tk, 2 * D, dtype=dt)
    else:
        st["qkv"] = _randn(g, Tk, 3 * D, dtype=dt)
    st["d_o"] = _randn(g, Tq, D, dtype=dt)
    return st


# ------------------------------------------------------------------------------------ prepare
def prepare(case, seed):
    st = {"case": case}
    kind = case["kind"]
    if kind == "gpt":
        lens, _ = _lengths(case)
        lo = _plan(case, lens)
        st.update(_model_inputs(case, seed, lo.total_rows))
        st.update(layout=lo, g=_grads(st["w"]), out=torch.empty_like(st["x"]), dx=torch.empty_like(st["x"]),
                  stage=ds.Stage(ds.DS_MODEL_GPT, _CODE[case["dtype"]], case["layers"], case["d"], case["heads"], case["ff"],
                                 max_rows=lo.total_rows, max_seqs=lo.n_seq, recompute=case["recompute"]))
    elif kind == "t5":
        lens, tgts = _lengths(case)
        lo = _plan(case, lens, tgts)
        st.update(_model_inputs(case, seed, lo.total_rows, lo.total_rows_tgt))
        st.update(layout=lo, g=_grads(st["w"]), gd=_grads(st["wd"]), out=torch.empty_like(st["y"]), dx=torch.empty_like(st["x"]),
                  dyin=torch.empty_like(st["y"]),
                  stage=ds.Stage(ds.DS_MODEL_T5, _CODE[case["dtype"]], case["layers"], case["d"], case["heads"], case["ff"],
                                 max_rows=lo.total_rows, max_seqs=lo.n_seq, n_dec_layers=case["dec_layers"],
                                 max_rows_tgt=lo.total_rows_tgt))
    elif kind == "iteration":
        los = _layouts(case)
        rows = [lo.total_rows for lo in los]
        st.update(_model_inputs(case, seed, sum(rows)))
        st.update(layouts=los, g=_grads(st["w"]), out=torch.empty_like(st["x"]), dx=torch.empty_like(st["x"]),
                  stage=ds.Stage(ds.DS_MODEL_GPT, _CODE[case["dtype"]], case["layers"], case["d"], case["heads"], case["ff"],
                                 max_rows=max(rows), max_seqs=max(lo.n_seq for lo in los)))
        st["at"] = [0] + list(np.cumsum(rows))
    elif kind == "attention":
        st.update(_attention_inputs(case, seed))
        q_row, k_row = np.cumsum(st["q_len"]) - st["q_len"], np.cumsum(st["k_len"]) - st["k_len"]
        st["rows"] = (_i32(q_row), _i32(st["q_len"]), _i32(k_row), _i32(st["k_len"]))
        st["max"] = (int(st["q_len"].max()), int(st["k_len"].max()))
        dt, h, Tq, D = _dtype(case), case["heads"], st["Tq"], st["D"]
        st["o"] = torch.empty(Tq, D, dtype=dt, device=DEV)
        st["lse"] = torch.empty(h, Tq, device=DEV)
        nbytes = ds.ds_attention_scratch_bytes(h, case["hd"], Tq, st["Tk"], len(st["q_len"]))
        st["scratch"] = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
        if case["bwd"]:
            st["delta"] = torch.empty(h, Tq, device=DEV)
            st["grads"] = {k: torch.empty_like(st[k]) for k in ("q", "kv", "qkv") if k in st}
            if not case["fwd"]:
                _attention_fwd(st)           # what the forward pass left behind
    elif kind == "mlp":
        g, dt, R, d, F = _gen(seed), _dtype(case), case["rows"], case["d"], case["ff"]
        st.update(x=_randn(g, R, d, dtype=dt), resid=_randn(g, R, d, dtype=dt), dy=_randn(g, R, d, dtype=dt),
                  w1=_randn(g, d, F, dtype=dt, scale=0.02), w2=_randn(g, F, d, dtype=dt, scale=0.02),
                  b1=_randn(g, F, dtype=dt, scale=0.02), b2=_randn(g, d, dtype=dt, scale=0.02))
        st.update(w1t=st["w1"].t().contiguous(), w2t=st["w2"].t().contiguous())     # [out][in] copies for the forward products
        e = lambda *s: torch.empty(*s, dtype=dt, device=DEV)  # noqa: E731
        st.update(dgelu=e(R, F), a=e(R, F), y=e(R, d), dz=e(R, F), dx=e(R, d), gw1=torch.empty(d, F, device=DEV),
                  gw2=torch.empty(F, d, device=DEV), ws=torch.empty(4 * max(3 * d * d, d * F), device=DEV))
    elif kind == "norm":
        g, dt, R, d = _gen(seed), _dtype(case), case["rows"], case["d"]
        st.update(x=_randn(g, R, d, dtype=dt), dy=_randn(g, R, d, dtype=dt), resid=_randn(g, R, d, dtype=dt),
                  g=_randn(g, d, dtype=dt, scale=0.02, shift=1.0), b=None if case["rms"] else _randn(g, d, dtype=dt, scale=0.02))
        st.update(y=torch.empty_like(st["x"]), dx=torch.empty_like(st["x"]), stats=torch.empty(2, R, device=DEV),
                  dg=torch.empty(d, device=DEV), db=None if case["rms"] else torch.empty(d, device=DEV),
                  partial=torch.empty(ds.ds_norm_bwd_scratch_floats(R, d), device=DEV))
    elif kind == "pack":
        lens, _ = _lengths(case)
        lo = _plan(case, lens)
        st.update(layout=lo, canon=_randn(_gen(seed), int(lens.sum()), case["d"], dtype=_dtype(case)))
        st.update(rows=torch.empty(lo.total_rows, case["d"], dtype=_dtype(case), device=DEV), back=torch.empty_like(st["canon"]))
    elif kind == "plan":
        # the same batch for every seed, its samples in another order: the cost of a plan stays that of the case
        lens, _ = _lengths(case)
        st["lens"] = np.ascontiguousarray(np.random.default_rng(seed).permutation(lens))
        st["cm"] = ds.make_cost_model(fixed=case["fixed"])
    else:
        raise ValueError(kind)
    return st


# ------------------------------------------------------------------------------------ run
def _attention_args(st):
    case, D = st["case"], st["D"]
    es = 2 if case["dtype"] == "bf16" else 4
    if case["cross"]:
        q, ldq, ldk = st["q"].data_ptr(), D, 2 * D
        k = st["kv"].data_ptr()
        v = k + D * es
    else:
        q, ldq, ldk = st["qkv"].data_ptr(), 3 * D, 3 * D
        k, v = q + D * es, q + 2 * D * es
    return (q, k, v), ldq, ldk, es


def _attention_fwd(st):
    case, (q, k, v), ldq, ldk = st["case"], *_attention_args(st)[:3]
    ds.ds_attention_fwd(q, k, v, st["o"], st["lse"], *st["rows"], case["heads"], case["hd"], case["causal"], *st["max"],
                        ldq, ldk, ldk, st["D"], st["Tq"], k_total_rows=st["Tk"], scratch=st["scratch"])


def _attention_bwd(st):
    case, ((q, k, v), ldq, ldk, es), D = st["case"], _attention_args(st), st["D"]
    gr = st["grads"]
    if case["cross"]:
        dq, dk = gr["q"].data_ptr(), gr["kv"].data_ptr()
        dv = dk + D * es
    else:
        dq = gr["qkv"].data_ptr()
        dk, dv = dq + D * es, dq + 2 * D * es
    ds.ds_attention_bwd(q, k, v, st["o"], st["d_o"], st["lse"], st["delta"], dq, dk, dv, *st["rows"], case["heads"],
                        case["hd"], case["causal"], *st["max"], ldq, ldk, ldk, D, st["Tq"], k_total_rows=st["Tk"],
                        scratch=st["scratch"])


def run(st):
    kind = st["case"]["kind"]
    if kind == "gpt":
        ds.stage_fwd_bwd(st["stage"], st["layout"], st["w"], st["x"], st["dy"], st["out"], st["dx"], st["g"])
        return {"out": st["out"], "dx": st["dx"], "g": st["g"]}
    if kind == "t5":
        ds.stage_fwd_bwd(st["stage"], st["layout"], st["w"], st["x"], st["dy"], st["out"], st["dx"], st["g"],
                         weights_dec=st["wd"], grads_dec=st["gd"], act_in_tgt=st["y"], grad_in_tgt=st["dyin"])
        return {"out": st["out"], "dx": st["dx"], "dy": st["dyin"], "g": st["g"], "gd": st["gd"]}
    if kind == "iteration":
        at = st["at"]
        st["stage"].weights_unchanged(False)             # new weights since the last iteration's optimizer step
        for i, lo in enumerate(st["layouts"]):
            r = slice(int(at[i]), int(at[i + 1]))
            ds.stage_fwd_bwd(st["stage"], lo, st["w"], st["x"][r], st["dy"][r], st["out"][r], st["dx"][r], st["g"],
                             accumulate=i > 0)
            if i == 0:
                st["stage"].weights_unchanged(True)
        return {"out": st["out"], "dx": st["dx"], "g": st["g"]}
    if kind == "attention":
        res = {}
        if st["case"]["fwd"]:
            _attention_fwd(st)
            res.update(o=st["o"], lse=st["lse"])
        if st["case"]["bwd"]:
            _attention_bwd(st)
            res.update(st["grads"])
        return res
    if kind == "mlp":
        R, d, F, ws = st["case"]["rows"], st["case"]["d"], st["case"]["ff"], st["ws"]
        ds.ds_gemm(st["x"], st["w1t"], st["dgelu"], R, F, d, trans_b=True, epilogue=ds.DS_EPI_GELU_D, bias=st["b1"], C2=st["a"], workspace=ws)
        ds.ds_gemm(st["a"], st["w2t"], st["y"], R, d, F, trans_b=True, epilogue=ds.DS_EPI_RESID, bias=st["b2"], R=st["resid"], workspace=ws)
        ds.ds_gemm(st["a"], st["dy"], st["gw2"], F, d, R, trans_a=True, epilogue=ds.DS_EPI_ACC32, workspace=ws)
        ds.ds_gemm(st["dy"], st["w2"], st["dz"], R, F, d, trans_b=True, epilogue=ds.DS_EPI_MULR, R=st["dgelu"], workspace=ws)
        ds.ds_gemm(st["x"], st["dz"], st["gw1"], d, F, R, trans_a=True, epilogue=ds.DS_EPI_ACC32, workspace=ws)
        ds.ds_gemm(st["dz"], st["w1"], st["dx"], R, d, F, trans_b=True, workspace=ws)
        return {k: st[k] for k in ("y", "gw2", "gw1", "dx")}
    if kind == "norm":
        rms = st["case"]["rms"]
        ds.ds_norm_fwd(st["x"], st["g"], st["b"], st["y"], st["stats"], rms=rms)
        ds.ds_norm_bwd(st["dy"], st["x"], st["g"], st["stats"], st["resid"], st["dx"], st["dg"], st["db"], st["partial"], rms=rms)
        return {"y": st["y"], "dx": st["dx"], "dg": st["dg"], "db": st["db"]}
    if kind == "pack":
        ds.ds_pack(st["layout"], st["canon"], st["rows"])
        ds.ds_unpack(st["layout"], st["rows"], st["back"])
        return {"rows": st["rows"], "back": st["back"]}
    case = st["case"]
    lo = ds.dp_plan(st["lens"], st["cm"], max(case["cap"], int(st["lens"].max())), case["stages"])
    return {"cuts": lo.cuts, "perm": lo.perm, "objective": lo.objective, "seq_row": lo.seq_row}


# ------------------------------------------------------------------------------------ work and tolerance
def _pairs(ql, kl, causal):
    ql, kl = np.asarray(ql, dtype=np.int64), np.asarray(kl, dtype=np.int64)
    return int((ql * (ql + 1) // 2).sum()) if causal else int((ql * kl).sum())


def work(case):
    """Non-padding tokens and the causal triangle only; each input read once, each output written once."""
    kind = case["kind"]
    es = 2 if case.get("dtype") == "bf16" else 4
    if kind in ("gpt", "iteration"):
        lens, _ = _lengths(case)
        T, d, F, L = int(lens.sum()), case["d"], case["ff"], case["layers"]
        n_w = (4 * d * d + 2 * d * F) * L
        return {"flops": 6 * n_w * T + 12 * d * _pairs(lens, lens, True) * L, "bytes": n_w * (es + 4) + 4 * T * d * es}
    if kind == "t5":
        lens, tgts = _lengths(case)
        T, U, d, F, L, M = int(lens.sum()), int(tgts.sum()), case["d"], case["ff"], case["layers"], case["dec_layers"]
        n_e, n_d = (4 * d * d + 3 * d * F) * L, (8 * d * d + 3 * d * F) * M
        flops = 6 * (n_e * T + (6 * d * d + 3 * d * F) * M * U + 2 * d * d * M * T)
        flops += 12 * d * (_pairs(lens, lens, False) * L + (_pairs(tgts, tgts, True) + _pairs(tgts, lens, False)) * M)
        return {"flops": flops, "bytes": (n_e + n_d) * (es + 4) + (2 * T + 4 * U) * d * es}
    if kind == "attention":
        lens, _ = _lengths(case)
        ql = np.maximum(lens // 6, 1) if case["cross"] else lens
        D, n, m = case["heads"] * case["hd"], int(ql.sum()), int(lens.sum())
        flops, nbytes = 0, 0
        if case["fwd"]:
            flops += 4 * D * _pairs(ql, lens, case["causal"])
            nbytes += (2 * n + 2 * m) * D * es + 4 * n * case["heads"]
        if case["bwd"]:
            # the scores again, dP, dV, dK, dQ; reads q, k, v, o, do, lse, writes dq, dk, dv
            flops += 10 * D * _pairs(ql, lens, case["causal"])
            nbytes += (4 * n + 4 * m) * D * es + 4 * n * case["heads"]
        return {"flops": flops, "bytes": nbytes}
    if kind == "mlp":
        R, d, F = case["rows"], case["d"], case["ff"]
        return {"flops": 12 * R * d * F, "bytes": 2 * d * F * (2 * es + 4) + R * d * es * 5}
    if kind == "norm":
        n = case["rows"] * case["d"]
        return {"flops": 16 * n, "bytes": 6 * n * es + 12 * case["rows"]}
    if kind == "pack":
        lens, _ = _lengths(case)
        return {"flops": 0, "bytes": 4 * int(lens.sum()) * case["d"] * es}
    lens, _ = _lengths(case)
    return {"flops": len(lens) ** 2, "bytes": 12 * len(lens)}


def tolerance(case):
    kind = case["kind"]
    if kind in ("plan", "pack"):
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 5e-6}
    if kind == "norm":
        return {"rel": 6e-3}
    return {"rel": 1e-2} if kind in ("attention", "mlp") else {"rel": 2e-2}


# ------------------------------------------------------------------------------------ exact
def _attend(q, k, v, heads, causal):
    """[l, D] each, 64 bits -> ([l, D], lse [heads, l])"""
    hd = q.shape[1] // heads
    q, k, v = (t.reshape(t.shape[0], heads, hd).transpose(0, 1).contiguous() for t in (q, k, v))
    s = torch.matmul(q, k.transpose(1, 2).contiguous()) / math.sqrt(hd)
    if causal:
        s = s.masked_fill(torch.ones(s.shape[1:], dtype=torch.bool, device=s.device).triu(1), float("-inf"))
    lse = torch.logsumexp(s, dim=2)
    o = torch.matmul(torch.softmax(s, dim=2), v)
    return o.transpose(0, 1).reshape(-1, heads * hd), lse


def _attend_all(q, k, v, q_row, q_len, k_row, k_len, heads, causal):
    """All sequences; rows that belong to none are zero."""
    order = np.argsort(q_row, kind="stable")
    parts, at = [], 0
    for i in order:
        a, n, b, m = int(q_row[i]), int(q_len[i]), int(k_row[i]), int(k_len[i])
        if a > at:
            parts.append(q.new_zeros(a - at, v.shape[1]))
        parts.append(_attend(q[a:a + n], k[b:b + m], v[b:b + m], heads, causal)[0])
        at = a + n
    if at < q.shape[0]:
        parts.append(q.new_zeros(q.shape[0] - at, v.shape[1]))
    return torch.cat(parts)


def _layer_norm(x, g, b):
    c = x - x.mean(1, keepdim=True)
    return c / torch.sqrt((c * c).mean(1, keepdim=True) + 1e-5) * g + b


def _rms_norm(x, g):
    return x / torch.sqrt((x * x).mean(1, keepdim=True) + 1e-6) * g


def _gelu(z):
    return torch.nn.functional.gelu(z, approximate="tanh")


def _valid(rows, row, length):
    v = torch.zeros(rows, 1, dtype=torch.float64, device=DEV)
    for a, n in zip(row, length):
        v[int(a):int(a) + int(n)] = 1.0
    return v


def _gpt_exact(x, dy, w, lo, heads):
    d = x.shape[1]
    valid = _valid(lo.total_rows, lo.seq_row, lo.seq_len)
    w = [{k: t.double().requires_grad_() for k, t in layer.items()} for layer in w]
    x = (x.double() * valid).requires_grad_()
    h = x
    for p in w:
        qkv = _layer_norm(h, p["ln1_g"], p["ln1_b"]) @ p["w_qkv"] + p["b_qkv"]
        o = _attend_all(qkv[:, :d], qkv[:, d:2 * d], qkv[:, 2 * d:], lo.seq_row, lo.seq_len, lo.seq_row, lo.seq_len, heads, True)
        h = (h + o @ p["w_o"] + p["b_o"]) * valid
        h = (h + _gelu(_layer_norm(h, p["ln2_g"], p["ln2_b"]) @ p["w_1"] + p["b_1"]) @ p["w_2"] + p["b_2"]) * valid
    h.backward(dy.double() * valid)
    return h.detach(), x.grad * valid, [{k: t.grad for k, t in p.items()} for p in w]


def _t5_exact(st, lo, heads):
    d = st["x"].shape[1]
    ve, vd = _valid(lo.total_rows, lo.seq_row, lo.seq_len), _valid(lo.total_rows_tgt, lo.seq_row_tgt, lo.seq_len_tgt)
    w, wd = ([{k: t.double().requires_grad_() for k, t in layer.items()} for layer in st[n]] for n in ("w", "wd"))
    x, y = (st["x"].double() * ve).requires_grad_(), (st["y"].double() * vd).requires_grad_()
    E, D = (lo.seq_row, lo.seq_len), (lo.seq_row_tgt, lo.seq_len_tgt)

    def self_attention(h, p, rows, causal, valid):
        qkv = _rms_norm(h, p["ln1_g"]) @ p["w_qkv"]
        return (h + _attend_all(qkv[:, :d], qkv[:, d:2 * d], qkv[:, 2 * d:], *rows, *rows, heads, causal) @ p["w_o"]) * valid

    def mlp(h, p, valid):
        u = _rms_norm(h, p["ln2_g"])
        return (h + (_gelu(u @ p["w_g"]) * (u @ p["w_u"])) @ p["w_2"]) * valid

    h = x
    for p in w:
        h = mlp(self_attention(h, p, E, False, ve), p, ve)
    t = y
    for p in wd:
        t = self_attention(t, p, D, True, vd)
        kv = h @ p["w_ckv"]
        t = (t + _attend_all(_rms_norm(t, p["lnc_g"]) @ p["w_cq"], kv[:, :d], kv[:, d:], *D, *E, heads, False) @ p["w_co"]) * vd
        t = mlp(t, p, vd)
    t.backward(st["dy"].double() * vd)
    grads = [[{k: v.grad for k, v in p.items()} for p in layers] for layers in (w, wd)]
    return {"out": t.detach(), "dx": x.grad * ve, "dy": y.grad * vd, "g": grads[0], "gd": grads[1]}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("gpt", "iteration", "t5"):
        lens, tgts = _lengths(case)
        if int(lens.sum()) * case["ff"] * case["layers"] > 1.2e9:        # tens of seconds and most of the card in 64 bits
            return None
    if kind == "gpt":
        lo = _plan(case, lens)
        st = _model_inputs(case, seed, lo.total_rows)
        out, dx, g = _gpt_exact(st["x"], st["dy"], st["w"], lo, case["heads"])
        return {"out": out, "dx": dx, "g": g}
    if kind == "t5":
        lo = _plan(case, lens, tgts)
        return _t5_exact(_model_inputs(case, seed, lo.total_rows, lo.total_rows_tgt), lo, case["heads"])
    if kind == "iteration":
        los = _layouts(case)
        st = _model_inputs(case, seed, sum(lo.total_rows for lo in los))
        outs, dxs, total, at = [], [], None, 0
        for lo in los:
            r = slice(at, at + lo.total_rows)
            out, dx, g = _gpt_exact(st["x"][r], st["dy"][r], st["w"], lo, case["heads"])
            outs.append(out)
            dxs.append(dx)
            total = g if total is None else [{k: a[k] + b[k] for k in a} for a, b in zip(total, g)]
            at += lo.total_rows
        return {"out": torch.cat(outs), "dx": torch.cat(dxs), "g": total}
    if kind == "attention":
        st = _attention_inputs(case, seed)
        D, h = st["D"], case["heads"]
        if case["cross"]:
            leaves = {"q": st["q"].double().requires_grad_(), "kv": st["kv"].double().requires_grad_()}
            q, k, v = leaves["q"], leaves["kv"][:, :D], leaves["kv"][:, D:]
        else:
            leaves = {"qkv": st["qkv"].double().requires_grad_()}
            q, k, v = (leaves["qkv"][:, i * D:(i + 1) * D] for i in range(3))
        outs, lses, a, b = [], [], 0, 0
        for n, m in zip(st["q_len"].tolist(), st["k_len"].tolist()):
            o, lse = _attend(q[a:a + n], k[b:b + m], v[b:b + m], h, case["causal"])
            if case["bwd"]:
                (o * st["d_o"][a:a + n].double()).sum().backward(retain_graph=False)
            outs.append(o.detach())
            lses.append(lse.detach())
            a, b = a + n, b + m
        res = {"o": torch.cat(outs), "lse": torch.cat(lses, dim=1)} if case["fwd"] else {}
        if case["bwd"]:
            res.update({k_: t.grad for k_, t in leaves.items()})
        return res
    if kind == "mlp":
        if case["rows"] * case["d"] * case["ff"] > 1e11:
            return None
        st = prepare(case, seed)
        x, resid, dy, w1, w2, b1, b2 = (st[k].double() for k in ("x", "resid", "dy", "w1", "w2", "b1", "b2"))
        del st
        x, w1, w2 = (t.requires_grad_() for t in (x, w1, w2))
        y = resid + _gelu(x @ w1 + b1) @ w2 + b2
        y.backward(dy)
        return {"y": y.detach(), "gw2": w2.grad, "gw1": w1.grad, "dx": x.grad}
    if kind == "norm":
        st = prepare(case, seed)
        x, g = st["x"].double().requires_grad_(), st["g"].double().requires_grad_()
        b = None if case["rms"] else st["b"].double().requires_grad_()
        y = _rms_norm(x, g) if case["rms"] else _layer_norm(x, g, b)
        y.backward(st["dy"].double())
        return {"y": y.detach(), "dx": x.grad + st["resid"].double(), "dg": g.grad, "db": None if b is None else b.grad}
    return None
