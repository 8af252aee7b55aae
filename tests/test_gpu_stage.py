"""GPU parity of stage_fwd_bwd against the per-sequence float64 oracle, through the C ABI.

Bar: normwise relative error <= 1e-4 for fp32 and <= 2e-2 for bf16 storage, for the outputs and input
gradients of EVERY SEQUENCE on its own and for each weight-gradient tensor, each with the elementwise
companion bound of helpers.check; padding rows of the outputs exactly zero; results
independent of the micro-batch layout (DP plan, padded DP plan, fixed padding, packing,
single-sequence micro-batches), with NaN planted in every padding row of the inputs."""
import numpy as np
import pytest
import torch

from oracle import stage as ost
from paper_2311_10418_amd import binding as ds
from paper_2311_10418_amd import workload as wl
from helpers import check, check_seqs, rel_err, run_gpt_stage

pytestmark = pytest.mark.gpu

TOL = {ds.DS_DTYPE_F32: 1e-4, ds.DS_DTYPE_BF16: 2e-2}


def _small_case(bf16, n_seq=None, seed=0):
    cfg = dict(wl.CONFIGS["gpt_small_fp32"])
    lens, _ = wl.draw_lengths(cfg["lengths"], seed=seed)
    if n_seq:
        lens = lens[:n_seq]
    params = wl.draw_params(wl.GPT_KEYS, cfg["n_layers"], cfg["d_model"], cfg["d_ff"], seed=seed, bf16=bf16)
    xs = wl.draw_embedded_tokens(lens, cfg["d_model"], seed=seed, bf16=bf16)
    dys = wl.draw_rows(lens, cfg["d_model"], seed=seed, tag=5, bf16=bf16)
    return cfg, lens, params, xs, dys


_ORACLE_CACHE = {}


def _oracle(key, xs, dys, params, h):
    if key not in _ORACLE_CACHE:
        _ORACLE_CACHE[key] = ost.gpt_stage_fwd_bwd(xs, dys, params, h)
    return _ORACLE_CACHE[key]


def _compare(tag, got, ref, tol):
    outs, dxs, grads, pad_o, pad_dx = got
    r_outs, r_dxs, r_grads = ref
    # outputs and input gradients: every sequence on its own; weight gradients: every tensor; each normwise AND elementwise
    errs = {"act_out": check_seqs(outs, r_outs, tol, tag + " act_out"), "grad_in": check_seqs(dxs, r_dxs, tol, tag + " grad_in")}
    for li, layer in enumerate(r_grads):
        for k, v in layer.items():
            errs["L%d.%s" % (li, k)] = check(grads[li][k], v, tol, "%s L%d.%s" % (tag, li, k))
    worst = max(errs, key=errs.get)
    print(tag, "worst", worst, "%.3e" % errs[worst])
    assert pad_o.size == 0 or np.all(pad_o == 0), tag
    assert pad_dx.size == 0 or np.all(pad_dx == 0), tag
    return errs


def _layouts(lens, cap, c):
    n = len(lens)
    yield "dp", ds.dp_plan(lens, ds.make_cost_model(), cap, c)
    yield "dp_overhead", ds.dp_plan(lens, ds.make_cost_model(fixed=2_000_000), cap, c)
    yield "fixed_pad", ds.ds_layout_from_cuts(lens, list(range(0, n, 8)) + [n], pad_to=int(max(lens)))
    yield "packed", ds.ds_layout_packed(lens, int(max(lens)), 4)
    yield "singletons", ds.ds_layout_from_cuts(lens, list(range(n + 1)))


@pytest.mark.parametrize("dtype_code", [ds.DS_DTYPE_F32, ds.DS_DTYPE_BF16])
def test_small_gpt_stage_matches_oracle_on_every_layout(dtype_code):
    bf16 = dtype_code == ds.DS_DTYPE_BF16
    cfg, lens, params, xs, dys = _small_case(bf16)
    ref = _oracle(("small", bf16), xs, dys, params, cfg["n_heads"])
    for name, lo in _layouts(lens, cfg["cap"], cfg["num_stages"]):
        got = run_gpt_stage(lo, cfg, params, xs, dys, dtype_code)
        _compare("%s/%s rows=%d tokens=%d" % ("bf16" if bf16 else "f32", name, lo.total_rows, lo.total_tokens),
                 got, ref, TOL[dtype_code])


def test_weight_gradients_accumulate_across_calls():
    cfg, lens, params, xs, dys = _small_case(True, n_seq=12)
    ref = _oracle(("small12", True), xs, dys, params, cfg["n_heads"])
    lo = ds.dp_plan(lens, ds.make_cost_model(fixed=2_000_000), cfg["cap"], cfg["num_stages"])
    stage = ds.Stage(ds.DS_MODEL_GPT, ds.DS_DTYPE_BF16, cfg["n_layers"], cfg["d_model"], cfg["n_heads"], cfg["d_ff"],
                     max_rows=lo.total_rows + 100, max_seqs=64)
    from helpers import params_to_dev, zero_grads_like
    grads = zero_grads_like(params_to_dev(params, torch.bfloat16))
    for g in grads:
        for v in g.values():
            v.fill_(123.0)                       # overwritten by the first (non-accumulating) call
    run_gpt_stage(lo, cfg, params, xs, dys, ds.DS_DTYPE_BF16, stage=stage, grads=grads, accumulate=False)
    got = run_gpt_stage(lo, cfg, params, xs, dys, ds.DS_DTYPE_BF16, stage=stage, grads=grads, accumulate=True)
    for li, layer in enumerate(ref[2]):
        for k, v in layer.items():
            check(got[2][li][k], 2 * v, 2e-2, "accumulated L%d.%s" % (li, k))
    # same stage object, another layout right after: tables are re-bound
    lo2 = ds.ds_layout_from_cuts(lens, list(range(len(lens) + 1)))
    got2 = run_gpt_stage(lo2, cfg, params, xs, dys, ds.DS_DTYPE_BF16, stage=stage)
    _compare("rebind", got2, ref, 2e-2)
    stage.close()


def test_weight_copies_are_reused_only_under_the_callers_promise():
    """Micro-batches of one iteration run on the same weights: with the promise the transposed copies are made once."""
    from helpers import params_to_dev, stream_from_seqs, to_np
    cfg, lens, params, xs, dys = _small_case(True, n_seq=12)
    lo = ds.dp_plan(lens, ds.make_cost_model(fixed=2_000_000), cfg["cap"], cfg["num_stages"])
    d = cfg["d_model"]
    stage = ds.Stage(ds.DS_MODEL_GPT, ds.DS_DTYPE_BF16, cfg["n_layers"], d, cfg["n_heads"], cfg["d_ff"],
                     max_rows=lo.total_rows, max_seqs=64)
    w = params_to_dev(params, torch.bfloat16)
    x = stream_from_seqs(xs, lo, d, torch.bfloat16, 0.0)
    dy = stream_from_seqs(dys, lo, d, torch.bfloat16, 0.0)

    def call():
        out, dx = torch.empty_like(x), torch.empty_like(x)
        g = [{k: torch.zeros(v.shape, dtype=torch.float32, device=x.device) for k, v in layer.items()} for layer in w]
        ds.stage_fwd_bwd(stage, lo, w, x, dy, out, dx, g)
        torch.cuda.synchronize()
        return to_np(out), to_np(dx), stage.last_launch_count()

    call()                                       # (the first call of a layout also builds the attention work lists)
    out0, dx0, n0 = call()
    stage.weights_unchanged(True)
    out1, dx1, n1 = call()                       # first call under the promise: same weights as before, copies reused
    assert n1 == n0 - 4 * cfg["n_layers"]
    assert np.array_equal(out0, out1) and np.array_equal(dx0, dx1)
    # an optimizer step: the promise is withdrawn, the new weights are seen
    stage.weights_unchanged(False)
    for layer in w:
        layer["w_2"].mul_(0.5)
    out2, _, n2 = call()
    assert n2 == n0 and not np.array_equal(out0, out2)
    # under the promise again, but with other weight tensors: the copies are made anew all the same
    stage.weights_unchanged(True)
    w = params_to_dev(params, torch.bfloat16)
    out3, dx3, n3 = call()
    assert n3 == n0 and np.array_equal(out0, out3) and np.array_equal(dx0, dx3)
    stage.close()


def test_layout_too_large_for_workspace_is_rejected():
    cfg, lens, params, xs, dys = _small_case(True, n_seq=6)
    lo = ds.ds_layout_from_cuts(lens, list(range(len(lens) + 1)))
    stage = ds.Stage(ds.DS_MODEL_GPT, ds.DS_DTYPE_BF16, 1, cfg["d_model"], cfg["n_heads"], cfg["d_ff"],
                     max_rows=lo.total_rows - 1, max_seqs=64)
    with pytest.raises(ds.DsError) as e:
        run_gpt_stage(lo, dict(cfg, n_layers=1), params[:1], xs, dys, ds.DS_DTYPE_BF16, stage=stage)
    assert e.value.code == ds.DS_ELAYOUT
    stage.close()


def _overlap_case(size):
    """A small padded batch, whose bias and norm gradients are summed in one launch at the end of a layer, and one whose tensors are too
    large for that (over 96 MiB): their column sums go to the stage's own stream."""
    if size == "together":
        cfg, lens, params, xs, dys = _small_case(True, n_seq=12)
        return cfg, params, xs, dys, ds.dp_plan(lens, ds.make_cost_model(fixed=2_000_000), cfg["cap"], cfg["num_stages"])
    cfg, lens = dict(n_layers=1, d_model=2048, n_heads=16, d_ff=512), np.asarray([450, 500] * 6)
    params = wl.draw_params(wl.GPT_KEYS, 1, 2048, 512, seed=13, bf16=True)
    xs, dys = wl.draw_rows(lens, 2048, seed=13, tag=3, bf16=True), wl.draw_rows(lens, 2048, seed=13, tag=5, bf16=True)
    return cfg, params, xs, dys, ds.ds_layout_from_cuts(lens, list(range(0, 13, 2)))


def _column_sum_launches(stage, call):
    stage.profile_enable(True)
    stage.profile_read()
    call()
    torch.cuda.synchronize()
    n = stage.profile_read()["colsum"][1]
    stage.profile_enable(False)
    return n


@pytest.mark.parametrize("size", ["together", "side stream"])
def test_stage_call_can_be_captured_in_a_graph_and_replays_identically(size):
    """With its layout already bound (one eager call), stage_fwd_bwd only enqueues kernels: it can be captured in a
    HIP graph; every replay, with eager work and synchronisation in between, reproduces the eager result bit for bit."""
    cfg, params, xs, dys, lo = _overlap_case(size)
    from helpers import params_to_dev, stream_from_seqs, zero_grads_like
    d = cfg["d_model"]
    stage = ds.Stage(ds.DS_MODEL_GPT, ds.DS_DTYPE_BF16, cfg["n_layers"], d, cfg["n_heads"], cfg["d_ff"],
                     max_rows=lo.total_rows, max_seqs=lo.n_seq)
    w = params_to_dev(params, torch.bfloat16)
    grads = zero_grads_like(w)
    x = stream_from_seqs(xs, lo, d, torch.bfloat16, 0.0)
    dy = stream_from_seqs(dys, lo, d, torch.bfloat16, 0.0)
    out, dx = torch.empty_like(x), torch.empty_like(x)

    def call():
        ds.stage_fwd_bwd(stage, lo, w, x, dy, out, dx, grads, accumulate=False)

    def snapshot():
        return [out.clone(), dx.clone()] + [g[k].clone() for g in grads for k in g]

    for _ in range(2):
        call()
    torch.cuda.synchronize()
    ref = snapshot()
    assert _column_sum_launches(stage, call) == cfg["n_layers"] * (1 if size == "together" else 4)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    torch.cuda.synchronize()
    for _ in range(3):
        out.fill_(3.0)
        dx.fill_(3.0)
        for g in grads:
            for v in g.values():
                v.fill_(3.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(ref, snapshot()):
            assert torch.equal(a, b)
        call()                                   # eager work between replays
        torch.cuda.synchronize()
    del graph
    stage.close()


@pytest.mark.parametrize("size", ["together", "side stream"])
def test_back_to_back_calls_on_a_caller_stream_without_host_synchronisation(size):
    """The bias-gradient column sums run on a stream of the stage's own and are joined before a call returns control of
    the caller's stream: calls enqueued back to back on a stream of the caller's, with nothing in between, leave the same
    bits as one call followed by a synchronisation, and buffers the caller overwrites right behind a call are not read
    late."""
    cfg, params, xs, dys, lo = _overlap_case(size)
    from helpers import params_to_dev, stream_from_seqs, zero_grads_like
    d = cfg["d_model"]
    stage = ds.Stage(ds.DS_MODEL_GPT, ds.DS_DTYPE_BF16, cfg["n_layers"], d, cfg["n_heads"], cfg["d_ff"],
                     max_rows=lo.total_rows, max_seqs=lo.n_seq)
    w = params_to_dev(params, torch.bfloat16)
    grads = zero_grads_like(w)
    x = stream_from_seqs(xs, lo, d, torch.bfloat16, 0.0)
    dy = stream_from_seqs(dys, lo, d, torch.bfloat16, 0.0)
    out, dx = torch.empty_like(x), torch.empty_like(x)
    ds.stage_fwd_bwd(stage, lo, w, x, dy, out, dx, grads, accumulate=False)
    torch.cuda.synchronize()
    ref = [out.clone(), dx.clone()] + [g[k].clone() for g in grads for k in g]
    assert _column_sum_launches(stage, lambda: ds.stage_fwd_bwd(stage, lo, w, x, dy, out, dx, grads, accumulate=False)) == \
        cfg["n_layers"] * (1 if size == "together" else 4)
    dy_copy = dy.clone()
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(st):
        for _ in range(4):
            ds.stage_fwd_bwd(stage, lo, w, x, dy, out, dx, grads, accumulate=False, stream=st.cuda_stream)
            dy.fill_(float("nan"))                  # the caller reuses its gradient buffer right behind the call ...
            dy.copy_(dy_copy)                       # ... and refills it for the next one, all in stream order
    torch.cuda.synchronize()
    for a, b in zip(ref, [out, dx] + [g[k] for g in grads for k in g]):
        assert torch.equal(a, b)
    stage.close()


@pytest.mark.parametrize("d_ff,rows", [(1024, [1, 127, 128, 129, 256, 257, 385]), (5632, [129, 257, 384, 385, 641, 769]),
                                       (8192, [2089, 2305])])
def test_bias_gradient_from_partial_column_sums(d_ff, rows):
    """The bias gradient of the MLP's first projection is summed from one partial row per 128 rows, of which an odd count is
    padded to an even one: even and odd counts, full and ragged last tiles, after a larger call with gradients a thousand
    times as large has filled the partial rows.  Every gradient is the one a fresh stage gives, bit for bit, and b_1 is
    the oracle's."""
    from helpers import params_to_dev
    cfg = dict(n_layers=1, d_model=256, n_heads=4, d_ff=d_ff)
    params = wl.draw_params(wl.GPT_KEYS, 1, 256, d_ff, seed=3, bf16=True)

    def case(r, scale=1.0):
        lens = np.array([r], np.int32)
        xs = wl.draw_embedded_tokens(lens, 256, seed=r, bf16=True)
        dys = [scale * y for y in wl.draw_rows(lens, 256, seed=r, tag=5, bf16=True)]
        return ds.ds_layout_from_cuts(lens, [0, 1]), xs, dys

    top = 2 * max(rows)
    used = ds.Stage(ds.DS_MODEL_GPT, ds.DS_DTYPE_BF16, 1, 256, 4, d_ff, max_rows=top, max_seqs=4)
    for r in rows:
        lo, xs, dys = case(top, 1000.0)
        run_gpt_stage(lo, cfg, params, xs, dys, ds.DS_DTYPE_BF16, stage=used)
        lo, xs, dys = case(r)
        got = run_gpt_stage(lo, cfg, params, xs, dys, ds.DS_DTYPE_BF16, stage=used)
        fresh = ds.Stage(ds.DS_MODEL_GPT, ds.DS_DTYPE_BF16, 1, 256, 4, d_ff, max_rows=top, max_seqs=4)
        want = run_gpt_stage(lo, cfg, params, xs, dys, ds.DS_DTYPE_BF16, stage=fresh)
        fresh.close()
        for k, v in want[2][0].items():
            assert np.array_equal(got[2][0][k], v), (r, k)
        ref = ost.gpt_stage_fwd_bwd(xs, dys, params, 4)
        check(got[2][0]["b_1"], ref[2][0]["b_1"], TOL[ds.DS_DTYPE_BF16], "b_1 %d" % r)
    used.close()


@pytest.mark.parametrize("rows", [641, 768, 897, 1024])
def test_bias_gradient_from_column_sums_of_lower_tiles(rows):
    """The same where the product is one round of 128 x 256 tiles, which give one partial row each: even and odd counts of tile rows."""
    lens = np.array([rows], np.int32)
    params = wl.draw_params(wl.GPT_KEYS, 1, 256, 8192, seed=4, bf16=True)
    xs = wl.draw_embedded_tokens(lens, 256, seed=rows, bf16=True)
    dys = wl.draw_rows(lens, 256, seed=rows, tag=5, bf16=True)
    lo = ds.ds_layout_from_cuts(lens, [0, 1])
    cfg = dict(n_layers=1, d_model=256, n_heads=4, d_ff=8192)
    stage = ds.Stage(ds.DS_MODEL_GPT, ds.DS_DTYPE_BF16, 1, 256, 4, 8192, max_rows=1024, max_seqs=4)
    run_gpt_stage(lo, cfg, params, xs, [1000.0 * y for y in dys], ds.DS_DTYPE_BF16, stage=stage)     # (fills the partial rows)
    got = run_gpt_stage(lo, cfg, params, xs, dys, ds.DS_DTYPE_BF16, stage=stage)
    stage.close()
    ref = ost.gpt_stage_fwd_bwd(xs, dys, params, 4)
    check(got[2][0]["b_1"], ref[2][0]["b_1"], TOL[ds.DS_DTYPE_BF16], "b_1 %d" % rows)


# d, d_ff, tokens -> the tile that the weight gradients of a layer go out with, in one launch: 64 x 64; 128 x 64; 128 x 128 one
# per CU; two per CU; 256 x 256; 256 x 256 with split contractions; fp32: ragged tiles of 64 x 128, whole and split.  Token counts that
# are no multiple of a K tile.
@pytest.mark.parametrize("d,F,tokens,code", [(256, 1024, 33, ds.DS_DTYPE_BF16), (256, 2048, 301, ds.DS_DTYPE_BF16),
                                             (512, 2048, 1001, ds.DS_DTYPE_BF16), (768, 3072, 1501, ds.DS_DTYPE_BF16),
                                             (1024, 4096, 701, ds.DS_DTYPE_BF16), (512, 1536, 9001, ds.DS_DTYPE_BF16),
                                             (192, 328, 77, ds.DS_DTYPE_F32), (192, 328, 1301, ds.DS_DTYPE_F32)])
def test_weight_gradients_of_a_layer_in_one_launch(d, F, tokens, code):
    """Every weight gradient against the oracle, overwritten (what was there before is gone) and then added to."""
    cfg = dict(d_model=d, d_ff=F, n_heads=d // 64, n_layers=1)
    rng = np.random.default_rng(d + tokens)
    lens = []
    while sum(lens) < tokens:
        lens.append(int(min(rng.integers(1, 300), tokens - sum(lens))))
    lens = np.asarray(lens)
    bf16 = code == ds.DS_DTYPE_BF16
    params = wl.draw_params(wl.GPT_KEYS, 1, d, F, seed=4, bf16=bf16)
    xs, dys = wl.draw_rows(lens, d, seed=4, tag=3, bf16=bf16), wl.draw_rows(lens, d, seed=4, tag=5, bf16=bf16)
    lo = ds.ds_layout_from_cuts(lens, list(range(len(lens) + 1)))
    ref = ost.gpt_stage_fwd_bwd(xs, dys, params, cfg["n_heads"])
    grads = [{k: torch.full(v.shape, 3.0, dtype=torch.float32, device="cuda:0") for k, v in params[0].items()}]
    _compare("%d %d %d" % (d, F, tokens), run_gpt_stage(lo, cfg, params, xs, dys, code, grads=grads), ref, TOL[code])
    twice = run_gpt_stage(lo, cfg, params, xs, dys, code, grads=grads, accumulate=True)[2]
    for k, v in ref[2][0].items():
        check(twice[0][k], 2 * v, TOL[code], k)


# rows up to and beyond what one work-group walks (512), row lanes with and without a row, narrow and wide norm kernels
@pytest.mark.parametrize("d,rows", [(256, 5), (256, 512), (256, 513), (768, 1100), (1536, 129)])
@pytest.mark.parametrize("dtype_code", [ds.DS_DTYPE_F32, ds.DS_DTYPE_BF16])
def test_bias_and_norm_gradients_summed_together(dtype_code, d, rows):
    """Bias and norm gradients of a layer, overwritten and then added to, against the oracle."""
    bf16, tol = dtype_code == ds.DS_DTYPE_BF16, TOL[dtype_code]
    cfg = dict(d_model=d, d_ff=256, n_heads=d // 64, n_layers=1)
    lens = np.asarray([5] if rows == 5 else [rows - 100, 99, 1])
    params = wl.draw_params(wl.GPT_KEYS, 1, d, 256, seed=6, bf16=bf16)
    xs, dys = wl.draw_rows(lens, d, seed=6, tag=3, bf16=bf16), wl.draw_rows(lens, d, seed=6, tag=5, bf16=bf16)
    lo = ds.ds_layout_from_cuts(lens, [0, len(lens)] if rows == 512 else list(range(len(lens) + 1)))
    ref = ost.gpt_stage_fwd_bwd(xs, dys, params, cfg["n_heads"])[2][0]
    grads = [{k: torch.full(v.shape, 3.0, dtype=torch.float32, device="cuda:0") for k, v in params[0].items()}]
    once = run_gpt_stage(lo, cfg, params, xs, dys, dtype_code, grads=grads)[2][0]
    twice = run_gpt_stage(lo, cfg, params, xs, dys, dtype_code, grads=grads, accumulate=True)[2][0]
    for k in ("b_qkv", "b_o", "b_1", "b_2", "ln1_g", "ln1_b", "ln2_g", "ln2_b"):
        check(once[k], ref[k], tol, k)
        check(twice[k], 2 * ref[k], tol, k)


@pytest.mark.parametrize("dtype_code", [ds.DS_DTYPE_F32, ds.DS_DTYPE_BF16])
def test_launch_count_of_a_first_and_a_later_call(dtype_code):
    """The first call with a layout makes both attention work lists in one launch more (bf16) and clears the padding rows of
    the attention buffers in another; later calls do neither."""
    cfg, lens, params, xs, dys = _small_case(True, n_seq=6)
    for cuts, first_more in (([0, 6], 1), (list(range(7)), 0)):           # padded to the longest; no padding
        lo = ds.ds_layout_from_cuts(lens, cuts)
        stage = ds.Stage(ds.DS_MODEL_GPT, dtype_code, cfg["n_layers"], cfg["d_model"], cfg["n_heads"], cfg["d_ff"],
                         max_rows=lo.total_rows, max_seqs=8)
        n = []
        for _ in range(3):
            run_gpt_stage(lo, cfg, params, xs, dys, dtype_code, stage=stage)
            n.append(stage.last_launch_count())
        stage.close()
        assert n[1] == n[2] and n[0] - n[1] == first_more + (dtype_code == ds.DS_DTYPE_BF16), (cuts, n)


# one layer without padding rows: the gradient that the layer hands down overwrites the one it was given.  Rows up to and beyond
# what one work-group walks, and beyond what is summed in one launch.
@pytest.mark.parametrize("dtype_code,d,rows", [(ds.DS_DTYPE_F32, 256, 300), (ds.DS_DTYPE_BF16, 256, 300), (ds.DS_DTYPE_BF16, 256, 900),
                                               (ds.DS_DTYPE_BF16, 1024, 10500)])
def test_gradient_returned_in_place(dtype_code, d, rows):
    """grad_in is grad_out: every gradient is the oracle's."""
    from helpers import params_to_dev, seqs_from_stream, stream_from_seqs, tdtype, to_np, zero_grads_like
    bf16, tol, F, h = dtype_code == ds.DS_DTYPE_BF16, TOL[dtype_code], 2 * d, d // 64
    lens = np.asarray([rows - rows // 3 - 1, rows // 3, 1] if rows < 1000 else [250] * (rows // 250))
    params = wl.draw_params(wl.GPT_KEYS, 1, d, F, seed=8, bf16=bf16)
    xs, dys = wl.draw_rows(lens, d, seed=8, tag=3, bf16=bf16), wl.draw_rows(lens, d, seed=8, tag=5, bf16=bf16)
    lo = ds.ds_layout_from_cuts(lens, list(range(len(lens) + 1)))
    assert lo.total_rows == lo.total_tokens
    _, r_dx, r_g = ost.gpt_stage_fwd_bwd(xs, dys, params, h)
    w = params_to_dev(params, tdtype(dtype_code))
    g = zero_grads_like(w)
    x, grad = (stream_from_seqs(v, lo, d, tdtype(dtype_code)) for v in (xs, dys))
    stage = ds.Stage(ds.DS_MODEL_GPT, dtype_code, 1, d, h, F, max_rows=lo.total_rows, max_seqs=lo.n_seq)
    ds.stage_fwd_bwd(stage, lo, w, x, grad, torch.empty_like(x), grad, g)
    torch.cuda.synchronize()
    check_seqs(seqs_from_stream(grad, lo)[0], r_dx, tol, "grad_in")
    for k, v in r_g[0].items():
        check(to_np(g[0][k]), v, tol, k)
    stage.close()


@pytest.mark.parametrize("cuts", [[0, 4, 9], list(range(10))])              # with and without padding rows
@pytest.mark.parametrize("dtype_code", [ds.DS_DTYPE_F32, ds.DS_DTYPE_BF16])
def test_outputs_as_their_own_gradient(dtype_code, cuts):
    """grad_out is act_out (the gradient of half the sum of squares): the backward pass starts from this call's outputs."""
    from helpers import params_to_dev, seqs_from_stream, stream_from_seqs, tdtype, to_np, zero_grads_like
    bf16, tol, d, F, h = dtype_code == ds.DS_DTYPE_BF16, TOL[dtype_code], 256, 512, 4
    lens = np.asarray([30, 7, 64, 1, 100, 33, 65, 12, 90])
    params = wl.draw_params(wl.GPT_KEYS, 2, d, F, seed=9, bf16=bf16)
    xs = wl.draw_rows(lens, d, seed=9, tag=3, bf16=bf16)
    lo = ds.ds_layout_from_cuts(lens, cuts)
    outs = ost.gpt_stage_fwd_bwd(xs, xs, params, h)[0]
    _, r_dx, r_g = ost.gpt_stage_fwd_bwd(xs, [wl.to_bf16_grid(o) if bf16 else o for o in outs], params, h)
    dt = tdtype(dtype_code)
    w = params_to_dev(params, dt)
    g = zero_grads_like(w)
    x = stream_from_seqs(xs, lo, d, dt)
    y, dx = torch.full_like(x, float("nan")), torch.empty_like(x)
    stage = ds.Stage(ds.DS_MODEL_GPT, dtype_code, 2, d, h, F, max_rows=lo.total_rows, max_seqs=lo.n_seq)
    ds.stage_fwd_bwd(stage, lo, w, x, y, y, dx, g)
    torch.cuda.synchronize()
    check_seqs(seqs_from_stream(y, lo)[0], outs, tol, "act_out")
    check_seqs(seqs_from_stream(dx, lo)[0], r_dx, tol, "grad_in")
    for layer, ref in zip(g, r_g):
        for k, v in ref.items():
            check(to_np(layer[k]), v, tol, k)
    stage.close()


@pytest.mark.parametrize("dtype_code", [ds.DS_DTYPE_F32, ds.DS_DTYPE_BF16])
def test_parameters_of_a_layer_that_share_a_gradient(dtype_code):
    """b_o and b_2, the gains and the biases of both norms, w_qkv and w_1 (of the same shape): summed in one buffer each."""
    from helpers import params_to_dev, stream_from_seqs, tdtype, to_np
    bf16, tol, d, F, h = dtype_code == ds.DS_DTYPE_BF16, TOL[dtype_code], 256, 768, 4
    lens = np.asarray([30, 7, 164, 1, 100, 333])
    params = wl.draw_params(wl.GPT_KEYS, 1, d, F, seed=10, bf16=bf16)
    xs, dys = wl.draw_rows(lens, d, seed=10, tag=3, bf16=bf16), wl.draw_rows(lens, d, seed=10, tag=5, bf16=bf16)
    lo = ds.ds_layout_from_cuts(lens, list(range(len(lens) + 1)))
    ref = ost.gpt_stage_fwd_bwd(xs, dys, params, h)[2][0]
    dt = tdtype(dtype_code)
    w = params_to_dev(params, dt)
    x, dy = stream_from_seqs(xs, lo, d, dt), stream_from_seqs(dys, lo, d, dt)
    stage = ds.Stage(ds.DS_MODEL_GPT, dtype_code, 1, d, h, F, max_rows=lo.total_rows, max_seqs=lo.n_seq)
    for _ in range(3):
        g = {k: torch.zeros(v.shape, dtype=torch.float32, device="cuda:0") for k, v in w[0].items()}
        for a, b in (("b_2", "b_o"), ("ln2_g", "ln1_g"), ("ln2_b", "ln1_b"), ("w_1", "w_qkv")):
            g[b] = g[a]
        ds.stage_fwd_bwd(stage, lo, w, x, dy, torch.empty_like(x), torch.empty_like(x), [g], accumulate=True)
        torch.cuda.synchronize()
        for a, b in (("b_2", "b_o"), ("ln2_g", "ln1_g"), ("ln2_b", "ln1_b"), ("w_1", "w_qkv")):
            check(to_np(g[a]), ref[a] + ref[b], tol, a)
        for k in ("w_2", "w_o", "b_1", "b_qkv"):
            check(to_np(g[k]), ref[k], tol, k)
    stage.close()


def test_fp32_layer_of_more_than_65535_gradient_tiles():
    """d = 4096, d_ff = 57 600: the weight gradients of a layer are 65 984 tiles of 64 x 128.  Against the same layer in 64 bits."""
    d, F, h, lens = 4096, 57600, 32, [5, 12]
    assert (2 * d * F + 4 * d * d) // (64 * 128) > 65535
    gen = torch.Generator(device="cuda:0").manual_seed(12)

    def rnd(*shape, scale=1.0):
        return torch.randn(*shape, device="cuda:0", generator=gen) * scale

    shapes = dict(w_qkv=(d, 3 * d), b_qkv=(3 * d,), w_o=(d, d), w_1=(d, F), b_1=(F,), w_2=(F, d))
    w = {k: rnd(*shapes.get(k, (d,)), scale=0.02) for k in wl.GPT_KEYS}
    w["ln1_g"] += 1
    w["ln2_g"] += 1
    x, dy = rnd(sum(lens), d), rnd(sum(lens), d)
    g = {k: torch.full(v.shape, 3.0, device="cuda:0") for k, v in w.items()}
    lo = ds.ds_layout_from_cuts(np.asarray(lens), [0, 1, 2])
    rows = [slice(int(r), int(r) + int(l)) for r, l in zip(lo.seq_row, lo.seq_len)]
    out, dx = torch.empty_like(x), torch.empty_like(x)
    stage = ds.Stage(ds.DS_MODEL_GPT, ds.DS_DTYPE_F32, 1, d, h, F, max_rows=sum(lens), max_seqs=2)
    ds.stage_fwd_bwd(stage, lo, [w], x, dy, out, dx, [g])
    torch.cuda.synchronize()
    stage.close()

    p = {k: v.double().requires_grad_() for k, v in w.items()}
    x64 = x.double().requires_grad_()
    qkv = torch.nn.functional.layer_norm(x64, (d,), p["ln1_g"], p["ln1_b"], 1e-5) @ p["w_qkv"] + p["b_qkv"]
    heads = []
    for r in rows:
        q, k, v = (t.view(-1, h, d // h).transpose(0, 1).contiguous() for t in qkv[r].split(d, dim=1))
        s = q @ k.transpose(1, 2).contiguous() / (d // h) ** 0.5
        s = s.masked_fill(torch.ones_like(s, dtype=torch.bool).triu(1), float("-inf"))
        heads.append((s.softmax(-1) @ v).transpose(0, 1).reshape(-1, d))
    order = sorted(range(len(rows)), key=lambda i: rows[i].start)
    x1 = x64 + torch.cat([heads[i] for i in order]) @ p["w_o"] + p["b_o"]
    z = torch.nn.functional.layer_norm(x1, (d,), p["ln2_g"], p["ln2_b"], 1e-5) @ p["w_1"] + p["b_1"]
    y = x1 + torch.nn.functional.gelu(z, approximate="tanh") @ p["w_2"] + p["b_2"]
    y.backward(dy.double())
    for k, a, b in [("act_out", out, y.detach()), ("grad_in", dx, x64.grad)] + [(k, g[k], p[k].grad) for k in w]:
        dev = (a.double() - b).abs()
        assert float(dev.norm() / b.norm()) <= TOL[ds.DS_DTYPE_F32], k
        assert float((dev / (8 * b.square().mean().sqrt() + b.abs())).max()) <= TOL[ds.DS_DTYPE_F32], k


@pytest.mark.parametrize("rows,launches", [(10_900, 1), (11_500, 4)])
def test_fp32_column_sums_together_and_on_the_side_stream(rows, launches):
    """d = 256, d_ff = 1024 in fp32: the summed tensors take 9 216 bytes a row, below and above 96 MiB.  Every bias and norm gradient is
    the oracle's."""
    from helpers import params_to_dev, stream_from_seqs, to_np
    d, F = 256, 1024
    lens = np.asarray([100] * (rows // 100))
    params = wl.draw_params(wl.GPT_KEYS, 1, d, F, seed=14)
    xs, dys = wl.draw_rows(lens, d, seed=14, tag=3), wl.draw_rows(lens, d, seed=14, tag=5)
    lo = ds.ds_layout_from_cuts(lens, list(range(len(lens) + 1)))
    ref = ost.gpt_stage_fwd_bwd(xs, dys, params, 4)[2][0]
    w = params_to_dev(params, torch.float32)
    x, dy = stream_from_seqs(xs, lo, d, torch.float32), stream_from_seqs(dys, lo, d, torch.float32)
    g = [{k: torch.full(v.shape, 3.0, device="cuda:0") for k, v in w[0].items()}]
    stage = ds.Stage(ds.DS_MODEL_GPT, ds.DS_DTYPE_F32, 1, d, 4, F, max_rows=rows, max_seqs=len(lens))
    out, dx = torch.empty_like(x), torch.empty_like(x)
    assert _column_sum_launches(stage, lambda: ds.stage_fwd_bwd(stage, lo, w, x, dy, out, dx, g)) == launches
    for k in ("b_qkv", "b_o", "b_1", "b_2", "ln1_g", "ln1_b", "ln2_g", "ln2_b"):
        check(to_np(g[0][k]), ref[k], TOL[ds.DS_DTYPE_F32], k)
    stage.close()
