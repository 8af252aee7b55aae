"""GPU parity of the building-block kernels, each called through the C ABI and compared with its plain
definition (numpy float64 on the same rounded inputs, or the oracle's per-sequence attention / norm
functions).  Every comparison bounds the normwise relative error by the stated tolerance AND every
single element's deviation by tolerance x (8 x rms(reference) + |reference element|) (helpers.both_err).  Sizes span several
tiles and a ragged tail."""
import numpy as np
import pytest
import torch

from oracle import stage as ost
from paper_2311_10418_amd import binding as ds
from paper_2311_10418_amd import workload as wl
from helpers import DEV, both_err, gemm_launches, to_dev, to_np

pytestmark = pytest.mark.gpu

BF, F32 = torch.bfloat16, torch.float32
TOL = {BF: 2e-2, F32: 1e-4}


def _rnd(rng, shape, dt, scale=1.0):
    a = (rng.standard_normal(shape) * scale).astype(np.float32)
    if dt == BF:
        a = wl.to_bf16_grid(a)
    return a


@pytest.mark.parametrize("dt,force", [(F32, True), (BF, True), (BF, False)])
@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, False)])
def test_gemm_plain(dt, force, ta, tb):
    rng = np.random.default_rng(1)
    if ta:
        M, N, K = 512, 768, 1000 + 37          # weight-gradient shape: ragged contraction over tokens
    else:
        M, N, K = 1000 + 37, 512, 320           # ragged M, several K steps
    A = _rnd(rng, (K, M) if ta else (M, K), dt)
    B = _rnd(rng, (N, K) if tb else (K, N), dt)
    bias = _rnd(rng, (N,), dt)
    ref = (A.T if ta else A).astype(np.float64) @ (B.T if tb else B).astype(np.float64) + bias
    dA, dB, db = to_dev(A, dt), to_dev(B, dt), to_dev(bias, dt)
    Cd = torch.zeros((M, N), dtype=dt, device=DEV)
    ds.ds_gemm(dA, dB, Cd, M, N, K, trans_a=ta, trans_b=tb, bias=db, force_generic=force)
    torch.cuda.synchronize()
    # bf16 output rounding: 2^-9 relative per element
    assert both_err(to_np(Cd), ref) <= (4e-3 if dt == BF else 1e-5)


@pytest.mark.parametrize("dt,force", [(F32, True), (BF, False)])
def test_gemm_epilogues(dt, force):
    rng = np.random.default_rng(2)
    M, N, K = 700, 256, 128
    A, B = _rnd(rng, (M, K), dt), _rnd(rng, (K, N), dt, 0.1)
    bias, R = _rnd(rng, (N,), dt), _rnd(rng, (M, N), dt)
    R2 = _rnd(rng, (M, N), dt)
    valid = np.where(rng.random(M) < 0.8, 1, -1).astype(np.int32)
    acc = A.astype(np.float64) @ B.astype(np.float64)
    dA, dB, db, dR, dR2 = (to_dev(x, dt) for x in (A, B, bias, R, R2))
    dvalid = torch.from_numpy(valid).to(DEV)
    tol = 6e-3 if dt == BF else 1e-5

    def run(epi, **kw):
        c = torch.zeros((M, N), dtype=dt, device=DEV)
        c2 = torch.zeros((M, N), dtype=dt, device=DEV)
        ds.ds_gemm(dA, dB, c, M, N, K, epilogue=epi, C2=c2, force_generic=force, **kw)
        torch.cuda.synchronize()
        return to_np(c), to_np(c2)

    z, a = run(ds.DS_EPI_GELU, bias=db)
    assert both_err(z, acc + bias) <= tol and both_err(a, ost.gelu(acc + bias)) <= tol
    c, _ = run(ds.DS_EPI_RESID, bias=db, R=dR, row_valid=dvalid)
    ref = (acc + bias + R) * (valid[:, None] >= 0)
    assert both_err(c, ref) <= tol and np.all(c[valid < 0] == 0)
    c, _ = run(ds.DS_EPI_DGELU, R=dR)
    assert both_err(c, acc * ost.gelu_grad(R.astype(np.float64))) <= tol
    gd, a = run(ds.DS_EPI_GELU_D, bias=db)                # derivative kept instead of the pre-activation
    assert both_err(gd, ost.gelu_grad(acc + bias)) <= tol and both_err(a, ost.gelu(acc + bias)) <= tol
    c, _ = run(ds.DS_EPI_MULR, R=dR)
    assert both_err(c, acc * R) <= tol
    zu, h = run(ds.DS_EPI_GATE, R=dR)
    assert both_err(zu, acc) <= tol and both_err(h, ost.gelu(R.astype(np.float64)) * acc) <= tol
    g1, g2 = run(ds.DS_EPI_DGATE, R=dR, R2=dR2)
    assert both_err(g1, acc * R2 * ost.gelu_grad(R.astype(np.float64))) <= tol
    assert both_err(g2, acc * ost.gelu(R.astype(np.float64))) <= tol


# 256 x 256 tiles for whole rounds over 256 compute units and other tiles for the rows behind them, from one to a tile and a half
# (one launch at K = 64)
@pytest.mark.parametrize("K", [64, 512])
@pytest.mark.parametrize("M", [8193, 8289, 8192 + 385])
def test_gemm_rows_behind_whole_rounds(M, K):
    rng = np.random.default_rng(M)
    N, tol = 2048, 6e-3
    A, B = _rnd(rng, (M, K), BF), _rnd(rng, (N, K), BF, 0.1)
    bias, R, R2 = _rnd(rng, (N,), BF), _rnd(rng, (M, N), BF), _rnd(rng, (M, N), BF)
    valid = np.where(rng.random(M) < 0.8, 1, -1).astype(np.int32)
    acc = A.astype(np.float64) @ B.T.astype(np.float64)
    dA, dB, db, dR, dR2 = (to_dev(x, BF) for x in (A, B, bias, R, R2))
    ws = torch.zeros(1 << 22, dtype=F32, device=DEV)

    def run(epi, dt=BF, **kw):
        c, c2 = torch.full((M, N), 3.0, dtype=dt, device=DEV), torch.full((M, N), 3.0, dtype=BF, device=DEV)
        ds.ds_gemm(dA, dB, c, M, N, K, trans_b=True, epilogue=epi, C2=c2, workspace=ws, **kw)
        torch.cuda.synchronize()
        return to_np(c), to_np(c2)

    assert both_err(run(ds.DS_EPI_NONE, bias=db)[0], acc + bias) <= tol
    c, _ = run(ds.DS_EPI_RESID, bias=db, R=dR, row_valid=torch.from_numpy(valid).to(DEV))
    assert both_err(c, (acc + bias + R) * (valid[:, None] >= 0)) <= tol and np.all(c[valid < 0] == 0)
    c, c2 = run(ds.DS_EPI_GELU_D, bias=db)
    assert both_err(c, ost.gelu_grad(acc + bias)) <= tol and both_err(c2, ost.gelu(acc + bias)) <= tol
    c, c2 = run(ds.DS_EPI_DGATE, R=dR, R2=dR2)
    assert both_err(c, acc * R2 * ost.gelu_grad(R.astype(np.float64))) <= tol and both_err(c2, acc * ost.gelu(R.astype(np.float64))) <= tol
    assert both_err(run(ds.DS_EPI_ACC32, dt=F32, accumulate=True)[0], acc + 3.0) <= 1e-5


@pytest.mark.parametrize("dt,force", [(F32, True), (BF, False)])
@pytest.mark.parametrize("M,N,K", [(256, 512, 3000 + 11), (768, 512, 1000 + 37), (512, 256, 31), (256, 256, 64)])
def test_gemm_weight_gradient_accumulates_in_fp32(dt, force, M, N, K):
    rng = np.random.default_rng(3)
    X, dY = _rnd(rng, (K, M), dt), _rnd(rng, (K, N), dt)
    ref = X.astype(np.float64).T @ dY.astype(np.float64)
    dX, ddY = to_dev(X, dt), to_dev(dY, dt)
    Cd = torch.full((M, N), 3.0, dtype=F32, device=DEV)
    ds.ds_gemm(dX, ddY, Cd, M, N, K, trans_a=True, epilogue=ds.DS_EPI_ACC32, accumulate=False, force_generic=force)
    ds.ds_gemm(dX, ddY, Cd, M, N, K, trans_a=True, epilogue=ds.DS_EPI_ACC32, accumulate=True, force_generic=force)
    torch.cuda.synchronize()
    assert both_err(to_np(Cd), 2 * ref) <= 1e-5


def _varlen_case(rng, lens, h, hd, dt, cross_lens=None):
    d = h * hd
    T = int(sum(lens)) + 5                       # 5 trailing rows never touched
    gap = 3
    rows, r = [], 0
    for l in lens:
        rows.append(r)
        r += l + gap                              # gaps play the role of padding rows
    T = r + 2
    qkv = _rnd(rng, (T, 3 * d), dt)
    d_o = _rnd(rng, (T, d), dt)
    return d, T, np.asarray(rows, np.int32), qkv, d_o


@pytest.mark.parametrize("dt,force", [(F32, True), (BF, True), (BF, False)])
@pytest.mark.parametrize("hd,causal", [(64, True), (128, True), (64, False), (128, False)])
def test_attention_self(dt, force, hd, causal):
    rng = np.random.default_rng(4)
    h = 2
    # lengths on both sides of every tile boundary (64-row steps, 128-row blocks), a few long ones for the middle steps
    lens = [1, 7, 63, 64, 65, 127, 128, 129, 130, 191, 192, 193, 200, 256, 257, 333, 700]
    d, T, rows, qkv, d_o = _varlen_case(rng, lens, h, hd, dt)
    dq = to_dev(qkv, dt)
    o = torch.zeros((T, d), dtype=dt, device=DEV)
    lse = torch.zeros((h, T), dtype=F32, device=DEV)
    delta = torch.zeros((h, T), dtype=F32, device=DEV)
    dqkv = torch.zeros((T, 3 * d), dtype=dt, device=DEV)
    ddo = to_dev(d_o, dt)
    # the sequence table is handed over in an arbitrary order: nothing may depend on ascending rows
    order = rng.permutation(len(lens))
    t_rows = torch.from_numpy(np.ascontiguousarray(rows[order])).to(DEV)
    t_lens = torch.tensor([lens[i] for i in order], dtype=torch.int32, device=DEV)
    scratch = torch.zeros(ds.ds_attention_scratch_bytes(h, hd, T, T, len(lens)), dtype=torch.uint8, device=DEV)
    es = dq.element_size()
    base = dq.data_ptr()
    ds.ds_attention_fwd(base, base + d * es, base + 2 * d * es, o, lse, t_rows, t_lens, t_rows, t_lens, h, hd, causal,
                        max(lens), max(lens), 3 * d, 3 * d, 3 * d, d, T, scratch=scratch, force_generic=force)
    gb = dqkv.data_ptr()
    ds.ds_attention_bwd(base, base + d * es, base + 2 * d * es, o, ddo, lse, delta, gb, gb + d * es, gb + 2 * d * es,
                        t_rows, t_lens, t_rows, t_lens, h, hd, causal, max(lens), max(lens), 3 * d, 3 * d, 3 * d, d, T,
                        scratch=scratch, force_generic=force)
    torch.cuda.synchronize()
    o_np, g_np, lse_np = to_np(o), to_np(dqkv), to_np(lse)
    tol = TOL[dt]
    touched = np.zeros(T, dtype=bool)
    for r0, l in zip(rows, lens):
        x = qkv[r0:r0 + l].astype(np.float64)
        q, k, v = x[:, :d], x[:, d:2 * d], x[:, 2 * d:]
        ref_o, cache = ost.attention_fwd(q, k, v, h, causal)
        # the backward kernels consume the ROUNDED forward output, as the oracle's gradient of the exact one
        rq, rk, rv = ost.attention_bwd(d_o[r0:r0 + l].astype(np.float64), cache)
        assert both_err(o_np[r0:r0 + l], ref_o) <= tol, (l, "o")
        assert both_err(g_np[r0:r0 + l, :d], rq) <= tol, (l, "dq")
        assert both_err(g_np[r0:r0 + l, d:2 * d], rk) <= tol, (l, "dk")
        assert both_err(g_np[r0:r0 + l, 2 * d:], rv) <= tol, (l, "dv")
        # log-sum-exp of the scaled scores, head 0, last row
        s = (q[-1, :hd] @ k[:, :hd].T) / np.sqrt(hd)      # the last query sees every key in both mask kinds
        assert abs(lse_np[0, r0 + l - 1] - np.log(np.exp(s - s.max()).sum()) - s.max()) <= 2e-2
        touched[r0:r0 + l] = True
    assert np.all(o_np[~touched] == 0) and np.all(g_np[~touched] == 0)      # padding rows are never written


@pytest.mark.parametrize("dt,force", [(F32, True), (BF, False)])
def test_attention_cross(dt, force):
    rng = np.random.default_rng(5)
    h, hd = 2, 64
    d = h * hd
    ql, kl = [3, 40, 129, 200, 64], [70, 5, 260, 700, 1000]      # the last two: many key steps / many query steps per block
    qr = np.array([0, 5, 50, 190, 400], np.int32)
    kr = np.array([2, 80, 90, 360, 1070], np.int32)
    Tq, Tk = 470, 2080
    q = _rnd(rng, (Tq, d), dt)
    kv = _rnd(rng, (Tk, 2 * d), dt)
    d_o = _rnd(rng, (Tq, d), dt)
    tq, tkv, tdo = to_dev(q, dt), to_dev(kv, dt), to_dev(d_o, dt)
    o = torch.zeros((Tq, d), dtype=dt, device=DEV)
    lse = torch.zeros((h, Tq), dtype=F32, device=DEV)
    delta = torch.zeros((h, Tq), dtype=F32, device=DEV)
    dq = torch.zeros((Tq, d), dtype=dt, device=DEV)
    dkv = torch.zeros((Tk, 2 * d), dtype=dt, device=DEV)
    es = tq.element_size()
    i32 = lambda a: torch.tensor(np.asarray(a), dtype=torch.int32, device=DEV)
    t_qr, t_ql, t_kr, t_kl = i32(qr), i32(ql), i32(kr), i32(kl)
    kb = tkv.data_ptr()
    scratch = torch.zeros(ds.ds_attention_scratch_bytes(h, hd, Tq, Tk, len(ql)), dtype=torch.uint8, device=DEV)
    ds.ds_attention_fwd(tq, kb, kb + d * es, o, lse, t_qr, t_ql, t_kr, t_kl, h, hd, False, max(ql), max(kl),
                        d, 2 * d, 2 * d, d, Tq, k_total_rows=Tk, scratch=scratch, force_generic=force)
    gb = dkv.data_ptr()
    ds.ds_attention_bwd(tq, kb, kb + d * es, o, tdo, lse, delta, dq, gb, gb + d * es, t_qr, t_ql, t_kr, t_kl, h, hd, False,
                        max(ql), max(kl), d, 2 * d, 2 * d, d, Tq, k_total_rows=Tk, scratch=scratch, force_generic=force)
    torch.cuda.synchronize()
    tol = TOL[dt]
    for i in range(len(ql)):
        qq = q[qr[i]:qr[i] + ql[i]].astype(np.float64)
        kk = kv[kr[i]:kr[i] + kl[i], :d].astype(np.float64)
        vv = kv[kr[i]:kr[i] + kl[i], d:].astype(np.float64)
        ref_o, cache = ost.attention_fwd(qq, kk, vv, h, False)
        rq, rk, rv = ost.attention_bwd(d_o[qr[i]:qr[i] + ql[i]].astype(np.float64), cache)
        assert both_err(to_np(o)[qr[i]:qr[i] + ql[i]], ref_o) <= tol
        assert both_err(to_np(dq)[qr[i]:qr[i] + ql[i]], rq) <= tol
        assert both_err(to_np(dkv)[kr[i]:kr[i] + kl[i], :d], rk) <= tol
        assert both_err(to_np(dkv)[kr[i]:kr[i] + kl[i], d:], rv) <= tol


@pytest.mark.parametrize("dt,force", [(F32, True), (BF, True), (BF, False)])
def test_attention_empty_sequences(dt, force):
    """q_len = 0: the sequence is skipped.  k_len = 0: its outputs and query gradients are zero, and nothing is
    fetched for it (its key rows are given as row 0 of the tensor, where a fetch of the row before would fall
    outside the allocation)."""
    rng = np.random.default_rng(15)
    h, hd = 2, 64
    d = h * hd
    ql, kl = [0, 37, 130], [50, 0, 140]
    qr = np.array([0, 4, 60], np.int32)
    kr = np.array([10, 0, 70], np.int32)
    Tq, Tk = 200, 220
    q = _rnd(rng, (Tq, d), dt)
    kv = _rnd(rng, (Tk, 2 * d), dt)
    d_o = _rnd(rng, (Tq, d), dt)
    tq, tkv, tdo = to_dev(q, dt), to_dev(kv, dt), to_dev(d_o, dt)
    o = torch.full((Tq, d), 7.0, dtype=dt, device=DEV)
    lse = torch.zeros((h, Tq), dtype=F32, device=DEV)
    delta = torch.zeros((h, Tq), dtype=F32, device=DEV)
    dq = torch.full((Tq, d), 7.0, dtype=dt, device=DEV)
    dkv = torch.zeros((Tk, 2 * d), dtype=dt, device=DEV)
    es = tq.element_size()
    i32 = lambda a: torch.tensor(np.asarray(a), dtype=torch.int32, device=DEV)
    t_qr, t_ql, t_kr, t_kl = i32(qr), i32(ql), i32(kr), i32(kl)
    kb = tkv.data_ptr()
    scratch = torch.zeros(ds.ds_attention_scratch_bytes(h, hd, Tq, Tk, 3), dtype=torch.uint8, device=DEV)
    ds.ds_attention_fwd(tq, kb, kb + d * es, o, lse, t_qr, t_ql, t_kr, t_kl, h, hd, False, max(ql), max(kl),
                        d, 2 * d, 2 * d, d, Tq, k_total_rows=Tk, scratch=scratch, force_generic=force)
    gb = dkv.data_ptr()
    ds.ds_attention_bwd(tq, kb, kb + d * es, o, tdo, lse, delta, dq, gb, gb + d * es, t_qr, t_ql, t_kr, t_kl, h, hd, False,
                        max(ql), max(kl), d, 2 * d, 2 * d, d, Tq, k_total_rows=Tk, scratch=scratch, force_generic=force)
    torch.cuda.synchronize()
    o_np, dq_np, dkv_np = to_np(o), to_np(dq), to_np(dkv)
    tol = TOL[dt]
    # the sequence without keys: zeros; rows of no sequence (and of the one without queries): untouched
    assert np.all(o_np[4:4 + 37] == 0) and np.all(dq_np[4:4 + 37] == 0)
    untouched = np.ones(Tq, dtype=bool)
    untouched[4:4 + 37] = False
    untouched[60:60 + 130] = False
    assert np.all(o_np[untouched] == 7.0) and np.all(dq_np[untouched] == 7.0)
    assert np.all(dkv_np[:70] == 0) and np.all(dkv_np[70 + 140:] == 0)       # keys of the query-less sequence get nothing
    # the ordinary sequence beside them is unaffected
    qq = q[60:190].astype(np.float64)
    kk = kv[70:210, :d].astype(np.float64)
    vv = kv[70:210, d:].astype(np.float64)
    ref_o, cache = ost.attention_fwd(qq, kk, vv, h, False)
    rq, rk, rv = ost.attention_bwd(d_o[60:190].astype(np.float64), cache)
    assert both_err(o_np[60:190], ref_o) <= tol
    assert both_err(dq_np[60:190], rq) <= tol
    assert both_err(dkv_np[70:210, :d], rk) <= tol
    assert both_err(dkv_np[70:210, d:], rv) <= tol


# ragged rows, columns (not a multiple of a tile) and K: 64 x 64 and 64 x 128 tiles of the fp32 products on the bf16 matrix cores
@pytest.mark.parametrize("form", ["NN", "NT"])
@pytest.mark.parametrize("M,N,K", [(4003, 264, 36), (2050, 520, 100), (4096, 256, 256), (8203, 520, 516), (4003, 264, 196), (2050, 520, 228)])
def test_gemm_f32_as_bf16_products(form, M, N, K):
    """Within the error of fp32 sums: per product less than 2^-22 is left out and every addition rounds by 2^-24, over K of them
    sqrt(K) 2^-24 in the mean; values from 2^-40 to 2^40 in the same row."""
    rng = np.random.default_rng(M + K)
    A = (_rnd(rng, (M, K), F32) * np.exp2(rng.integers(-40, 41, (M, 1)))).astype(np.float32)
    B = _rnd(rng, (N, K) if form == "NT" else (K, N), F32)
    c = torch.full((M, N), 3.0, dtype=F32, device=DEV)
    ds.ds_gemm(to_dev(A, F32), to_dev(B, F32), c, M, N, K, trans_b=form == "NT")
    torch.cuda.synchronize()
    ref = A.astype(np.float64) @ (B.T if form == "NT" else B).astype(np.float64)
    err = np.linalg.norm(to_np(c) - ref, axis=1) / np.linalg.norm(ref, axis=1)          # every row on its own scale
    assert err.max() <= 4 * np.sqrt(K) * 2.0 ** -24


def test_gemm_f32_operands_beyond_4_gib():
    """Ones, 1216 x (2^20 + 4) both (4.75 GiB each): every result is the length of the contraction, whose last K tile holds 4 values."""
    M, K = 1216, (1 << 20) + 4
    a, c = torch.ones((M, K), dtype=F32, device=DEV), torch.zeros((M, M), dtype=F32, device=DEV)
    b = torch.ones_like(a)
    ds.ds_gemm(a, b, c, M, M, K, trans_b=True)
    torch.cuda.synchronize()
    assert bool((c == K).all())


@pytest.mark.parametrize("K", [64, 192])                                     # fp32 products and bf16 ones
def test_gemm_f32_values_that_bf16_products_do_not_represent(K):
    """Inf, NaN, values next to the largest and rows of tiny ones: as with fp32 products."""
    rng = np.random.default_rng(77)
    M, N = 4096, 256
    A, B = _rnd(rng, (M, K), F32), _rnd(rng, (K, N), F32)
    A[3, 5], A[700, 1], A[701, 2], A[1500, 3] = np.inf, np.nan, -np.inf, 3.4e38
    A[2000] *= np.float32(1e-36)
    B[:, 17] *= np.float32(0.25)
    c = torch.zeros((M, N), dtype=F32, device=DEV)
    ds.ds_gemm(to_dev(A, F32), to_dev(B, F32), c, M, N, K)
    torch.cuda.synchronize()
    c = c.cpu().numpy()
    with np.errstate(all="ignore"):
        ref = A.astype(np.float64) @ B.astype(np.float64)
        ref32 = ref.astype(np.float32)
    special = [3, 700, 701, 1500]
    for r in special[:3]:
        assert np.array_equal(np.isnan(c[r]), np.isnan(ref32[r])) and np.array_equal(np.isposinf(c[r]), np.isposinf(ref32[r]))
    ok = np.isfinite(ref32[1500])
    assert np.all(np.abs(c[1500][ok] - ref[1500][ok]) <= 1e-6 * np.abs(ref[1500][ok]).max())
    rest = np.setdiff1d(np.arange(M), special)
    err = np.linalg.norm(c[rest].astype(np.float64) - ref[rest], axis=1) / np.linalg.norm(ref[rest], axis=1)
    assert err.max() <= 4 * np.sqrt(K) * 2.0 ** -24


@pytest.mark.parametrize("form", ["NN", "NT"])
@pytest.mark.parametrize("N,K", [(264, 4), (264, 36), (264, 192), (264, 228), (1024, 516)])
def test_gemm_f32_one_product_per_result(form, N, K):
    """Rows with one value: a result is one product, rounded by 2^-24 where it is added up, and by less than 2^-26 in all where the seven
    small ones of its eight bf16 products are (each by at most 2^-23 of their sum, which is below 2^-7 of it)."""
    rng = np.random.default_rng(K)
    M = 4100
    A, B = np.zeros((M, K), np.float32), _rnd(rng, (K, N), F32)
    A[np.arange(M), rng.integers(0, K, M)] = rng.standard_normal(M)
    c = torch.zeros((M, N), dtype=F32, device=DEV)
    ds.ds_gemm(to_dev(A, F32), to_dev(B.T if form == "NT" else B, F32), c, M, N, K, trans_b=form == "NT")
    torch.cuda.synchronize()
    ref = A.astype(np.float64) @ B.astype(np.float64)
    assert np.all(np.abs(c.cpu().numpy() - ref) <= (2.0 ** -24 + 2.0 ** -26) * np.abs(ref))


@pytest.mark.parametrize("form", ["NN", "NT"])
@pytest.mark.parametrize("N", [264, 1024])                                    # 64 x 64 and 64 x 128 tiles
def test_gemm_f32_products_next_to_overflow(form, N):
    """Products and sums up to the largest float are finite, as with fp32 products, whatever their bf16 parts round to; larger ones
    are infinite.  K = 512: one addition rounds by 2^-24, and there are at most three."""
    M, K = 4100, 512
    A, B = np.zeros((M, K)), np.zeros((K, N))
    A[:, 0], B[0] = 1.8446e19, 1.8446e19                                       # 3.4026e38, their upper 8 bits rounded up: 2^128
    A[1::4, 7], B[7] = -2.0 ** 100, 2.0 ** 27                                  # 3.4026e38 - 1.7014e38
    A[2::4, 0], A[2::4, 70], B[70] = 2.0 ** 63, 1.7e38 / 2.0 ** 20, 2.0 ** 20    # 1.7014e38 + 1.7e38
    A[3::4, 300], B[300] = 1e30, 1e8                                           # 3.4026e38 + 1e38: beyond it
    A, B = A.astype(np.float32), B.astype(np.float32)
    c = torch.zeros((M, N), dtype=F32, device=DEV)
    ds.ds_gemm(to_dev(A, F32), to_dev(B.T if form == "NT" else B, F32), c, M, N, K, trans_b=form == "NT")
    torch.cuda.synchronize()
    ref, c = A.astype(np.float64) @ B.astype(np.float64), c.cpu().numpy().astype(np.float64)
    beyond = ref > np.finfo(np.float32).max
    assert beyond[3::4].all() and not beyond[0::4].any() and not beyond[1::4].any() and not beyond[2::4].any()
    assert np.all(np.isposinf(c[beyond])) and np.all(np.abs(c - ref)[~beyond] <= 3 * 2.0 ** -24 * ref[~beyond])


@pytest.mark.parametrize("form", ["NN", "NT"])
@pytest.mark.parametrize("exponent", [-112, -124])
def test_gemm_f32_tiny_values_beside_larger_ones(form, exponent):
    """A value below 2^-110 keeps all its bits also where its neighbours are larger: one product per result counts, which fp32 rounds
    by 2^-24."""
    rng = np.random.default_rng(-exponent)
    M, N, K = 4096, 256, 192
    A, B = np.zeros((M, K), np.float32), _rnd(rng, (K, N), F32)
    A[:, 3], A[:, 2] = rng.uniform(1, 2, M) * 2.0 ** exponent, 2.0 ** -100
    B[2], B[3] = 0, B[3] * np.float32(2.0 ** 60)
    c = torch.zeros((M, N), dtype=F32, device=DEV)
    ds.ds_gemm(to_dev(A, F32), to_dev(B.T if form == "NT" else B, F32), c, M, N, K, trans_b=form == "NT")
    torch.cuda.synchronize()
    ref = A.astype(np.float64) @ B.astype(np.float64)
    assert np.all(np.abs(c.cpu().numpy() - ref) <= 2.0 ** -24 * np.abs(ref))


@pytest.mark.parametrize("dt", [F32, BF])
@pytest.mark.parametrize("rms", [False, True])
@pytest.mark.parametrize("d", [256, 1024, 1536, 2048, 3072, 4096])
def test_norm_forward_backward(dt, rms, d):
    _norm_case(dt, rms, d, 1000 + 3)


@pytest.mark.parametrize("dt,rms", [(BF, False), (F32, True)])
def test_norm_wide_rows_more_rows_than_work_groups(dt, rms):
    """d = 4096 runs a pair of wavefronts per row; with more rows than work-groups each pair walks several rows."""
    _norm_case(dt, rms, 4096, 4500)


def _norm_case(dt, rms, d, rows):
    rng = np.random.default_rng(6)
    x = _rnd(rng, (rows, d), dt, 2.0) + (0 if rms else 0.5)
    if dt == BF:
        x = wl.to_bf16_grid(x)
    g = _rnd(rng, (d,), dt, 0.1) + 1.0
    if dt == BF:
        g = wl.to_bf16_grid(g)
    b = _rnd(rng, (d,), dt, 0.1)
    dy = _rnd(rng, (rows, d), dt)
    resid = _rnd(rng, (rows, d), dt)
    tx, tg, tb, tdy, tres = (to_dev(a, dt) for a in (x, g, b, dy, resid))
    y = torch.zeros_like(tx)
    dx = torch.zeros_like(tx)
    stats = torch.zeros((2, rows), dtype=F32, device=DEV)
    dg = torch.full((d,), 1.0, dtype=F32, device=DEV)
    db = torch.full((d,), 1.0, dtype=F32, device=DEV)
    partial = torch.zeros(ds.ds_norm_bwd_scratch_floats(rows, d), dtype=F32, device=DEV)
    ds.ds_norm_fwd(tx, tg, None if rms else tb, y, stats, rms=rms)
    ds.ds_norm_bwd(tdy, tx, tg, stats, tres, dx, dg, None if rms else db, partial, rms=rms, accumulate=True)
    torch.cuda.synchronize()
    X, G, DY = x.astype(np.float64), g.astype(np.float64), dy.astype(np.float64)
    if rms:
        ref_y, cache = ost.rmsnorm_fwd(X, G)
        ref_dx, ref_dg = ost.rmsnorm_bwd(DY, cache, G)
        ref_db = None
    else:
        ref_y, cache = ost.layernorm_fwd(X, G, b.astype(np.float64))
        ref_dx, ref_dg, ref_db = ost.layernorm_bwd(DY, cache, G)
    tol = 6e-3 if dt == BF else 2e-5
    assert both_err(to_np(y), ref_y) <= tol
    assert both_err(to_np(dx), ref_dx + resid) <= tol
    assert both_err(to_np(dg), ref_dg + 1.0) <= 1e-4
    if not rms:
        assert both_err(to_np(db), ref_db + 1.0) <= 1e-4


@pytest.mark.parametrize("dt", [F32, BF])
def test_colsum(dt):
    rng = np.random.default_rng(7)
    rows, n = 5000 + 7, 1536
    x = _rnd(rng, (rows, n), dt)
    tx = to_dev(x, dt)
    out = torch.full((n,), 2.0, dtype=F32, device=DEV)
    partial = torch.zeros(ds.ds_norm_bwd_scratch_floats(rows, n), dtype=F32, device=DEV)
    ds.ds_colsum(tx, out, partial, accumulate=True)
    ds.ds_colsum(tx, out, partial, accumulate=False)
    torch.cuda.synchronize()
    assert both_err(to_np(out), x.astype(np.float64).sum(axis=0)) <= 1e-5


def test_pack_unpack_roundtrip():
    lens = np.array([5, 3, 9, 3, 7, 2], dtype=np.int32)
    lo = ds.dp_plan(lens, ds.make_cost_model(fixed=10 ** 6, lin=1), 18, 2)
    d = 16
    canon = torch.arange(int(lens.sum()) * d, dtype=F32, device=DEV).reshape(-1, d).contiguous()
    stream = torch.full((lo.total_rows, d), float("nan"), dtype=F32, device=DEV)
    ds.ds_pack(lo, canon, stream)
    host = stream.cpu().numpy()
    off = np.concatenate([[0], np.cumsum(lens)])
    valid = np.zeros(lo.total_rows, bool)
    for s in range(lo.n_seq):
        i = int(lo.perm[s])
        r = int(lo.seq_row[s])
        np.testing.assert_array_equal(host[r:r + lens[i]], canon.cpu().numpy()[off[i]:off[i + 1]])
        valid[r:r + lens[i]] = True
    assert np.all(host[~valid] == 0)
    back = torch.zeros_like(canon)
    ds.ds_unpack(lo, stream, back)
    assert torch.equal(back, canon)


# ---- the direct-to-LDS matrix-core kernel (NT / TN forms) at operator level, with and without the split-K workspace

def _ws(floats):
    return torch.zeros(floats, dtype=F32, device=DEV)


@pytest.mark.parametrize("use_ws", [False, True])
@pytest.mark.parametrize("M,N,K", [(700, 256, 128), (1037, 512, 1024), (5157, 3328, 1024)])
def test_gemm_nt_epilogues(use_ws, M, N, K):
    """C = A B^T with B given as [N, K] (forward with transposed weights, input gradients): every epilogue, ragged M; the first
    two shapes run on 64 x 64 tiles, the last one on 128 x 128 tiles without a workspace and on 256 x 256 tiles with one
    (whole rounds unsplit, the remaining tiles split over K).  test_gemm_every_macro_tile_nt has the rest."""
    rng = np.random.default_rng(12)
    A, B = _rnd(rng, (M, K), BF), _rnd(rng, (N, K), BF, 0.1)
    bias, R, R2 = _rnd(rng, (N,), BF), _rnd(rng, (M, N), BF), _rnd(rng, (M, N), BF)
    valid = np.where(rng.random(M) < 0.8, 1, -1).astype(np.int32)
    acc = A.astype(np.float64) @ B.astype(np.float64).T
    dA, dB, db, dR, dR2 = (to_dev(x, BF) for x in (A, B, bias, R, R2))
    dvalid = torch.from_numpy(valid).to(DEV)
    ws = _ws(40 * 256 * 256) if use_ws else None
    tol = 6e-3

    def run(epi, **kw):
        c = torch.zeros((M, N), dtype=BF, device=DEV)
        c2 = torch.zeros((M, N), dtype=BF, device=DEV)
        ds.ds_gemm(dA, dB, c, M, N, K, trans_b=True, epilogue=epi, C2=c2, workspace=ws, **kw)
        torch.cuda.synchronize()
        return to_np(c), to_np(c2)

    c, _ = run(ds.DS_EPI_NONE)
    assert both_err(c, acc) <= tol
    c, _ = run(ds.DS_EPI_NONE, bias=db)
    assert both_err(c, acc + bias) <= tol
    z, a = run(ds.DS_EPI_GELU, bias=db)
    assert both_err(z, acc + bias) <= tol and both_err(a, ost.gelu(acc + bias)) <= tol
    c, _ = run(ds.DS_EPI_RESID, bias=db, R=dR, row_valid=dvalid)
    assert both_err(c, (acc + bias + R) * (valid[:, None] >= 0)) <= tol and np.all(c[valid < 0] == 0)
    c, _ = run(ds.DS_EPI_DGELU, R=dR)
    assert both_err(c, acc * ost.gelu_grad(R.astype(np.float64))) <= tol
    gd, a = run(ds.DS_EPI_GELU_D, bias=db)                # derivative kept instead of the pre-activation
    assert both_err(gd, ost.gelu_grad(acc + bias)) <= tol and both_err(a, ost.gelu(acc + bias)) <= tol
    c, _ = run(ds.DS_EPI_MULR, R=dR)
    assert both_err(c, acc * R) <= tol
    zu, h = run(ds.DS_EPI_GATE, R=dR)
    assert both_err(zu, acc) <= tol and both_err(h, ost.gelu(R.astype(np.float64)) * acc) <= tol
    g1, g2 = run(ds.DS_EPI_DGATE, R=dR, R2=dR2)
    assert both_err(g1, acc * R2 * ost.gelu_grad(R.astype(np.float64))) <= tol
    assert both_err(g2, acc * ost.gelu(R.astype(np.float64))) <= tol


@pytest.mark.parametrize("M,N,K", [(512, 768, 2085), (256, 256, 4100), (2048, 2048, 1031)])
def test_gemm_weight_gradient_split_over_the_contraction(M, N, K):
    """dW = X^T dY with a workspace, in which the contraction may be cut into ranges (ragged last tile) whose partial sums a
    second kernel adds (256 x 256 x 4100 is; the others run whole, on 64 x 64 and 128 x 128 tiles); overwrite and
    accumulate; same result as without a workspace up to summation order."""
    rng = np.random.default_rng(13)
    X, dY = _rnd(rng, (K, M), BF), _rnd(rng, (K, N), BF)
    ref = X.astype(np.float64).T @ dY.astype(np.float64)
    dX, ddY = to_dev(X, BF), to_dev(dY, BF)
    ws = _ws(4 * M * N + 4096)
    Cd = torch.full((M, N), 3.0, dtype=F32, device=DEV)
    ds.ds_gemm(dX, ddY, Cd, M, N, K, trans_a=True, epilogue=ds.DS_EPI_ACC32, accumulate=False, workspace=ws)
    torch.cuda.synchronize()
    assert both_err(to_np(Cd), ref) <= 1e-5
    ds.ds_gemm(dX, ddY, Cd, M, N, K, trans_a=True, epilogue=ds.DS_EPI_ACC32, accumulate=True, workspace=ws)
    torch.cuda.synchronize()
    assert both_err(to_np(Cd), 2 * ref) <= 1e-5
    plain = torch.zeros((M, N), dtype=F32, device=DEV)
    ds.ds_gemm(dX, ddY, plain, M, N, K, trans_a=True, epilogue=ds.DS_EPI_ACC32, accumulate=False)
    torch.cuda.synchronize()
    assert both_err(to_np(plain), ref) <= 1e-5


def _close(got, want, tol):
    """both_err(...) <= tol on the device."""
    err = got.double() - want
    return float(err.norm() / want.norm()) <= tol and bool((err.abs() <= tol * (8 * want.square().mean().sqrt() + want.abs())).all())


def _nt_epilogues_on_device(M, N, K, ws, epilogues, form, repeat=False):
    """C = A B^T with each of the epilogues against float64 on the device, 6e-3 (bf16: one rounding, 2^-9 of each value; fp32 output 1e-5); the
    row behind the last one of both outputs is not written; every product goes out as `form` says.  repeat: again on another stream and a third
    time, bit for bit the same."""
    rng = np.random.default_rng(21)
    dA, dB = to_dev(_rnd(rng, (M, K), BF), BF), to_dev(_rnd(rng, (N, K), BF, 0.1), BF)
    db = to_dev(_rnd(rng, (N,), BF), BF)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(21)
    dR, dR2 = (torch.randn((M, N), device=DEV, generator=gen).to(BF) for _ in range(2))
    valid = torch.from_numpy(np.where(rng.random(M) < 0.9, 1, -1).astype(np.int32)).to(DEV)
    acc, b, r = torch.matmul(dA.double(), dB.double().t().contiguous()), db.double(), dR.double()
    side = torch.cuda.Stream()
    torch.cuda.synchronize()

    def gelu(z):
        return torch.nn.functional.gelu(z, approximate="tanh")

    def gelu_grad(z):
        u = 0.7978845608028654 * (z + 0.044715 * z ** 3)
        t = torch.tanh(u)
        return 0.5 * (1 + t) + 0.5 * z * (1 - t * t) * 0.7978845608028654 * (1 + 3 * 0.044715 * z * z)

    cases = {ds.DS_EPI_NONE: (dict(bias=db), lambda: (acc + b, None)),
             ds.DS_EPI_GELU: (dict(bias=db), lambda: (acc + b, gelu(acc + b))),
             ds.DS_EPI_RESID: (dict(bias=db, R=dR, row_valid=valid), lambda: ((acc + b + r) * (valid >= 0).double()[:, None], None)),
             ds.DS_EPI_DGELU: (dict(R=dR), lambda: (acc * gelu_grad(r), None)),
             ds.DS_EPI_ACC32: (dict(), lambda: (acc, None)),
             ds.DS_EPI_GATE: (dict(R=dR), lambda: (acc, gelu(r) * acc)),
             ds.DS_EPI_DGATE: (dict(R=dR, R2=dR2), lambda: (acc * dR2.double() * gelu_grad(r), acc * gelu(r))),
             ds.DS_EPI_GELU_D: (dict(bias=db), lambda: (gelu_grad(acc + b), gelu(acc + b))),
             ds.DS_EPI_MULR: (dict(R=dR), lambda: (acc * r, None))}
    for epi in epilogues:
        assert form(gemm_launches(M, N, K, epilogue=epi, ws_floats=0 if ws is None else ws.numel())), epi
        kw, ref = cases[epi]
        want, want2 = ref()
        f32 = epi == ds.DS_EPI_ACC32
        for times in ((1, 2) if f32 else (1,)):
            first = None
            for stream in ((None, side.cuda_stream, None) if repeat else (None,)):
                c = torch.full((M + 1, N), 7.0, dtype=F32 if f32 else BF, device=DEV)
                c2 = torch.full((M + 1, N), 7.0, dtype=BF, device=DEV)
                if times == 2:
                    c[:M] = want.float()
                torch.cuda.synchronize()
                ds.ds_gemm(dA, dB, c, M, N, K, trans_b=True, epilogue=epi, C2=c2, workspace=ws, stream=stream, accumulate=times == 2, **kw)
                torch.cuda.synchronize()
                if first is None:
                    first = c, c2
                    assert _close(c[:M], times * want, 1e-5 if f32 else 6e-3), (epi, times)
                    if want2 is not None:
                        assert _close(c2[:M], want2, 6e-3), epi
                    assert bool((c[M] == 7.0).all()) and bool((c2[M if want2 is not None else 0:] == 7.0).all()), epi
                else:
                    assert torch.equal(c, first[0]) and torch.equal(c2, first[1]), epi


EVERY_EPILOGUE = (ds.DS_EPI_NONE, ds.DS_EPI_GELU, ds.DS_EPI_RESID, ds.DS_EPI_DGELU, ds.DS_EPI_ACC32, ds.DS_EPI_GATE, ds.DS_EPI_DGATE,
                  ds.DS_EPI_GELU_D, ds.DS_EPI_MULR)


@pytest.mark.parametrize("M,N,K,ws_floats,whole,pieces", [(10713, 4608, 512, 0, 756, 1), (4767, 8192, 4096, 1 << 24, 512, 2)])
def test_gemm_nt_persistent_form(M, N, K, ws_floats, whole, pieces):
    """A launch with at least two unsplit tiles per compute unit takes the persistent form of the NT kernel (resident
    work-groups drawing tiles from per-XCD counters): three rounds, the last partly filled, with a ragged last row of tiles; two rounds with split
    pieces of the other tiles behind them.  Every epilogue but the fp32 output of the second; each three times, bit for bit the same (the counters a
    launch leaves behind are those the next one starts from)."""
    def form(l):
        return len(l) == 1 and l[0]["persistent"] and (l[0]["whole"], l[0]["pieces"]) == (whole, pieces)

    _nt_epilogues_on_device(M, N, K, _ws(ws_floats) if ws_floats else None, [e for e in EVERY_EPILOGUE if pieces == 1 or e != ds.DS_EPI_ACC32], form, repeat=True)


def test_mfma_probe_runs_and_is_deterministic():
    """The measurement aid: the loop really runs (sums differ from zero on random operands, are zero on zeros) and
    gives the same sums every time."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(5)
    ops = torch.randn(24 * 512 * 8, device=DEV, generator=gen).to(BF)
    sink = torch.zeros(2 * 512, dtype=F32, device=DEV)
    ds.ds_mfma_probe(ops, sink, 2, 3)
    torch.cuda.synchronize()
    first = to_np(sink)
    assert np.all(np.isfinite(first)) and np.count_nonzero(first) > 900
    assert np.array_equal(first[:512], first[512:])             # every work-group computes the same
    ds.ds_mfma_probe(ops, sink, 2, 3)
    torch.cuda.synchronize()
    assert np.array_equal(first, to_np(sink))
    ds.ds_mfma_probe(torch.zeros_like(ops), sink, 2, 3)
    torch.cuda.synchronize()
    assert np.count_nonzero(to_np(sink)) == 0
    with pytest.raises(ds.DsError):
        ds.ds_mfma_probe(ops, sink, 0, 3)


@pytest.mark.parametrize("form,M,N,K,use_ws", [
    ("nn", 1, 8, 4, False), ("nn", 65, 72, 36, False), ("nn", 300, 1032, 132, False), ("nn", 129, 264, 4100, True),
    ("nt", 64, 64, 32, False), ("nt", 63, 200, 100, False), ("nt", 4200, 1032, 64, False),       # the last: more tiles than two per CU
    ("tn", 4, 8, 1, False), ("tn", 68, 200, 31, False), ("tn", 256, 256, 7684, True), ("tn", 260, 520, 129, True)])
def test_gemm_f32_matrix_cores(form, M, N, K, use_ws):
    """Edges of the 64-row and 64-column tiles, of the 32-deep K tiles and of the split contraction, against float64."""
    rng = np.random.default_rng(31)
    ta, tb = form == "tn", form == "nt"
    A, B = _rnd(rng, (K, M) if ta else (M, K), F32), _rnd(rng, (N, K) if tb else (K, N), F32)
    bias, R = _rnd(rng, (N,), F32), _rnd(rng, (M, N), F32)
    acc = (A.T if ta else A).astype(np.float64) @ (B.T if tb else B).astype(np.float64)
    dA, dB, db, dR = (to_dev(x, F32) for x in (A, B, bias, R))
    c, c2 = (torch.full((M, N), 3.0, dtype=F32, device=DEV) for _ in range(2))
    kw = dict(trans_a=ta, trans_b=tb, workspace=_ws(1 << 22) if use_ws else None)
    # fp32 sums of K products in any order: K 2^-24 relative to the sum of magnitudes, about sqrt(K) 2^-24 of the result
    tol = 1e-5
    ds.ds_gemm(dA, dB, c, M, N, K, bias=db, **kw)
    torch.cuda.synchronize()
    assert both_err(to_np(c), acc + bias) <= tol
    ds.ds_gemm(dA, dB, c, M, N, K, epilogue=ds.DS_EPI_ACC32, accumulate=False, **kw)
    ds.ds_gemm(dA, dB, c, M, N, K, epilogue=ds.DS_EPI_ACC32, accumulate=True, **kw)
    torch.cuda.synchronize()
    assert both_err(to_np(c), 2 * acc) <= tol
    ds.ds_gemm(dA, dB, c, M, N, K, epilogue=ds.DS_EPI_RESID, R=dR, bias=db, **kw)
    torch.cuda.synchronize()
    assert both_err(to_np(c), acc + bias + R) <= tol
    ds.ds_gemm(dA, dB, c, M, N, K, epilogue=ds.DS_EPI_DGATE, R=dR, R2=dR, C2=c2, **kw)
    torch.cuda.synchronize()
    Rd = R.astype(np.float64)
    assert both_err(to_np(c), acc * Rd * ost.gelu_grad(Rd)) <= tol and both_err(to_np(c2), acc * ost.gelu(Rd)) <= tol


@pytest.mark.parametrize("hd,causal", [(8, True), (24, False), (32, True), (40, True), (64, True), (64, False), (96, True), (128, True), (128, False)])
def test_attention_f32_matrix_cores(hd, causal):
    """Every padded head size (32, 64, 96, 128) and lengths on both sides of the 16-column, 32- / 64-row tile edges."""
    rng = np.random.default_rng(32)
    h = 2
    lens = [1, 15, 16, 17, 31, 33, 63, 64, 65, 127, 129, 200, 333]
    d, T, rows, qkv, d_o = _varlen_case(rng, lens, h, hd, F32)
    dq, ddo = to_dev(qkv, F32), to_dev(d_o, F32)
    o, lse, delta = torch.zeros((T, d), device=DEV), torch.zeros((h, T), device=DEV), torch.zeros((h, T), device=DEV)
    dqkv = torch.zeros((T, 3 * d), device=DEV)
    order = rng.permutation(len(lens))
    t_rows = torch.from_numpy(np.ascontiguousarray(rows[order])).to(DEV)
    t_lens = torch.tensor([lens[i] for i in order], dtype=torch.int32, device=DEV)
    b, gb, table = dq.data_ptr(), dqkv.data_ptr(), (t_rows, t_lens, t_rows, t_lens)
    ds.ds_attention_fwd(b, b + 4 * d, b + 8 * d, o, lse, *table, h, hd, causal, max(lens), max(lens), 3 * d, 3 * d, 3 * d, d, T)
    ds.ds_attention_bwd(b, b + 4 * d, b + 8 * d, o, ddo, lse, delta, gb, gb + 4 * d, gb + 8 * d, *table, h, hd, causal,
                        max(lens), max(lens), 3 * d, 3 * d, 3 * d, d, T)
    torch.cuda.synchronize()
    o_np, g_np, lse_np = to_np(o), to_np(dqkv), to_np(lse)
    touched = np.zeros(T, dtype=bool)
    for r0, l in zip(rows, lens):
        x = qkv[r0:r0 + l].astype(np.float64)
        q, k, v = x[:, :d], x[:, d:2 * d], x[:, 2 * d:]
        ref_o, cache = ost.attention_fwd(q, k, v, h, causal)
        refs = ost.attention_bwd(d_o[r0:r0 + l].astype(np.float64), cache)
        assert both_err(o_np[r0:r0 + l], ref_o) <= TOL[F32], (l, "o")
        for i, ref in enumerate(refs):
            assert both_err(g_np[r0:r0 + l, i * d:(i + 1) * d], ref) <= TOL[F32], (l, "dq dk dv"[3 * i:3 * i + 2])
        s = (q[-1, -hd:] @ k[:, -hd:].T) / np.sqrt(hd)                     # last head, last row: sees every key
        assert abs(lse_np[-1, r0 + l - 1] - np.log(np.exp(s - s.max()).sum()) - s.max()) <= 1e-5
        touched[r0:r0 + l] = True
    assert np.all(o_np[~touched] == 0) and np.all(g_np[~touched] == 0)


# few blocks; 1 008 of them, which go last to first in the causal forward and dQ kernels
@pytest.mark.parametrize("h,lens", [(2, [130, 0, 64, 1]), (8, [130, 0, 64, 1] + 80 * [65])])
@pytest.mark.parametrize("causal", [True, False])
def test_attention_f32_odd_and_even_numbers_of_blocks(causal, h, lens):
    """The number of 64-column blocks per grid row may be more than the longest sequence needs, by the kernel's choice or the
    caller's: the same results."""
    rng = np.random.default_rng(34)
    hd = 64
    d, T, rows, qkv, d_o = _varlen_case(rng, lens, h, hd, F32)
    dq, ddo = to_dev(qkv, F32), to_dev(d_o, F32)
    t_rows, t_lens = torch.from_numpy(rows).to(DEV), torch.tensor(lens, dtype=torch.int32, device=DEV)
    b, table, got = dq.data_ptr(), (t_rows, t_lens, t_rows, t_lens), []
    for max_len in (130, 193, 600):
        o, lse, delta = torch.zeros((T, d), device=DEV), torch.zeros((h, T), device=DEV), torch.zeros((h, T), device=DEV)
        dqkv = torch.zeros((T, 3 * d), device=DEV)
        gb = dqkv.data_ptr()
        ds.ds_attention_fwd(b, b + 4 * d, b + 8 * d, o, lse, *table, h, hd, causal, max_len, max_len, 3 * d, 3 * d, 3 * d, d, T)
        ds.ds_attention_bwd(b, b + 4 * d, b + 8 * d, o, ddo, lse, delta, gb, gb + 4 * d, gb + 8 * d, *table, h, hd, causal,
                            max_len, max_len, 3 * d, 3 * d, 3 * d, d, T)
        torch.cuda.synchronize()
        got.append([to_np(x) for x in (o, lse, dqkv)])
    for x, y, z in zip(*got):
        assert np.array_equal(x, y) and np.array_equal(x, z)
    for r0, l in zip(rows, lens):
        x = qkv[r0:r0 + l].astype(np.float64)
        if l:
            ref_o, cache = ost.attention_fwd(x[:, :d], x[:, d:2 * d], x[:, 2 * d:], h, causal)
            assert both_err(got[0][0][r0:r0 + l], ref_o) <= TOL[F32], l
            for i, ref in enumerate(ost.attention_bwd(d_o[r0:r0 + l].astype(np.float64), cache)):
                assert both_err(got[0][2][r0:r0 + l, i * d:(i + 1) * d], ref) <= TOL[F32], (l, i)


@pytest.mark.parametrize("dt", [F32, BF])
@pytest.mark.parametrize("rows,n", [(1, 8), (31, 264), (33, 2048), (128, 520), (4097, 256), (9000, 4104)])
def test_column_reductions_at_their_edges(dt, rows, n):
    """One to many partial rows (32 rows per work-group, four in flight; both widths of the second kernel), added to what is
    there.  Sums of at most 9000 fp32 values: 1e-5."""
    rng = np.random.default_rng(33)
    x = _rnd(rng, (rows, n), dt)
    xd = to_dev(x, dt)
    partial = torch.empty(2048 * max(n, 1024), device=DEV)
    out = torch.full((n,), 2.0, device=DEV)
    ds.ds_colsum(xd, out, partial, accumulate=True)
    torch.cuda.synchronize()
    assert both_err(to_np(out), x.astype(np.float64).sum(0) + 2.0) <= 1e-5
    if n <= 4096:
        for rms in (False, True):
            dy, g = _rnd(rng, (rows, n), dt), (1.0 + _rnd(rng, (n,), F32, 0.02)).astype(np.float32)
            b = _rnd(rng, (n,), dt, 0.02)
            g = wl.to_bf16_grid(g) if dt == BF else g
            dyd, gd, bd = to_dev(dy, dt), to_dev(g, dt), to_dev(b, dt)
            y, dx, stats = torch.empty_like(xd), torch.empty_like(xd), torch.empty(2, rows, device=DEV)
            dg, db = torch.full((n,), 3.0, device=DEV), torch.full((n,), 4.0, device=DEV)
            part = torch.empty(ds.ds_norm_bwd_scratch_floats(rows, n), device=DEV)
            ds.ds_norm_fwd(xd, gd, None if rms else bd, y, stats, rms=rms)
            ds.ds_norm_bwd(dyd, xd, gd, stats, None, dx, dg, db, part, rms=rms, accumulate=True)
            torch.cuda.synchronize()
            x64, dy64 = x.astype(np.float64), dy.astype(np.float64)
            c = x64 if rms else x64 - x64.mean(1, keepdims=True)
            xh = c / np.sqrt((c * c).mean(1, keepdims=True) + (1e-6 if rms else 1e-5))
            assert both_err(to_np(dg), (dy64 * xh).sum(0) + 3.0) <= 1e-5
            if not rms:
                assert both_err(to_np(db), dy64.sum(0) + 4.0) <= 1e-5


def test_attention_worklist_many_sequences():
    """More sequences than threads of the list kernel, every length class present, empty ones among them: every block of
    every sequence is visited once (the outputs are complete), on the query and on the key side."""
    rng = np.random.default_rng(34)
    h, hd, n = 1, 64, 2300
    lens = rng.integers(0, 40, n).astype(np.int32)
    lens[rng.integers(0, n, 40)] = rng.integers(100, 1400, 40)
    rows = np.cumsum(lens) - lens
    T, d = int(lens.sum()), h * hd
    qkv, d_o = to_dev(_rnd(rng, (T, 3 * d), BF), BF), to_dev(_rnd(rng, (T, d), BF), BF)
    table = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(DEV) for a in (rows, lens, rows, lens)]
    res = []
    for force in (False, True):
        o, lse, delta = torch.full((T, d), 7.0, dtype=BF, device=DEV), torch.zeros((h, T), device=DEV), torch.zeros((h, T), device=DEV)
        g = torch.full((T, 3 * d), 7.0, dtype=BF, device=DEV)
        scratch = torch.zeros(ds.ds_attention_scratch_bytes(h, hd, T, T, n), dtype=torch.uint8, device=DEV)
        b, gb = qkv.data_ptr(), g.data_ptr()
        ds.ds_attention_fwd(b, b + 2 * d, b + 4 * d, o, lse, *table, h, hd, True, 1400, 1400, 3 * d, 3 * d, 3 * d, d, T,
                            scratch=scratch, force_generic=force)
        ds.ds_attention_bwd(b, b + 2 * d, b + 4 * d, o, d_o, lse, delta, gb, gb + 2 * d, gb + 4 * d, *table, h, hd, True, 1400, 1400,
                            3 * d, 3 * d, 3 * d, d, T, scratch=scratch, force_generic=force)
        torch.cuda.synchronize()
        res.append((to_np(o), to_np(g)))
    for got, ref in zip(*res):
        assert both_err(got, ref) <= TOL[BF]


@pytest.mark.parametrize("M,N,K", [(1, 256, 64), (63, 256, 128), (65, 256, 1024), (129, 512, 320), (250, 1024, 256), (300, 256, 4096), (756, 2048, 2048)])
def test_gemm_smaller_tiles_nt(M, N, K):
    """Launches too small for 256 x 256 tiles: row edges of the 64- and 128-row tiles, one to many K tiles, with and without
    a workspace to split the contraction; rows beyond M stay untouched."""
    rng = np.random.default_rng(35)
    A, B = _rnd(rng, (M, K), BF), _rnd(rng, (N, K), BF, 0.1)
    bias, R = _rnd(rng, (N,), BF), _rnd(rng, (M, N), BF)
    acc = A.astype(np.float64) @ B.astype(np.float64).T
    dA, dB, db, dR = (to_dev(x, BF) for x in (A, B, bias, R))
    valid = np.where(rng.random(M) < 0.8, 1, -1).astype(np.int32)
    for ws in (None, _ws(1 << 22)):
        c, c2 = (torch.full((M + 3, N), 7.0, dtype=BF, device=DEV) for _ in range(2))
        ds.ds_gemm(dA, dB, c, M, N, K, trans_b=True, bias=db, workspace=ws)
        torch.cuda.synchronize()
        assert both_err(to_np(c)[:M], acc + bias) <= 4e-3 and np.all(to_np(c)[M:] == 7.0)       # one bf16 rounding: 2^-9
        ds.ds_gemm(dA, dB, c, M, N, K, trans_b=True, epilogue=ds.DS_EPI_RESID, bias=db, R=dR, row_valid=torch.from_numpy(valid).to(DEV), workspace=ws)
        torch.cuda.synchronize()
        assert both_err(to_np(c)[:M], (acc + bias + R) * (valid[:, None] >= 0)) <= 4e-3 and np.all(to_np(c)[:M][valid < 0] == 0)
        ds.ds_gemm(dA, dB, c, M, N, K, trans_b=True, epilogue=ds.DS_EPI_GELU_D, bias=db, C2=c2, workspace=ws)
        torch.cuda.synchronize()
        assert both_err(to_np(c)[:M], ost.gelu_grad(acc + bias)) <= 4e-3 and both_err(to_np(c2)[:M], ost.gelu(acc + bias)) <= 4e-3
        assert np.all(to_np(c)[M:] == 7.0) and np.all(to_np(c2)[M:] == 7.0)


@pytest.mark.parametrize("M,N,K", [(256, 256, 1), (256, 512, 31), (512, 256, 64), (256, 1024, 250), (768, 256, 577), (256, 256, 9001), (2048, 2048, 756)])
def test_gemm_smaller_tiles_weight_gradient(M, N, K):
    """The same for weight gradients: ragged contractions around the 64-deep K tile, split and whole; fp32 sums: 1e-5."""
    rng = np.random.default_rng(36)
    X, dY = _rnd(rng, (K, M), BF), _rnd(rng, (K, N), BF)
    ref = X.astype(np.float64).T @ dY.astype(np.float64)
    # rows behind the last valid one hold NaN: the bounds check must keep them out of the sums
    dX, ddY = (torch.cat([to_dev(a, BF), torch.full((64, a.shape[1]), float("nan"), dtype=BF, device=DEV)]) for a in (X, dY))
    for ws in (None, _ws(1 << 22)):
        c = torch.full((M, N), 3.0, dtype=F32, device=DEV)
        ds.ds_gemm(dX, ddY, c, M, N, K, trans_a=True, epilogue=ds.DS_EPI_ACC32, accumulate=False, workspace=ws)
        ds.ds_gemm(dX, ddY, c, M, N, K, trans_a=True, epilogue=ds.DS_EPI_ACC32, accumulate=True, workspace=ws)
        torch.cuda.synchronize()
        assert both_err(to_np(c), 2 * ref) <= 1e-5


@pytest.mark.parametrize("dt", [F32, BF])
@pytest.mark.parametrize("form,n,d", [("dp", 1, 8), ("dp", 40, 264), ("packed", 60, 128), ("fixed", 600, 24), ("dp", 1000, 16), ("target", 300, 72), ("packed", 2500, 8), ("target", 3000, 264)])
def test_pack_unpack_forms(dt, form, n, d):
    """Layouts in and out of row order, gaps at every kind of place, more sequences than one launch's arguments hold (few enough
    for several launches, and so many that the row map goes through memory), a target stream: every value moved once, padding rows zeroed over what was there."""
    rng = np.random.default_rng(37)
    lens = np.clip(np.rint(rng.lognormal(2.5, 0.8, n)), 1, 90).astype(np.int32)
    if form == "packed":
        lo = ds.ds_layout_packed(lens, 96, 3)
    elif form == "fixed":
        lo = ds.ds_layout_from_cuts(lens, list(range(0, n, 7)) + [n], perm=rng.permutation(n).astype(np.int32), pad_to=95)
    elif form == "target":
        lo = ds.ds_layout_from_cuts(np.full(n, 3, np.int32), list(range(0, n, 7)) + [n], lengths_tgt=lens)
    else:
        lo = ds.dp_plan(lens, ds.make_cost_model(fixed=3_000_00, lin=1), 1024, 2)
    which = 1 if form == "target" else 0
    rows = lo.total_rows_tgt if which else lo.total_rows
    seq_row, seq_len = (lo.seq_row_tgt, lo.seq_len_tgt) if which else (lo.seq_row, lo.seq_len)
    canon = _rnd(rng, (int(lens.sum()), d), dt)
    start = np.cumsum(lens) - lens
    ref = np.zeros((rows, d))
    for s in range(n):
        i = int(lo.perm[s])
        ref[seq_row[s]:seq_row[s] + seq_len[s]] = canon[start[i]:start[i] + lens[i]]
    cd, stream = to_dev(canon, dt), torch.full((rows + 1, d), 7.0, dtype=dt, device=DEV)
    ds.ds_pack(lo, cd, stream, which=which)
    back = torch.full((canon.shape[0] + 1, d), 7.0, dtype=dt, device=DEV)
    ds.ds_unpack(lo, stream, back, which=which)
    torch.cuda.synchronize()
    assert np.array_equal(to_np(stream)[:rows], ref) and np.all(to_np(stream)[rows] == 7.0)
    assert np.array_equal(to_np(back)[:-1], canon) and np.all(to_np(back)[-1] == 7.0)


@pytest.mark.parametrize("causal", [False, True])
def test_attention_128_items_without_steps(causal):
    """Head size 128, many more (key block, head) pairs than compute units, so that every work-group of the dK/dV kernel takes
    several: among them blocks that no query sees (sequences without queries, causal ones with more keys than queries),
    whose gradients are zero and which pass no barrier but the draw's.  Against the generic kernels, sequence by sequence (P
    and dS rounded to bf16, 2^-9 of each term; the gradients of a few keys under many queries are tens of times those of
    many keys, so that one scale for all sequences would say nothing); twice on one scratch, bit for bit the same."""
    rng = np.random.default_rng(38)
    h, hd, n = 8, 128, 150
    d = h * hd
    kl = rng.integers(64, 600, n).astype(np.int32)
    ql = np.where(rng.random(n) < 0.4, 0, rng.integers(32, 300, n)).astype(np.int32)
    qr, kr = (np.cumsum(a) - a for a in (ql, kl))
    Tq, Tk = int(ql.sum()), int(kl.sum())
    assert h * int(((kl + 127) // 128).sum()) > 3 * 256
    q, kv, d_o = (to_dev(_rnd(rng, s, BF), BF) for s in ((Tq, d), (Tk, 2 * d), (Tq, d)))
    table = [torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(DEV) for a in (qr, ql, kr, kl)]
    scratch = torch.zeros(ds.ds_attention_scratch_bytes(h, hd, Tq, Tk, n), dtype=torch.uint8, device=DEV)
    mx = (int(ql.max()), int(kl.max()))
    res = []
    for force in (False, False, True):
        o, lse, delta = torch.zeros((Tq, d), dtype=BF, device=DEV), torch.zeros((h, Tq), device=DEV), torch.zeros((h, Tq), device=DEV)
        dq, dkv = (torch.full((t, w), 7.0, dtype=BF, device=DEV) for t, w in ((Tq, d), (Tk, 2 * d)))
        b, gb = kv.data_ptr(), dkv.data_ptr()
        ds.ds_attention_fwd(q, b, b + 2 * d, o, lse, *table, h, hd, causal, *mx, d, 2 * d, 2 * d, d, Tq, k_total_rows=Tk,
                            scratch=scratch, force_generic=force)
        ds.ds_attention_bwd(q, b, b + 2 * d, o, d_o, lse, delta, dq, gb, gb + 2 * d, *table, h, hd, causal, *mx, d, 2 * d, 2 * d, d,
                            Tq, k_total_rows=Tk, scratch=scratch, force_generic=force)
        torch.cuda.synchronize()
        res.append([to_np(x) for x in (o, dq, dkv)])
    unseen = np.concatenate([np.arange(l) >= (m if causal or m == 0 else l) for l, m in zip(kl, ql)])
    assert unseen.sum() > 1000 and np.all(res[0][2][unseen] == 0)
    for got, again in zip(res[0], res[1]):
        assert np.array_equal(got, again)
    (o, dq, dkv), _, (ref_o, ref_dq, ref_dkv) = res
    for i in np.flatnonzero(ql):
        qs, ks = slice(qr[i], qr[i] + ql[i]), slice(kr[i], kr[i] + (min(kl[i], ql[i]) if causal else kl[i]))
        assert both_err(o[qs], ref_o[qs]) <= TOL[BF] and both_err(dq[qs], ref_dq[qs]) <= TOL[BF], i
        assert both_err(dkv[ks, :d], ref_dkv[ks, :d]) <= TOL[BF] and both_err(dkv[ks, d:], ref_dkv[ks, d:]) <= TOL[BF], i


@pytest.mark.parametrize("hd", [32, 64, 96, 128])
def test_attention_f32_causal_with_values_that_are_not_finite(hd):
    """An infinity or NaN in one token of a causal sequence: everything that does not see the token is what it is without it,
    everything else is not finite where the generic kernels, which read only what a row sees, say so.  The token lies at
    the start, in the middle and at the end of 16-token blocks and of tiles."""
    rng = np.random.default_rng(39)
    h = 2
    poison = [(l, part, pos, val) for part in "qkvo" for l, pos, val in
              ((40, 25, np.inf), (70, 69, np.nan), (130, 64, -np.inf), (200, 15, np.nan), (200, 143, np.inf), (33, 0, -np.inf))]
    lens = [p[0] for p in poison]
    d, T, rows, qkv, d_o = _varlen_case(rng, lens, h, hd, F32)
    for (l, part, pos, val), r0 in zip(poison, rows):
        if part == "o":
            d_o[r0 + pos, hd + 5] = val
        else:
            qkv[r0 + pos, "qkv".index(part) * d + hd + 5] = val             # second head only
    x, ddo = to_dev(qkv, F32), to_dev(d_o, F32)
    t_rows, t_lens = torch.from_numpy(rows).to(DEV), torch.tensor(lens, dtype=torch.int32, device=DEV)
    res = []
    for force in (False, True):
        o, lse, delta = torch.zeros((T, d), device=DEV), torch.zeros((h, T), device=DEV), torch.zeros((h, T), device=DEV)
        g = torch.zeros((T, 3 * d), device=DEV)
        b, gb, table = x.data_ptr(), g.data_ptr(), (t_rows, t_lens, t_rows, t_lens)
        ds.ds_attention_fwd(b, b + 4 * d, b + 8 * d, o, lse, *table, h, hd, True, max(lens), max(lens), 3 * d, 3 * d, 3 * d, d, T, force_generic=force)
        ds.ds_attention_bwd(b, b + 4 * d, b + 8 * d, o, ddo, lse, delta, gb, gb + 4 * d, gb + 8 * d, *table, h, hd, True,
                            max(lens), max(lens), 3 * d, 3 * d, 3 * d, d, T, force_generic=force)
        torch.cuda.synchronize()
        res.append(np.concatenate([to_np(o), to_np(g)], axis=1))
    for p, r0 in zip(poison, rows):
        got, ref = (r[r0:r0 + p[0]] for r in res)
        assert np.array_equal(np.isfinite(got), np.isfinite(ref)), p
        if p[1] != "o" or p[2] > 0:
            assert not np.isfinite(ref).all(), p
        assert np.isfinite(ref[:p[2], :d]).all(), p                         # outputs in front of the token
        for i in range(4):
            a, b = (np.where(np.isfinite(m), m, 0.0)[:, i * d:(i + 1) * d] for m in (got, ref))
            assert both_err(a, b) <= TOL[F32], (p, i)


@pytest.mark.parametrize("hd", [64, 128])
def test_attention_bf16_hidden_half_blocks_with_values_that_are_not_finite(hd):
    """dK / dV, causal: the kernel multiplies 32-query halves of its 64-query blocks by zero where a wavefront's 32 keys see none
    of a half's queries.  An infinity or NaN in a query (Q or dO) reaches no key of a later group of 32, and the copies of
    the last row that fill a ragged block add nothing to it."""
    rng = np.random.default_rng(40)
    h = 2
    cases = [(200, "q", 10, np.inf), (200, "o", 10, np.nan), (300, "q", 150, np.nan), (300, "o", 159, -np.inf), (96, "o", 95, np.inf)]
    lens = [c[0] for c in cases]
    d, T, rows, qkv, d_o = _varlen_case(rng, lens, h, hd, BF)
    for (l, part, pos, val), r0 in zip(cases, rows):
        (d_o if part == "o" else qkv)[r0 + pos, hd + 5] = val
    x, ddo = to_dev(qkv, BF), to_dev(d_o, BF)
    t_rows, t_lens = torch.from_numpy(rows).to(DEV), torch.tensor(lens, dtype=torch.int32, device=DEV)
    scratch = torch.zeros(ds.ds_attention_scratch_bytes(h, hd, T, T, len(lens)), dtype=torch.uint8, device=DEV)
    res = []
    for force in (False, True):
        o, lse, delta = torch.zeros((T, d), dtype=BF, device=DEV), torch.zeros((h, T), device=DEV), torch.zeros((h, T), device=DEV)
        g = torch.zeros((T, 3 * d), dtype=BF, device=DEV)
        b, gb, table = x.data_ptr(), g.data_ptr(), (t_rows, t_lens, t_rows, t_lens)
        ds.ds_attention_fwd(b, b + 2 * d, b + 4 * d, o, lse, *table, h, hd, True, max(lens), max(lens), 3 * d, 3 * d, 3 * d, d, T,
                            scratch=scratch, force_generic=force)
        ds.ds_attention_bwd(b, b + 2 * d, b + 4 * d, o, ddo, lse, delta, gb, gb + 2 * d, gb + 4 * d, *table, h, hd, True,
                            max(lens), max(lens), 3 * d, 3 * d, 3 * d, d, T, scratch=scratch, force_generic=force)
        torch.cuda.synchronize()
        res.append(to_np(g)[:, d:])
    for (l, part, pos, val), r0 in zip(cases, rows):
        got, ref = (r[r0:r0 + l] for r in res)
        seen = pos // 32 * 32 + 32                                          # keys from here on do not meet the query
        assert np.isfinite(got[seen:]).all() and np.isfinite(ref[pos + 1:]).all()
        if seen < l:
            for i in range(2):
                assert both_err(got[seen:, i * d:(i + 1) * d], ref[seen:, i * d:(i + 1) * d]) <= TOL[BF]
    assert np.isinf(got[:, d + hd + 5]).all() and np.array_equal(np.isnan(got[:, d:]), np.isnan(ref[:, d:]))       # dV of the last case


@pytest.mark.parametrize("M,N,K,ws_floats,tile", [
    # three stages: one to five K tiles, row edges, the contraction split
    (129, 5632, 64, 0, "128x64"), (129, 5632, 128, 0, "128x64"), (129, 5632, 320, 0, "128x64"), (256, 8192, 320, 0, "128x64"), (641, 512, 4096, 1 << 22, "128x64"),
    # four stages
    (383, 5632, 320, 0, "128x128"), (384, 5632, 320, 0, "128x128"), (385, 5632, 320, 0, "128x128"), (385, 7680, 256, 0, "128x128"), (129, 2304, 8192, 1 << 22, "128x128"),
    # the same with two groups of wavefronts: 32, 33 and, split, more K tiles
    (383, 5632, 2048, 0, "128x128"), (385, 5632, 2112, 0, "128x128"), (129, 2304, 16384, 1 << 22, "128x128"),
    # two stages: two, three and five K tiles, many, the contraction split
    (1281, 6144, 128, 0, "128x128/2"), (513, 7424, 192, 0, "128x128/2"), (767, 6144, 320, 0, "128x128/2"), (768, 6144, 320, 0, "128x128/2"), (769, 6144, 320, 0, "128x128/2"),
    (756, 6144, 2048, 0, "128x128/2"), (385, 4864, 8192, 1 << 22, "128x128/2"),
    # whole tiles of one and three K tiles; whole tiles and a split remainder; every tile split
    (3073, 4608, 64, 0, "256"), (3073, 4608, 192, 0, "256"), (5157, 3328, 1024, 40 << 16, "256 and pieces"), (336, 6144, 8192, 1 << 26, "256 pieces")])
def test_gemm_every_macro_tile_nt(M, N, K, ws_floats, tile):
    """C = A B^T at shapes that the estimates send to each of the macro tiles, whole and split over the contraction (on 256 compute units).
    bf16 results: one rounding, 2^-9 of each value."""
    for epi in (ds.DS_EPI_NONE, ds.DS_EPI_MULR):
        l, = gemm_launches(M, N, K, epilogue=epi, ws_floats=ws_floats)
        assert l["tile"] == tile.split()[0]
        assert (l["pieces"] > 1, l["whole"] > 0) == ("pieces" in tile, "256" in tile and tile != "256 pieces")
    rng = np.random.default_rng(41)
    dA, dB, dR = (to_dev(_rnd(rng, s, BF, f), BF) for s, f in (((M, K), 1.0), ((N, K), 0.1), ((M, N), 1.0)))
    acc = torch.matmul(dA.double(), dB.double().t().contiguous())
    ws = _ws(ws_floats) if ws_floats else None
    c = torch.full((M + 1, N), 7.0, dtype=BF, device=DEV)
    for kw, ref in ((dict(), acc), (dict(epilogue=ds.DS_EPI_MULR, R=dR), acc * dR.double())):
        c.fill_(7.0)
        ds.ds_gemm(dA, dB, c, M, N, K, trans_b=True, workspace=ws, **kw)
        torch.cuda.synchronize()
        assert both_err(to_np(c)[:M], ref.cpu().numpy()) <= 4e-3 and np.all(to_np(c)[M] == 7.0)


@pytest.mark.parametrize("M,N,K,ws_floats,tiles", [
    # one tile for both or for overwriting and adding; one and three (ragged) K tiles, split; four stages, whole and split
    (256, 4352, 33, 0, "128x64"), (256, 4352, 129, 0, "128x64"), (256, 1536, 6000, 1 << 22, "128x64"), (1792, 1792, 577, 0, "128x128 64x64"), (256, 2816, 9001, 1 << 22, "128x128"),
    # two groups of wavefronts: 33 (the last one ragged) and, split, more K tiles
    (1792, 1792, 2049, 0, "128x128"), (256, 2816, 20001, 1 << 22, "128x128"),
    # two stages: two to four K tiles
    (2560, 3328, 129, 0, "256 128x128/2"), (2560, 3328, 200, 0, "256 128x128/2"), (2560, 6656, 65, 0, "128x128/2"),
    # 64-deep K tiles: one, a ragged few, ranges of the contraction, whole tiles and split ones (two pieces and seven)
    (10240, 3328, 1, 0, "256"), (10240, 3328, 97, 0, "256"), (256, 5632, 12000, 1 << 24, "256"), (10240, 3328, 250, 1 << 22, "256"), (9472, 1792, 971, 1 << 24, "256")])
def test_gemm_every_macro_tile_weight_gradient(M, N, K, ws_floats, tiles):
    """The same for weight gradients, overwriting and adding; rows behind the last one hold NaN.  fp32 sums: 1e-5."""
    for adds, tile in zip((False, True), (tiles.split() * 2)[:2]):
        l, = gemm_launches(M, N, K, trans_a=True, epilogue=ds.DS_EPI_ACC32, ws_floats=ws_floats, accumulate=adds)
        assert l["tile"] == tile and (l["splits"] > 1 or l["pieces"] > 1) == (K in (6000, 9001, 20001, 12000, 250, 971))
    rng = np.random.default_rng(42)
    X, dY = _rnd(rng, (K, M), BF), _rnd(rng, (K, N), BF)
    dX, ddY = (torch.cat([to_dev(a, BF), torch.full((64, a.shape[1]), float("nan"), dtype=BF, device=DEV)]) for a in (X, dY))
    ref = torch.matmul(dX[:K].double().t().contiguous(), ddY[:K].double()).cpu().numpy()
    ws = _ws(ws_floats) if ws_floats else None
    c = torch.full((M, N), 3.0, dtype=F32, device=DEV)
    ds.ds_gemm(dX, ddY, c, M, N, K, trans_a=True, epilogue=ds.DS_EPI_ACC32, accumulate=False, workspace=ws)
    torch.cuda.synchronize()
    assert both_err(to_np(c), ref) <= 1e-5
    ds.ds_gemm(dX, ddY, c, M, N, K, trans_a=True, epilogue=ds.DS_EPI_ACC32, accumulate=True, workspace=ws)
    torch.cuda.synchronize()
    assert both_err(to_np(c), 2 * ref) <= 1e-5


@pytest.mark.parametrize("K", [64, 128, 192, 320, 384, 448])
@pytest.mark.parametrize("M", [6145, 6181, 6272])
def test_gemm_ring_of_k_tiles_nt(M, K):
    """256 x 256 tiles whose K loop is shorter than, as long as and longer than the ring of LDS units (one to seven K tiles), persistent
    (800 tiles, three rounds and some behind); the last tile row has 1, 37 and 128 rows."""
    def form(l):
        return len(l) == 1 and l[0]["persistent"] and l[0]["whole"] == 800

    _nt_epilogues_on_device(M, 8192, K, _ws(1 << 22), (ds.DS_EPI_NONE, ds.DS_EPI_RESID, ds.DS_EPI_GATE) if K != 320 else EVERY_EPILOGUE, form)


@pytest.mark.parametrize("M,N,K,tile", [
    *[(M, 3072, K, "192") for M in (3456, 3457, 3647) for K in (64, 128, 192, 320, 448)], (3457, 3072, 576, "192"), (3647, 3072, 2048, "192"),
    *[(M, 8192, K, "128") for M in (769, 897, 1024) for K in (64, 128, 192, 320, 448)], (897, 8192, 576, "128"), (1009, 8192, 2048, "128")])
def test_gemm_lower_tiles_nt(M, N, K, tile):
    """Launches of one round on lower tiles, 192 x 256 and 128 x 256: full last tile rows, ones of a single row and one row short, K
    loops around the length of the ring of LDS units and long ones; every epilogue that goes there on both sides of it and in the long ones."""
    every = [e for e in EVERY_EPILOGUE if tile != "128" or e != ds.DS_EPI_DGELU]

    def form(l):
        return [x["tile"] for x in l] == [tile]

    _nt_epilogues_on_device(M, N, K, _ws(1 << 22), every if K in (192, 576, 2048) else (ds.DS_EPI_NONE, ds.DS_EPI_RESID), form)


@pytest.mark.parametrize("K", [1, 63, 65, 128, 200, 321, 450])
def test_gemm_ring_of_k_tiles_weight_gradient(K):
    """The same for weight gradients (576 tiles, one work-group each): one to eight K tiles, the last one ragged, overwriting and adding; rows
    behind the last one hold NaN.  fp32 sums: 1e-5."""
    M, N = 8192, 4608
    assert gemm_launches(M, N, K, trans_a=True, epilogue=ds.DS_EPI_ACC32)[0]["whole"] == 576
    rng = np.random.default_rng(44)
    dX, ddY = (torch.cat([to_dev(_rnd(rng, (K, n), BF), BF), torch.full((64, n), float("nan"), dtype=BF, device=DEV)]) for n in (M, N))
    ref = torch.matmul(dX[:K].double().t().contiguous(), ddY[:K].double())
    c = torch.full((M, N), 3.0, dtype=F32, device=DEV)
    for times in (1, 2):
        ds.ds_gemm(dX, ddY, c, M, N, K, trans_a=True, epilogue=ds.DS_EPI_ACC32, accumulate=times == 2)
        torch.cuda.synchronize()
        want = times * ref
        assert float((c.double() - want).norm() / want.norm()) <= 1e-5
        assert bool(((c.double() - want).abs() <= 1e-5 * (8 * want.square().mean().sqrt() + want.abs())).all())


@pytest.mark.parametrize("M,N,K,tile", [
    (300, 2304, 512, "64x64"), (129, 5632, 128, "128x64"), (385, 7680, 256, "128x128"), (1281, 6144, 128, "128x128/2"),
    (897, 8192, 192, "128"), (1537, 3840, 1024, "128"), (3457, 3072, 192, "192"),
    (3073, 4608, 64, "256"), (4133, 8192, 128, "256"), (10713, 4608, 512, "256")])              # (the last two persistent)
def test_gemm_bias_is_the_last_term(M, N, K, tile):
    """Products 2^24 and -2^24 at the two ends of the contraction cancel before the bias is added, on whatever tile: the output is the bias
    itself (a sum that starts with the bias loses it)."""
    rng = np.random.default_rng(46)
    a, b = torch.zeros((M, K), dtype=BF, device=DEV), torch.zeros((N, K), dtype=BF, device=DEV)
    a[:, 0] = a[:, K - 1] = 4096.0
    b[:, 0], b[:, K - 1] = 4096.0, -4096.0
    bias = to_dev(_rnd(rng, (N,), BF), BF)
    r = to_dev(_rnd(rng, (M, N), BF), BF)
    want = bias.float().expand(M, N)
    c, c2 = (torch.empty((M, N), dtype=BF, device=DEV) for _ in range(2))
    for epi, kw, ref in ((ds.DS_EPI_NONE, {}, want), (ds.DS_EPI_RESID, dict(R=r), want + r.float()), (ds.DS_EPI_GELU, {}, want),
                         (ds.DS_EPI_GATE, dict(R=r), want), (ds.DS_EPI_MULR, dict(R=r), want * r.float())):
        assert [x["tile"] for x in gemm_launches(M, N, K, epilogue=epi)] == [tile]
        ds.ds_gemm(a, b, c, M, N, K, trans_b=True, epilogue=epi, bias=bias, C2=c2, **kw)
        torch.cuda.synchronize()
        assert torch.equal(c, ref.to(BF)), epi


@pytest.mark.parametrize("generic", [False, True])
def test_gelu_derivative_from_the_logistic_term(generic):
    """fp32, arguments that are powers of two: GELU(z) / z is the logistic term s, and GELU'(z) = s (1 + z (1 - s) 2 u') in that order of
    operations (what a stage's outputs depend on from one version to the next), bit for bit."""
    f32 = np.float32
    z = np.array([sign * 2.0 ** e for e in range(-12, 4) for sign in (1, -1)], f32)
    M, N, K = 64, z.size, 8
    a, b = torch.zeros((M, K), device=DEV), torch.zeros((N, K), device=DEV)
    a[:, 0] = 1.0
    b[:, 0] = torch.from_numpy(z).to(DEV)
    grad, gelu = (torch.empty((M, N), device=DEV) for _ in range(2))
    ds.ds_gemm(a, b, grad, M, N, K, trans_b=True, epilogue=ds.DS_EPI_GELU_D, C2=gelu, force_generic=generic)
    back = torch.empty((M, N), device=DEV)
    b[:, 0] = 1.0
    ds.ds_gemm(a, b, back, M, N, K, trans_b=True, epilogue=ds.DS_EPI_DGELU, R=torch.from_numpy(z).to(DEV).expand(M, N).contiguous(), force_generic=generic)
    torch.cuda.synchronize()

    def fma(x, y, t):                                       # (the product is exact in 64 bits)
        return f32(np.float64(x) * np.float64(y) + np.float64(t))

    c2 = f32(2) * f32(0.7978845608028654)
    c6a = f32(3) * f32(0.044715) * c2
    for i in range(N):
        s = f32(gelu[0, i].item()) / z[i]
        assert abs(float(s) - 1 / (1 + np.exp(-2 * 0.7978845608028654 * (float(z[i]) + 0.044715 * float(z[i]) ** 3)))) <= 2e-6
        want = s * fma(z[i] * fma(c6a, z[i] * z[i], c2), f32(1) - s, f32(1))
        assert bool((grad[:, i] == float(want)).all()) and bool((back[:, i] == float(want)).all()), z[i]


@pytest.mark.parametrize("N", [(1 << 24) - 256, 1 << 24])
def test_gemm_widest_outputs_nt(N):
    """The widest output on 256 x 256 tiles (128 rows of bf16 are 2^32 - 65 536 bytes) and the next one, on smaller tiles; 130 rows.  Every column
    against others of the same product where it is cheap: all rows of 4 096 columns, and the row behind the last one."""
    M, K = 130, 64
    assert gemm_launches(M, N, K, epilogue=ds.DS_EPI_MULR)[0]["tile"] == ("256" if N < 1 << 24 else "64x64")
    gen = torch.Generator(device=DEV)
    gen.manual_seed(6)
    a = torch.randn((M, K), device=DEV, generator=gen).to(BF)
    b = torch.empty((N, K), dtype=BF, device=DEV)
    r = torch.empty((M, N), dtype=BF, device=DEV)
    for t in (b, r):
        for part in t.view(-1).split(1 << 26):
            part.copy_(torch.randn(part.numel(), device=DEV, generator=gen))
    c = torch.full((M + 1, N), 7.0, dtype=BF, device=DEV)
    ds.ds_gemm(a, b, c, M, N, K, trans_b=True, epilogue=ds.DS_EPI_MULR, R=r)
    torch.cuda.synchronize()
    cols = torch.cat([torch.arange(512), torch.arange(N - 512, N), torch.randint(0, N, (3072,), generator=torch.Generator().manual_seed(7))]).to(DEV)
    want = torch.matmul(a.double(), b[cols].double().t().contiguous()) * r[:, cols].double()
    got = c[:M][:, cols].double()
    assert float((got - want).norm() / want.norm()) <= 4e-3
    assert bool(((got - want).abs() <= 4e-3 * (8 * want.square().mean().sqrt() + want.abs())).all())
    assert bool((c[M] == 7.0).all())


@pytest.mark.parametrize("M,N", [(256, (1 << 23) - 256), (256, 1 << 23), (1 << 23, 256)])
def test_gemm_widest_weight_gradients(M, N):
    """The same for weight gradients of three tokens: fp32 outputs of 2^31 elements; 256 x 256 tiles up to 2^23 - 256 columns."""
    K = 3
    assert gemm_launches(M, N, K, trans_a=True, epilogue=ds.DS_EPI_ACC32)[0]["tile"] == ("128x128/2" if N == 1 << 23 else "256")
    gen = torch.Generator(device=DEV)
    gen.manual_seed(8)
    x, dy = (torch.randn((K, n), device=DEV, generator=gen).to(BF) for n in (M, N))
    c = torch.full((M, N), 7.0, device=DEV)
    ds.ds_gemm(x, dy, c, M, N, K, trans_a=True, epilogue=ds.DS_EPI_ACC32)
    torch.cuda.synchronize()
    for i in range(0, max(M, N), 1 << 20):                   # (in pieces along the wide side)
        s = slice(i, min(i + (1 << 20), max(M, N)))
        got, want = (c[:, s], x.float().t() @ dy[:, s].float()) if N > M else (c[s], x[:, s].float().t() @ dy.float())
        assert bool(((got - want).abs() <= 1e-5).all()), i      # three products of a few units each: 2^-23 of their sum


def test_gemm_weight_gradient_pieces_of_whole_steps():
    """A contraction is cut into pieces of whole 32-row steps, the products' depth: of 375 steps ten times 35 and once 25.  Every step adds 1, and 2^24 in
    the first row swallows the ones of its own piece, one at a time (2^24 + 1 rounds back); the others are counted exactly and added piece by piece."""
    M, N, K = 256, 5632, 12000
    l, = gemm_launches(M, N, K, trans_a=True, epilogue=ds.DS_EPI_ACC32, ws_floats=1 << 24)
    assert (l["tile"], l["splits"]) == ("256", 11)
    x, dy = torch.zeros((K, M), dtype=BF, device=DEV), torch.zeros((K, N), dtype=BF, device=DEV)
    x[::32] = 1.0
    dy[::32] = 1.0
    x[0] = dy[0] = 4096.0
    c = torch.zeros((M, N), dtype=F32, device=DEV)
    ds.ds_gemm(x, dy, c, M, N, K, trans_a=True, epilogue=ds.DS_EPI_ACC32, workspace=_ws(1 << 24))
    torch.cuda.synchronize()
    want = np.float32(2 ** 24)
    for n in [35] * 9 + [25]:
        want = np.float32(want + np.float32(n))
    assert bool((c == float(want)).all()), (c.unique(), want)
