"""Token-wise chunked neighbours (Sec. 5.4): oracle pins and host-side checks (no GPU), and GPU
parity of libfpdt_tokenwise.so against the oracle."""
import math
import os
import re
import subprocess
import sys

import numpy as np
import pytest
import torch

import launch_rules
from oracle import tokenwise as otw
from paper_2408_16978_amd import tokenwise as TW

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


# ------------------------------------------------------------------ oracle pins (CPU)
def test_cross_entropy_oracle_against_torch_autograd():
    r = np.random.default_rng(1)
    rows, hidden, vocab = 37, 16, 53
    H, W = r.standard_normal((rows, hidden)), r.standard_normal((vocab, hidden))
    t = r.integers(0, vocab, rows)
    out = otw.cross_entropy(H, W, t, grad_scale=0.25)
    h = torch.tensor(H, requires_grad=True)
    w = torch.tensor(W, requires_grad=True)
    loss = torch.nn.functional.cross_entropy(h @ w.T, torch.tensor(t), reduction="none")
    (0.25 * loss.sum()).backward()
    np.testing.assert_allclose(out["loss"], loss.detach().numpy(), rtol=1e-12, atol=1e-12)
    np.testing.assert_allclose(out["lse"], torch.logsumexp(h @ w.T, dim=1).detach().numpy(), rtol=1e-12)
    np.testing.assert_allclose(out["dH"], h.grad.numpy(), rtol=1e-11, atol=1e-13)
    np.testing.assert_allclose(out["dW"], w.grad.numpy(), rtol=1e-11, atol=1e-13)


def test_cross_entropy_oracle_closed_forms():
    r = np.random.default_rng(2)
    rows, hidden, vocab = 9, 4, 11
    H = r.standard_normal((rows, hidden))
    t = r.integers(0, vocab, rows)
    # W = 0: uniform distribution, loss = log(vocab), dH = 0, dW = (1/vocab - onehot)^T H
    out = otw.cross_entropy(H, np.zeros((vocab, hidden)), t)
    np.testing.assert_allclose(out["loss"], math.log(vocab), rtol=1e-15)
    np.testing.assert_allclose(out["dH"], 0.0, atol=1e-15)
    G = np.full((rows, vocab), 1.0 / vocab)
    G[np.arange(rows), t] -= 1.0
    np.testing.assert_allclose(out["dW"], G.T @ H, atol=1e-14)
    # the gradient with respect to the logits sums to zero per row: sum_v dW[v, :] = 0
    W = r.standard_normal((vocab, hidden))
    out = otw.cross_entropy(H, W, t)
    np.testing.assert_allclose(out["dW"].sum(axis=0), 0.0, atol=1e-13)
    # shifting every logit of a row by a constant (H -> H, W -> W + 1 u^T with H u = const) ...
    # simpler shift invariance: adding the same vector to every row of W adds H_r . v to all
    # logits of row r, which changes neither the loss nor dH's projection on that direction
    v = r.standard_normal(hidden)
    out2 = otw.cross_entropy(H, W + v, t)
    np.testing.assert_allclose(out2["loss"], out["loss"], atol=1e-12)


@pytest.mark.parametrize("swiglu", [False, True])
def test_ffn_and_linear_oracles_against_torch_autograd(swiglu):
    r = np.random.default_rng(3 + swiglu)
    rows, n_model, n_ffn = 23, 12, 29
    X, dY = r.standard_normal((rows, n_model)), r.standard_normal((rows, n_model))
    W1, W3 = r.standard_normal((n_ffn, n_model)), r.standard_normal((n_ffn, n_model))
    W2 = r.standard_normal((n_model, n_ffn))
    out = otw.ffn(X, W1, W2, W3 if swiglu else None, dY)
    x, w1, w3, w2 = (torch.tensor(a, requires_grad=True) for a in (X, W1, W3, W2))
    F = torch.nn.functional
    y = (F.silu(x @ w1.T) * (x @ w3.T)) @ w2.T if swiglu else F.gelu(x @ w1.T) @ w2.T
    (y * torch.tensor(dY)).sum().backward()
    np.testing.assert_allclose(out["Y"], y.detach().numpy(), rtol=1e-11, atol=1e-12)
    for k, t in (("dX", x), ("dW1", w1), ("dW2", w2)) + ((("dW3", w3),) if swiglu else ()):
        np.testing.assert_allclose(out[k], t.grad.numpy(), rtol=1e-10, atol=1e-11, err_msg=k)
    assert ("dW3" in out) == swiglu
    # the linear projection is the FFN's first GEMM: pin it the same way
    x2, w = torch.tensor(X, requires_grad=True), torch.tensor(W1, requires_grad=True)
    dy2 = r.standard_normal((rows, n_ffn))
    lin = otw.linear(X, W1, dY=dy2)
    ((x2 @ w.T) * torch.tensor(dy2)).sum().backward()
    np.testing.assert_allclose(lin["Y"], (x2 @ w.T).detach().numpy(), rtol=1e-12, atol=1e-13)
    np.testing.assert_allclose(lin["dX"], x2.grad.numpy(), rtol=1e-12, atol=1e-13)
    np.testing.assert_allclose(lin["dW"], w.grad.numpy(), rtol=1e-12, atol=1e-13)


def test_ffn_oracle_closed_forms_and_finite_differences():
    r = np.random.default_rng(5)
    rows, n_model, n_ffn = 5, 4, 6
    X = r.standard_normal((rows, n_model))
    W1, W3 = r.standard_normal((n_ffn, n_model)), r.standard_normal((n_ffn, n_model))
    W2 = r.standard_normal((n_model, n_ffn))
    # gelu(0) = silu(0) = 0: X = 0 gives Y = 0; gelu'(0) = silu'(0) = 1/2
    z = np.zeros_like(X)
    assert np.all(otw.ffn(z, W1, W2)["Y"] == 0) and np.all(otw.ffn(z, W1, W2, W3)["Y"] == 0)
    dY = r.standard_normal((rows, n_model))
    np.testing.assert_allclose(otw.ffn(z, W1, W2, None, dY)["dX"], 0.5 * dY @ W2 @ W1, atol=1e-14)
    # large positive pre-activations: gelu(a) -> a, so the block is the product of its two matrices
    Xp, W1p = np.abs(X) + 1, np.abs(W1) * 10 + 10
    np.testing.assert_allclose(otw.ffn(Xp, W1p, W2)["Y"], Xp @ W1p.T @ W2.T, rtol=1e-12)
    # large negative: gelu(a) -> 0
    np.testing.assert_allclose(otw.ffn(Xp, -W1p, W2)["Y"], 0, atol=1e-12)
    # SwiGLU is linear in W3 and in W2
    a = otw.ffn(X, W1, W2, W3)["Y"]
    np.testing.assert_allclose(otw.ffn(X, W1, W2, 3 * W3)["Y"], 3 * a, rtol=1e-13)
    # central finite differences of L = sum(Y * dY) in one coordinate of each argument
    eps = 1e-6
    for sw in (False, True):
        g = otw.ffn(X, W1, W2, W3 if sw else None, dY)
        L = lambda X_, W1_, W2_, W3_: float((otw.ffn(X_, W1_, W2_, W3_ if sw else None)["Y"] * dY).sum())
        for name, arr, idx in (("dX", 0, (2, 1)), ("dW1", 1, (3, 2)), ("dW2", 2, (1, 4))) + ((("dW3", 3, (5, 0)),) if sw else ()):
            args_p = [X.copy(), W1.copy(), W2.copy(), W3.copy()]
            args_m = [X.copy(), W1.copy(), W2.copy(), W3.copy()]
            args_p[arr][idx] += eps
            args_m[arr][idx] -= eps
            fd = (L(*args_p) - L(*args_m)) / (2 * eps)
            assert abs(fd - g[name][idx]) < 1e-6 * max(1.0, abs(fd)), (sw, name, fd, g[name][idx])


# ------------------------------------------------------------------ host-side ABI checks (CPU)
def test_tokenwise_library_exports_and_rejects_bad_arguments():
    text = open(os.path.join(ROOT, "include", "fpdt_tokenwise.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    names = sorted(set(re.findall(r"\b(fpdt_tw_[a-z_0-9]+)\s*\(", text)))
    assert {"fpdt_tw_loss_fwd_bwd", "fpdt_tw_loss_workspace_bytes", "fpdt_tw_last_error"} <= set(names)
    L = TW.load()
    for n in names:
        assert hasattr(L, n), n
        assert callable(getattr(TW, n)), n
    # chunk = ceil(rows / n_chunks): fp32 logits + bf16 gradient of one chunk, each 256-aligned
    assert TW.fpdt_tw_loss_workspace_bytes(1000, 64, 512, 3) == 334 * 512 * 4 + (334 * 512 * 2 + 255) // 256 * 256
    assert TW.fpdt_tw_loss_workspace_bytes(0, 64, 512, 1) == 0
    assert TW.fpdt_tw_loss_workspace_bytes(10, 64, 512, 11) == 0
    p = 0x1000
    call = lambda **kw: L.fpdt_tw_loss_fwd_bwd(*[kw.get(k, d) for k, d in (
        ("H", p), ("W", p), ("t", p), ("gs", 1.0), ("loss", p), ("lse", p), ("dH", p), ("dW", p), ("rows", 1024),
        ("hidden", 64), ("vocab", 512), ("n", 4), ("ws", 0x100000), ("wsb", 1 << 40), ("st", None))])
    assert call(H=None) == 1 and "NULL" in TW.fpdt_tw_last_error()
    assert call(rows=0) == 1
    assert call(n=0) == 1
    assert call(n=2000) == 1
    assert call(gs=float("nan")) == 1
    assert call(ws=None) == 3
    assert call(wsb=16) == 3
    assert call(ws=0x100010) == 3
    # feed-forward workspace: [chunk, n_ffn] bf16 tiles, 2 (GELU) or 3 (SwiGLU), one more backward
    tile = (250 * 1024 * 2 + 255) // 256 * 256
    assert TW.fpdt_tw_ffn_workspace_bytes(1000, 256, 1024, TW.FPDT_TW_GELU, 4, False) == 2 * tile
    assert TW.fpdt_tw_ffn_workspace_bytes(1000, 256, 1024, TW.FPDT_TW_SWIGLU, 4, False) == 3 * tile
    assert TW.fpdt_tw_ffn_workspace_bytes(1000, 256, 1024, TW.FPDT_TW_SWIGLU, 4, True) == 4 * tile
    assert TW.fpdt_tw_ffn_workspace_bytes(1000, 256, 1024, 7, 4, True) == 0
    assert L.fpdt_tw_ffn_fwd(p, p, None, p, p, 1000, 256, 1024, TW.FPDT_TW_SWIGLU, 4, 0x100000, 1 << 40, None) == 1
    assert "W3" in TW.fpdt_tw_last_error()
    assert L.fpdt_tw_ffn_fwd(p, p, None, p, p, 1000, 256, 1024, TW.FPDT_TW_GELU, 4, 0x100000, 16, None) == 3
    assert L.fpdt_tw_ffn_bwd(p, p, None, p, p, None, None, None, None, 1000, 256, 1024, TW.FPDT_TW_GELU, 4,
                             0x100000, 1 << 40, None) == 1
    assert L.fpdt_tw_linear_fwd(p, p, None, 1000, 256, 768, 4, None) == 1
    assert L.fpdt_tw_linear_fwd(p, p, p, 1000, 256, 768, 0, None) == 1
    assert L.fpdt_tw_linear_bwd(p, p, p, None, None, 1000, 0, 768, 4, None) == 1


# ------------------------------------------------------------------ GPU parity
def _case(rows, hidden, vocab, seed):
    g = torch.Generator().manual_seed(seed)
    H = torch.randn(rows, hidden, generator=g).to(torch.bfloat16)
    W = (torch.randn(vocab, hidden, generator=g) * hidden ** -0.5).to(torch.bfloat16)
    t = torch.randint(0, vocab, (rows,), generator=g, dtype=torch.int32)
    return H, W, t


@pytest.mark.gpu
@pytest.mark.parametrize("rows,hidden,vocab,n_chunks", [(1000, 256, 1536, 3), (512, 128, 4099, 8), (96, 64, 320, 1)])
def test_gpu_loss_matches_oracle(rows, hidden, vocab, n_chunks):
    print("[case] chunked loss", rows, hidden, vocab, n_chunks, flush=True)
    H, W, t = _case(rows, hidden, vocab, 31)
    ref = otw.cross_entropy(H.double().numpy(), W.double().numpy(), t.numpy(), grad_scale=1.0 / rows)
    Hd, Wd, td = H.cuda(), W.cuda(), t.cuda()
    loss = torch.empty(rows, device="cuda")
    lse = torch.empty(rows, device="cuda")
    dH = torch.empty_like(Hd)
    dW = torch.zeros(vocab, hidden, device="cuda")
    ws = torch.empty(TW.fpdt_tw_loss_workspace_bytes(rows, hidden, vocab, n_chunks), dtype=torch.uint8, device="cuda")
    TW.fpdt_tw_loss_fwd_bwd(Hd, Wd, td, 1.0 / rows, loss, lse, dH, dW, n_chunks, ws)
    torch.cuda.synchronize()
    # logits are exact bf16 products accumulated in fp32: loss and lse to fp32 round-off
    np.testing.assert_allclose(loss.cpu().numpy(), ref["loss"], atol=2e-4)
    np.testing.assert_allclose(lse.cpu().numpy(), ref["lse"], atol=2e-4)
    # gradients: the logit gradient is rounded to bf16 before its two GEMMs and dH is stored in
    # bf16: per row (dH) / per vocabulary row (dW) 2e-2 of the reference row's RMS + storage half-ulp
    for name, got, r in (("dH", dH.float().cpu().numpy(), ref["dH"]), ("dW", dW.cpu().numpy(), ref["dW"])):
        rms = np.sqrt((r ** 2).mean(axis=1, keepdims=True))
        budget = 2e-2 * rms + 2.0 ** -9 * np.abs(r) + 1e-9
        assert (np.abs(got - r) <= budget).all(), (name, float((np.abs(got - r) / budget).max()))
    # dW is accumulated into: a second call doubles it; the chunk count does not change anything
    # beyond fp32 summation order
    TW.fpdt_tw_loss_fwd_bwd(Hd, Wd, td, 1.0 / rows, loss, lse, dH, dW, n_chunks, ws)
    torch.cuda.synchronize()
    np.testing.assert_allclose(dW.cpu().numpy(), 2 * ref["dW"], atol=2 * float(np.abs(ref["dW"]).max()) * 2e-2 + 1e-9)
    if n_chunks > 1:
        loss1 = torch.empty(rows, device="cuda")
        ws1 = torch.empty(TW.fpdt_tw_loss_workspace_bytes(rows, hidden, vocab, 1), dtype=torch.uint8, device="cuda")
        TW.fpdt_tw_loss_fwd_bwd(Hd, Wd, td, 1.0 / rows, loss1, lse, None, None, 1, ws1)
        torch.cuda.synchronize()
        np.testing.assert_allclose(loss1.cpu().numpy(), loss.cpu().numpy(), atol=1e-5)
        assert ws.numel() < ws1.numel()


@pytest.mark.gpu
def test_gpu_loss_rejects_small_workspace():
    H, W, t = _case(64, 64, 128, 32)
    out = torch.empty(64, device="cuda")
    ws = torch.empty(256, dtype=torch.uint8, device="cuda")
    with pytest.raises(TW.FpdtTwError) as e:
        TW.fpdt_tw_loss_fwd_bwd(H.cuda(), W.cuda(), t.cuda(), 1.0, out, out.clone(), None, None, 1, ws)
    assert e.value.status == 3


def _rowwise_ok(name, got, ref, rel=2e-2):
    """|got - ref| <= rel * rms(ref row) + half a bf16 ulp of ref (at most 2^-8 |ref|: 8 significand
    bits), element by element."""
    rms = np.sqrt((ref ** 2).mean(axis=1, keepdims=True))
    budget = rel * rms + 2.0 ** -8 * np.abs(ref) + 1e-9
    err = np.abs(got - ref)
    assert (err <= budget).all(), (name, float((err / budget).max()))


@pytest.mark.gpu
@pytest.mark.parametrize("rows,n_in,n_out,n_chunks", [(1000, 256, 768, 3), (333, 136, 520, 7)])
def test_gpu_linear_matches_oracle(rows, n_in, n_out, n_chunks):
    print("[case] chunked linear", rows, n_in, n_out, n_chunks, flush=True)
    g = torch.Generator().manual_seed(41)
    X = torch.randn(rows, n_in, generator=g).to(torch.bfloat16)
    W = (torch.randn(n_out, n_in, generator=g) * n_in ** -0.5).to(torch.bfloat16)
    dY = torch.randn(rows, n_out, generator=g).to(torch.bfloat16)
    ref = otw.linear(X.double().numpy(), W.double().numpy(), dY.double().numpy())
    Xd, Wd, dYd = X.cuda(), W.cuda(), dY.cuda()
    Y = torch.empty(rows, n_out, dtype=torch.bfloat16, device="cuda")
    dX = torch.empty_like(Xd)
    dW = torch.zeros(n_out, n_in, device="cuda")
    TW.fpdt_tw_linear_fwd(Xd, Wd, Y, n_chunks)
    TW.fpdt_tw_linear_bwd(Xd, Wd, dYd, dX, dW, n_chunks)
    torch.cuda.synchronize()
    # fp32 accumulation of exact products, one rounding to bf16 on store
    _rowwise_ok("Y", Y.float().cpu().numpy(), ref["Y"], rel=1e-4)
    _rowwise_ok("dX", dX.float().cpu().numpy(), ref["dX"], rel=1e-4)
    np.testing.assert_allclose(dW.cpu().numpy(), ref["dW"], atol=1e-4 * float(np.abs(ref["dW"]).max()))
    # one chunk gives the same bits for Y and dX (each row is its own dot products)
    Y1, dX1 = torch.empty_like(Y), torch.empty_like(dX)
    TW.fpdt_tw_linear_fwd(Xd, Wd, Y1, 1)
    TW.fpdt_tw_linear_bwd(Xd, Wd, dYd, dX1, None, 1)
    torch.cuda.synchronize()
    _rowwise_ok("Y vs one chunk", Y.float().cpu().numpy(), Y1.float().cpu().numpy().astype(np.float64), rel=1e-4)
    _rowwise_ok("dX vs one chunk", dX.float().cpu().numpy(), dX1.float().cpu().numpy().astype(np.float64), rel=1e-4)


@pytest.mark.gpu
@pytest.mark.parametrize("act,rows,n_model,n_ffn,n_chunks", [
    ("gelu", 1000, 256, 1024, 4), ("swiglu", 1000, 256, 688, 4), ("swiglu", 257, 128, 349, 5), ("gelu", 64, 64, 256, 1)])
def test_gpu_ffn_matches_oracle(act, rows, n_model, n_ffn, n_chunks):
    print("[case] chunked ffn", act, rows, n_model, n_ffn, n_chunks, flush=True)
    sw = act == "swiglu"
    code = TW.FPDT_TW_SWIGLU if sw else TW.FPDT_TW_GELU
    g = torch.Generator().manual_seed(43)
    X = torch.randn(rows, n_model, generator=g).to(torch.bfloat16)
    W1 = (torch.randn(n_ffn, n_model, generator=g) * n_model ** -0.5).to(torch.bfloat16)
    W3 = (torch.randn(n_ffn, n_model, generator=g) * n_model ** -0.5).to(torch.bfloat16)
    W2 = (torch.randn(n_model, n_ffn, generator=g) * n_ffn ** -0.5).to(torch.bfloat16)
    dY = torch.randn(rows, n_model, generator=g).to(torch.bfloat16)
    f64 = lambda t: t.double().numpy()
    ref = otw.ffn(f64(X), f64(W1), f64(W2), f64(W3) if sw else None, f64(dY))
    Xd, W1d, W2d, dYd = X.cuda(), W1.cuda(), W2.cuda(), dY.cuda()
    W3d = W3.cuda() if sw else None
    Y, dX = torch.empty_like(Xd), torch.empty_like(Xd)
    dW1 = torch.zeros(n_ffn, n_model, device="cuda")
    dW3 = torch.zeros(n_ffn, n_model, device="cuda") if sw else None
    dW2 = torch.zeros(n_model, n_ffn, device="cuda")
    wf = torch.empty(TW.fpdt_tw_ffn_workspace_bytes(rows, n_model, n_ffn, code, n_chunks, False), dtype=torch.uint8, device="cuda")
    wb = torch.empty(TW.fpdt_tw_ffn_workspace_bytes(rows, n_model, n_ffn, code, n_chunks, True), dtype=torch.uint8, device="cuda")
    TW.fpdt_tw_ffn_fwd(Xd, W1d, W3d, W2d, Y, code, n_chunks, wf)
    TW.fpdt_tw_ffn_bwd(Xd, W1d, W3d, W2d, dYd, dX, dW1, dW3, dW2, code, n_chunks, wb)
    torch.cuda.synchronize()
    # intermediates [chunk, n_ffn] are rounded to bf16 between GEMMs (relative 2^-9 each, independent
    # across the contraction): 2e-2 of the reference row's RMS covers them with a wide margin
    _rowwise_ok("Y", Y.float().cpu().numpy(), ref["Y"])
    _rowwise_ok("dX", dX.float().cpu().numpy(), ref["dX"])
    _rowwise_ok("dW1", dW1.cpu().numpy(), ref["dW1"])
    _rowwise_ok("dW2", dW2.cpu().numpy(), ref["dW2"])
    if sw:
        _rowwise_ok("dW3", dW3.cpu().numpy(), ref["dW3"])
    # the weight gradients are accumulated into, dX is overwritten
    TW.fpdt_tw_ffn_bwd(Xd, W1d, W3d, W2d, dYd, dX, dW1, None, None, code, n_chunks, wb)
    torch.cuda.synchronize()
    _rowwise_ok("dW1 twice", dW1.cpu().numpy(), 2 * ref["dW1"])
    _rowwise_ok("dX again", dX.float().cpu().numpy(), ref["dX"])
    _rowwise_ok("dW2 untouched", dW2.cpu().numpy(), ref["dW2"])
    if n_chunks > 1:
        w1 = TW.fpdt_tw_ffn_workspace_bytes(rows, n_model, n_ffn, code, 1, True)
        assert wb.numel() * 2 < w1


# ------------------------------------------------------------------ Llama-8B widths, sampled
@pytest.mark.gpu
def test_gpu_ffn_llama_widths_sampled_rows_and_weight_slices():
    """Model 4096, FFN 14336, SwiGLU, 8192 tokens in 4 chunks.  Rows are independent, so the
    oracle evaluated on sampled rows gives their Y and dX exactly; a hidden unit's weight
    gradients depend only on its own column of the intermediates, so the oracle evaluated on
    a slice of hidden units gives those rows of dW1 / dW3 and columns of dW2 exactly."""
    rows, n_model, n_ffn, n_chunks = 8192, 4096, 14336, 4
    print("[case] ffn llama widths", rows, n_model, n_ffn, n_chunks, flush=True)
    g = torch.Generator(device="cuda").manual_seed(47)
    bf = lambda *s, std=1.0: (torch.randn(*s, device="cuda", generator=g) * std).to(torch.bfloat16)
    X, dY = bf(rows, n_model), bf(rows, n_model)
    W1, W3, W2 = bf(n_ffn, n_model, std=n_model ** -0.5), bf(n_ffn, n_model, std=n_model ** -0.5), bf(n_model, n_ffn, std=n_ffn ** -0.5)
    code = TW.FPDT_TW_SWIGLU
    Y, dX = torch.empty_like(X), torch.empty_like(X)
    dW1, dW3, dW2 = (torch.zeros_like(w, dtype=torch.float32) for w in (W1, W3, W2))
    wb = torch.empty(TW.fpdt_tw_ffn_workspace_bytes(rows, n_model, n_ffn, code, n_chunks, True), dtype=torch.uint8, device="cuda")
    TW.fpdt_tw_ffn_fwd(X, W1, W3, W2, Y, code, n_chunks, wb)
    TW.fpdt_tw_ffn_bwd(X, W1, W3, W2, dY, dX, dW1, dW3, dW2, code, n_chunks, wb)
    torch.cuda.synchronize()
    f64 = lambda t: t.double().cpu().numpy()
    r = np.random.default_rng(5)
    rs = np.sort(r.choice(rows, 24, replace=False))
    rs[0], rs[-1] = 0, rows - 1
    ref = otw.ffn(f64(X[rs]), f64(W1), f64(W2), f64(W3), f64(dY[rs]))
    _rowwise_ok("Y rows", f64(Y[rs]), ref["Y"])
    _rowwise_ok("dX rows", f64(dX[rs]), ref["dX"])
    del ref
    fs = np.sort(r.choice(n_ffn, 12, replace=False))
    fs[0], fs[-1] = 0, n_ffn - 1
    ref = otw.ffn(f64(X), f64(W1[fs]), f64(W2[:, fs]), f64(W3[fs]), f64(dY))
    _rowwise_ok("dW1 slice", f64(dW1[fs]), ref["dW1"])
    _rowwise_ok("dW3 slice", f64(dW3[fs]), ref["dW3"])
    _rowwise_ok("dW2 slice", f64(dW2[:, fs]).T.copy(), ref["dW2"].T.copy())


@pytest.mark.gpu
def test_gpu_loss_llama_vocabulary():
    """Hidden 4096, vocabulary 128256 (Llama-3), 1024 tokens in 4 chunks, against the full oracle."""
    rows, hidden, vocab, n_chunks = 1024, 4096, 128256, 4
    print("[case] loss llama vocabulary", rows, hidden, vocab, n_chunks, flush=True)
    g = torch.Generator(device="cuda").manual_seed(53)
    H = torch.randn(rows, hidden, device="cuda", generator=g).to(torch.bfloat16)
    W = (torch.randn(vocab, hidden, device="cuda", generator=g) * hidden ** -0.5).to(torch.bfloat16)
    t = torch.randint(0, vocab, (rows,), device="cuda", generator=g, dtype=torch.int32)
    loss, lse = torch.empty(rows, device="cuda"), torch.empty(rows, device="cuda")
    dH = torch.empty_like(H)
    dW = torch.zeros(vocab, hidden, device="cuda")
    ws = torch.empty(TW.fpdt_tw_loss_workspace_bytes(rows, hidden, vocab, n_chunks), dtype=torch.uint8, device="cuda")
    TW.fpdt_tw_loss_fwd_bwd(H, W, t, 1.0 / rows, loss, lse, dH, dW, n_chunks, ws)
    torch.cuda.synchronize()
    print("[step] oracle", flush=True)
    ref = otw.cross_entropy(H.double().cpu().numpy(), W.double().cpu().numpy(), t.cpu().numpy(), grad_scale=1.0 / rows)
    print("[step] compare", flush=True)
    # 4096-term fp32 dot products of O(1) logits: a few 1e-5 of round-off each
    np.testing.assert_allclose(loss.cpu().numpy(), ref["loss"], atol=1e-3)
    np.testing.assert_allclose(lse.cpu().numpy(), ref["lse"], atol=1e-3)
    _rowwise_ok("dH", dH.float().cpu().numpy(), ref["dH"])
    # a vocabulary row that is nobody's target has a gradient of ~1024 probabilities of ~1e-5 each,
    # every one rounded to bf16 before the GEMM: same relative budget per row
    _rowwise_ok("dW", dW.cpu().numpy(), ref["dW"])


@pytest.mark.gpu
def test_gpu_tokenwise_calls_replay_from_a_graph():
    """FFN forward + backward and the fused loss captured in one HIP graph (library GEMMs and the
    row / activation kernels on the captured stream), replayed three times with eager work in
    between; every replay equals the eager result bit for bit."""
    rows, n_model, n_ffn, vocab, n_chunks = 1024, 256, 688, 1536, 4
    print("[case] token-wise graph", rows, n_model, n_ffn, vocab, flush=True)
    g = torch.Generator(device="cuda").manual_seed(61)
    bf = lambda *s, std=1.0: (torch.randn(*s, device="cuda", generator=g) * std).to(torch.bfloat16)
    X, dY = bf(rows, n_model), bf(rows, n_model)
    W1, W3, W2 = bf(n_ffn, n_model, std=n_model ** -0.5), bf(n_ffn, n_model, std=n_model ** -0.5), bf(n_model, n_ffn, std=n_ffn ** -0.5)
    Wv = bf(vocab, n_model, std=n_model ** -0.5)
    tgt = torch.randint(0, vocab, (rows,), device="cuda", generator=g, dtype=torch.int32)
    code = TW.FPDT_TW_SWIGLU
    Y, dX, dH = torch.empty_like(X), torch.empty_like(X), torch.empty_like(X)
    dW1, dW3, dW2 = (torch.zeros_like(w, dtype=torch.float32) for w in (W1, W3, W2))
    dWv = torch.zeros_like(Wv, dtype=torch.float32)
    loss, lse = torch.empty(rows, device="cuda"), torch.empty(rows, device="cuda")
    wb = torch.empty(TW.fpdt_tw_ffn_workspace_bytes(rows, n_model, n_ffn, code, n_chunks, True), dtype=torch.uint8, device="cuda")
    wl = torch.empty(TW.fpdt_tw_loss_workspace_bytes(rows, n_model, vocab, n_chunks), dtype=torch.uint8, device="cuda")

    def step():
        TW.fpdt_tw_ffn_fwd(X, W1, W3, W2, Y, code, n_chunks, wb)
        TW.fpdt_tw_ffn_bwd(X, W1, W3, W2, dY, dX, dW1, dW3, dW2, code, n_chunks, wb)
        TW.fpdt_tw_loss_fwd_bwd(Y, Wv, tgt, 1.0 / rows, loss, lse, dH, dWv, n_chunks, wl)

    outs = {"Y": Y, "dX": dX, "dH": dH, "dW1": dW1, "dW3": dW3, "dW2": dW2, "dWv": dWv, "loss": loss, "lse": lse}

    def reset():  # written outputs are poisoned, accumulated-into ones start from zero
        for n, t in outs.items():
            t.zero_() if n.startswith("dW") else t.fill_(float("nan"))

    step()  # first call: sizes the library's operand scratch pool and loads its kernels outside any capture
    reset()
    step()
    torch.cuda.synchronize()
    want = {n: t.clone() for n, t in outs.items()}
    gr = torch.cuda.CUDAGraph()
    with torch.cuda.graph(gr, stream=torch.cuda.Stream()):
        step()
    for rep in range(3):
        reset()
        torch.cuda.synchronize()
        gr.replay()
        torch.cuda.synchronize()
        for n, t in outs.items():
            assert torch.equal(t.view(torch.uint8), want[n].view(torch.uint8)), (n, rep)


# ------------------------------------------------------------------ edges of the dense products
@pytest.mark.gpu
@pytest.mark.parametrize("rows,n_in,n_out,n_chunks,offset", [
    (1, 8, 8, 1, 0),         # one element row, less than one k stage
    (63, 40, 72, 2, 0),      # ragged k (not a multiple of 32), less than a tile in every direction
    (257, 264, 248, 1, 0),   # one row / column past and short of the large tile
    (300, 4096, 64, 1, 0),   # long k, few tiles: the k range is split
    (129, 1000, 1001, 3, 0),  # odd widths: no row is 16-byte aligned
    (200, 96, 520, 1, 1),    # operands that start 2 bytes behind a 16-byte boundary
    (1030, 2048, 1160, 4, 0),
    (4100, 1032, 4200, 1, 0)])  # more tiles than compute units (Y), few and all divided (dX, dW)
def test_gpu_linear_tile_edges(rows, n_in, n_out, n_chunks, offset):
    """Forward, dX and dW of the projection against fp64 at the edges of the product's tiles, k stages and
    splits.  Exact bf16 products summed in fp32: rel 1e-4 of a row's rms (k <= 4096 terms, error of about
    sqrt(k) 2^-24 of the rms, under 1e-5) plus half a bf16 ulp of the stored value."""
    print("[case] linear edges", rows, n_in, n_out, n_chunks, offset, flush=True)
    g = torch.Generator(device="cuda").manual_seed(rows + n_in)

    def bf(r, c, std=1.0):
        flat = torch.empty(r * c + offset, dtype=torch.bfloat16, device="cuda")
        t = flat[offset:].view(r, c)
        t.copy_(torch.randn(r, c, device="cuda", generator=g) * std)
        return t

    X, W, dY = bf(rows, n_in), bf(n_out, n_in, n_in ** -0.5), bf(rows, n_out)
    Y, dX = torch.full_like(dY, float("nan")), torch.full_like(X, float("nan"))
    dW = torch.ones(n_out, n_in, device="cuda")
    TW.fpdt_tw_linear_fwd(X, W, Y, n_chunks)
    TW.fpdt_tw_linear_bwd(X, W, dY, dX, dW, n_chunks)
    torch.cuda.synchronize()
    f64 = lambda t: t.double().cpu().numpy()
    ref = otw.linear(f64(X), f64(W), f64(dY))
    _rowwise_ok("Y", f64(Y), ref["Y"], rel=1e-4)
    _rowwise_ok("dX", f64(dX), ref["dX"], rel=1e-4)
    np.testing.assert_allclose(f64(dW), 1 + ref["dW"], atol=1e-4 * max(1.0, float(np.abs(ref["dW"]).max())))


@pytest.mark.gpu
def test_gpu_linear_rows_of_eight_million():
    """Rows longer than the product kernel's 32-bit offsets: the contraction runs in segments.  2^23 + 40 terms
    of exact products, summed in fp32 over segments of 2^22: about sqrt(2^22 / 32) 2^-24 = 2e-5 of the rms."""
    n_in, n_out, rows = (1 << 23) + 40, 8, 9
    print("[case] linear long rows", rows, n_in, n_out, flush=True)
    g = torch.Generator(device="cuda").manual_seed(3)
    X = torch.randn(rows, n_in, device="cuda", generator=g).to(torch.bfloat16)
    W = (torch.randn(n_out, n_in, device="cuda", generator=g) * n_in ** -0.5).to(torch.bfloat16)
    Y = torch.empty(rows, n_out, dtype=torch.bfloat16, device="cuda")
    TW.fpdt_tw_linear_fwd(X, W, Y, 1)
    torch.cuda.synchronize()
    ref = (X.double() @ W.double().t()).cpu().numpy()
    _rowwise_ok("Y", Y.double().cpu().numpy(), ref, rel=4e-4)


@pytest.mark.gpu
@pytest.mark.parametrize("rows,n,n_chunks", [(4100, 1024, 1), (700, 264, 3), (33, 40, 1), (300, 8192, 2)])
def test_gpu_linear_in_place(rows, n, n_chunks):
    """Y in the place of X and dX in that of dY: against the same calls on tensors of their own (another
    chunking of the same sums at most: half a bf16 ulp of the stored value plus fp32 rounding)."""
    print("[case] linear in place", rows, n, n_chunks, flush=True)
    g = torch.Generator(device="cuda").manual_seed(rows)
    X = torch.randn(rows, n, device="cuda", generator=g).to(torch.bfloat16)
    W = (torch.randn(n, n, device="cuda", generator=g) * n ** -0.5).to(torch.bfloat16)
    f64 = lambda t: t.double().cpu().numpy()
    ref = otw.linear(f64(X), f64(W), f64(X))
    Y, dX = X.clone(), X.clone()
    TW.fpdt_tw_linear_fwd(Y, W, Y, n_chunks)
    TW.fpdt_tw_linear_bwd(X, W, dX, dX, None, n_chunks)
    torch.cuda.synchronize()
    _rowwise_ok("Y", f64(Y), ref["Y"], rel=1e-4)
    _rowwise_ok("dX", f64(dX), ref["dX"], rel=1e-4)


@pytest.mark.gpu
@pytest.mark.parametrize("n_in,in_place", [(2049, False), (264, True)])
def test_gpu_linear_copies_one_chunk_at_a_time(n_in, in_place):
    """A projection whose X cannot be read where it is copies a chunk, not all of X, to scratch: with X of
    4.3 GB (2.2 GB in place) in 64 chunks the pool, which is kept, takes under 512 MiB."""
    n_out, n_chunks = (n_in if in_place else 8), 64
    rows = (1 << 20) if not in_place else (1 << 22)
    print("[case] linear chunk copies", rows, n_in, in_place, flush=True)
    X = torch.zeros(rows, n_in, dtype=torch.bfloat16, device="cuda")
    W = torch.zeros(n_out, n_in, dtype=torch.bfloat16, device="cuda")
    Y = X if in_place else torch.empty(rows, n_out, dtype=torch.bfloat16, device="cuda")
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    TW.fpdt_tw_linear_fwd(X, W, Y, n_chunks)
    torch.cuda.synchronize()
    assert before - torch.cuda.mem_get_info()[0] <= 512 << 20
    assert not bool(Y.any())


@pytest.mark.gpu
@pytest.mark.parametrize("rows,n_in,n_out", [(2, (1 << 28) + 8, 3), (3, 8, (1 << 28) + 24), (33, (1 << 28) + 1, 1), (2, (1 << 28) - 3, 2)])
def test_gpu_linear_rows_of_two_hundred_million(rows, n_in, n_out):
    """Gradients where consecutive rows of k lie further apart than the product kernel's 32-bit offsets reach:
    the columns run in segments.  Every element against sums of exact products in fp32 (up to 33 terms; where
    the long width is contracted, against sums in fp64 with the bound of long rows above)."""
    print("[case] linear very long rows", rows, n_in, n_out, flush=True)
    g = torch.Generator(device="cuda").manual_seed(4)

    def bf(r, c):  # (randn takes its time at this size)
        return torch.randint(-127, 128, (r, c), device="cuda", generator=g, dtype=torch.int8).to(torch.bfloat16) / 64

    X, W, dY = bf(rows, n_in), bf(n_out, n_in), bf(rows, n_out)
    dX, dW = torch.full_like(X, float("nan")), torch.ones(n_out, n_in, device="cuda")
    TW.fpdt_tw_linear_bwd(X, W, dY, dX, dW, 1)
    torch.cuda.synchronize()
    if n_out < 1000:
        for r in range(rows):
            want = sum(dY[r, k].float() * W[k].float() for k in range(n_out))
            assert bool(((dX[r].float() - want).abs() <= 2.0 ** -8 * want.abs() + 1e-5).all()), r
    else:
        _rowwise_ok("dX", dX.double().cpu().numpy(), (dY.double() @ W.double()).cpu().numpy(), rel=4e-4)
    for o in range(0, n_out, max(1, n_out // 3)):
        want = 1 + sum(dY[r, o:o + max(1, n_out // 3), None].float() * X[r].float() for r in range(rows))
        assert bool(((dW[o:o + max(1, n_out // 3)] - want).abs() <= 1e-5 * want.abs() + 1e-5).all()), o


@pytest.mark.gpu
def test_gpu_second_call_of_a_size_finds_its_scratch():
    """The first call of a size grows the scratch pool, twice here (200 MB of logit gradients, then a 400 MB copy
    of a weight whose rows are not 16-byte aligned); the second one must not, as it may be captured.  In a
    process of its own, whose pool is empty."""
    code = """
import torch
from paper_2408_16978_amd import tokenwise as TW
rows, hidden, vocab = 500, 1001, 200000
bf = lambda *s: (torch.randn(*s, device="cuda") * hidden ** -0.25).to(torch.bfloat16)
H, W = bf(rows, hidden), bf(vocab, hidden)
target = torch.randint(0, vocab, (rows,), device="cuda", dtype=torch.int32)
loss, lse, dH = torch.empty(rows, device="cuda"), torch.empty(rows, device="cuda"), torch.empty_like(H)
ws = torch.empty(TW.fpdt_tw_loss_workspace_bytes(rows, hidden, vocab, 2), dtype=torch.uint8, device="cuda")
call = lambda: TW.fpdt_tw_loss_fwd_bwd(H, W, target, 1.0 / rows, loss, lse, dH, None, 2, ws)
call()
torch.cuda.synchronize()
want = dH.clone()
graph = torch.cuda.CUDAGraph()
with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
    call()
for rep in range(3):
    dH.fill_(float("nan"))
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(dH, want), rep
print("replayed")
"""
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "replayed" in r.stdout, r.stderr[-2000:]


# ------------------------------------------------------------------ every layout of a product
# (M, N, K) and what is launched for them: the output tile in units of 64, and whether its tiles run whole,
# divided along k, or some each.  Ragged in all three; widths that are read in place, but for the last three.
# (1 x 4 tiles of both kinds are not chosen for more than 64 rows.)
PRODUCTS = [((72, 72, 72), (1, 4, "whole")), ((72, 72, 648), (1, 4, "divided")), ((40, 67248, 792), (1, 4, "mixed")),
            ((4304, 72, 1288), (2, 2, "divided")), ((67872, 72, 752), (2, 2, "mixed")),
            ((17104, 72, 72), (2, 4, "whole")), ((1488, 72, 5496), (2, 4, "divided")), ((5448, 1384, 4632), (2, 4, "mixed")),
            ((33368, 72, 72), (3, 4, "whole")), ((136, 7392, 1304), (3, 4, "divided")), ((3544, 6824, 2328), (3, 4, "mixed")),
            ((49552, 72, 72), (4, 4, "whole")), ((6248, 264, 2448), (4, 4, "divided")), ((6536, 2312, 712), (4, 4, "mixed")),
            ((6541, 2317, 711), (4, 4, "mixed")), ((1501, 251, 5003), (1, 4, "divided")), ((1630, 2695, 33), (2, 2, "whole"))]


def test_products_cover_the_rule():
    assert all(launch_rules.product(*size) == plan for size, plan in PRODUCTS)
    seen = {plan for _, plan in PRODUCTS}
    r = np.random.default_rng(6)
    for _ in range(20000):
        M, N, K = (int(np.exp(r.uniform(np.log(8), np.log(140000)))) for _ in range(3))
        assert launch_rules.product(M, N, K) in seen, (M, N, K)


@pytest.mark.gpu
@pytest.mark.parametrize("size,plan", PRODUCTS)
def test_gpu_every_layout_of_a_product(size, plan):
    """The five forms that the operations multiply in, each at the (M, N, K) of the case: X W^T as bf16 (Y) and
    fp32 (logits), dY W (dX), dY^T X += (dW) and the bf16 product that adds to another (dX of SwiGLU).
    Against fp64: exact bf16 products summed in fp32, sqrt(k) 2^-24 of the rms at most (under 3e-5 at k =
    67248) and half an ulp of a bf16 output.  SwiGLU's reference has the operation's bf16 intermediates; where
    fp32 and fp64 sums round one of them differently, the result moves by an ulp of it: of the summand that
    is added to, 2^-8 of at most five times the rms, 2e-2 of it (of one of k terms, far less).  The logits through their log-sum-exp, in which every one of them counts, and the targets'."""
    M, N, K = size
    print("[case] product", size, plan, flush=True)
    assert launch_rules.product(M, N, K) == plan
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    bf = lambda *s, std=1.0: (torch.randn(*s, device="cuda", generator=g) * std).to(torch.bfloat16)

    def rowwise(name, got, ref, rel):
        budget = rel * ref.pow(2).mean(1, keepdim=True).sqrt() + 2.0 ** -8 * ref.abs() + 1e-9
        assert bool(((got.double() - ref).abs() <= budget).all()), name

    A, Bn, Bt = bf(M, K), bf(N, K, std=K ** -0.5), bf(K, N, std=K ** -0.5)
    Y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    TW.fpdt_tw_linear_fwd(A, Bn, Y, 1)
    logits = A.double() @ Bn.double().t()
    rowwise("Y", Y, logits, 1e-4)
    target = torch.randint(0, N, (M,), device="cuda", generator=g, dtype=torch.int32)
    loss, lse = torch.empty(M, device="cuda"), torch.empty(M, device="cuda")
    ws = torch.empty(TW.fpdt_tw_loss_workspace_bytes(M, K, N, 1), dtype=torch.uint8, device="cuda")
    TW.fpdt_tw_loss_fwd_bwd(A, Bn, target, 1.0, loss, lse, None, None, 1, ws)
    want = torch.logsumexp(logits, 1)
    assert float((lse.double() - want).abs().max()) <= 2e-5
    assert float((loss.double() - (want - logits.gather(1, target.long()[:, None])[:, 0])).abs().max()) <= 1e-4
    dX = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    TW.fpdt_tw_linear_bwd(dX, Bt, A, dX, None, 1)
    rowwise("dX", dX, A.double() @ Bt.double(), 1e-4)
    At, dW = bf(K, M), torch.ones(M, N, device="cuda")
    TW.fpdt_tw_linear_bwd(Bt, torch.empty(M, N, dtype=torch.bfloat16, device="cuda"), At, None, dW, 1)
    ref = At.double().t() @ Bt.double()
    assert float((dW.double() - 1 - ref).abs().max()) <= 1e-4 * max(1.0, float(ref.abs().max()))
    # rows M, model width N, hidden width K
    X, dY = bf(M, N), bf(M, N)
    W1, W3, W2 = bf(K, N, std=N ** -0.5), bf(K, N, std=N ** -0.5), bf(N, K, std=K ** -0.5)
    ws = torch.empty(TW.fpdt_tw_ffn_workspace_bytes(M, N, K, TW.FPDT_TW_SWIGLU, 1, True), dtype=torch.uint8, device="cuda")
    TW.fpdt_tw_ffn_bwd(X, W1, W3, W2, dY, dX, None, None, None, TW.FPDT_TW_SWIGLU, 1, ws)
    bf64 = lambda t: t.to(torch.bfloat16).double()  # the roundings between the products, which are part of the operation
    a, b, dh = bf64(X.double() @ W1.double().t()), bf64(X.double() @ W3.double().t()), bf64(dY.double() @ W2.double())
    sg = torch.sigmoid(a)
    first = bf64(bf64(dh * b * sg * (1 + a * (1 - sg))) @ W1.double())
    rowwise("SwiGLU dX", dX, first + bf64(dh * a * sg) @ W3.double(), 2e-2)


@pytest.mark.gpu
@pytest.mark.parametrize("n_in", [(1 << 23) - 3, (1 << 23) - 63, (1 << 23) - 64])
def test_gpu_linear_rows_just_short_of_eight_million(n_in):
    """Widths that are within the product kernel's offsets, but whose copies' rounded rows would not be."""
    n_out, rows = 8, 9
    print("[case] linear rows just short of the limit", n_in, flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    X = torch.randn(rows, n_in, device="cuda", generator=g).to(torch.bfloat16)
    W = (torch.randn(n_out, n_in, device="cuda", generator=g) * n_in ** -0.5).to(torch.bfloat16)
    Y = torch.empty(rows, n_out, dtype=torch.bfloat16, device="cuda")
    TW.fpdt_tw_linear_fwd(X, W, Y, 1)
    torch.cuda.synchronize()
    _rowwise_ok("Y", Y.double().cpu().numpy(), (X.double() @ W.double().t()).cpu().numpy(), rel=4e-4)


@pytest.mark.gpu
def test_gpu_linear_two_billion_columns():
    """n_out = 2^31 - 1, the largest that the argument holds: the last tile of C would reach behind 2^31.  Rows of
    W are zero but for some at its ends and around 2^30, where the segments meet."""
    n_in, n_out = 32, (1 << 31) - 1
    print("[case] linear two billion columns", flush=True)
    if torch.cuda.mem_get_info()[0] < 160 << 30:
        torch.cuda.empty_cache()
    X = torch.randn(1, n_in, device="cuda").to(torch.bfloat16)
    W = torch.zeros(n_out, n_in, dtype=torch.bfloat16, device="cuda")
    parts = [slice(0, 300), slice((1 << 30) - 300, (1 << 30) + 300), slice(n_out - 300, n_out)]
    for p in parts:
        W[p] = torch.randn(W[p].shape, device="cuda").to(torch.bfloat16)
    Y = torch.ones(1, n_out, dtype=torch.bfloat16, device="cuda")
    TW.fpdt_tw_linear_fwd(X, W, Y, 1)
    torch.cuda.synchronize()
    for p in parts:
        _rowwise_ok("Y", Y[:, p].double().cpu().numpy(), (X.double() @ W[p].double().t()).cpu().numpy(), rel=1e-4)
        Y[:, p] = 0
    assert int(torch.count_nonzero(Y)) == 0
    del W, Y
    torch.cuda.empty_cache()
