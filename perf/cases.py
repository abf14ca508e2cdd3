"""The work that users of this library have it do, as timed cases.

A case is a dict of plain values.  `listed()` names the representative ones, `draw(rng)` gives
further cases of the same kinds over the ranges they stand for, `prepare(case, seed)` makes what a
program holds before the call (tensors, workspaces), `run(state)` is one pass through the public
entry points, `work(case)` the bytes and operations the pass cannot do without, `tolerance(case)`
how far another correct implementation of the same precision may be off.

Kinds:
  attn      forward and backward of the chunked causal attention (resident, offloaded, block-sparse)
  fwd       the forward that needs no workspace, as inference code calls it
  linear    the QKV projection in front of the attention, forward and backward
  ffn       the feed-forward block, forward and backward
  loss      the cross-entropy with its vocabulary projection, forward and backward in one call
"""
import random

import torch

from paper_2408_16978_amd import binding as B
from paper_2408_16978_amd import inputs, runner
from paper_2408_16978_amd import tokenwise as TW


def _attn(dtype, S, chunk, Hq, Hkv, D, kv_host=False, act_host=False, store_ds=False, keep=1.0, mask_seed=0):
    return {"kind": "attn", "dtype": dtype, "S": S, "chunk": chunk, "Hq": Hq, "Hkv": Hkv, "D": D,
            "kv_host": kv_host, "act_host": act_host, "store_ds": store_ds, "keep": keep, "mask_seed": mask_seed}


def listed():
    cases = {
        # the fp32 accuracy configuration: four chunks of 256 tokens, latency and launches count
        "f32_1k": _attn("f32", 1024, 256, 2, 2, 64),
        # the shortest bf16 call: a prompt of 2K tokens through the forward that allocates nothing
        "fwd_2k": {"kind": "fwd", "S": 2048, "Hq": 8, "Hkv": 2, "D": 128},
        # one training step of a Llama-8B head share at an ordinary context length, everything in HBM
        "llama_8k": _attn("bf16", 8192, 8192, 8, 2, 128),
        # GPT-2.7B head share, 64K tokens in chunks of 8K, head dimension 80
        "gpt_64k": _attn("bf16", 65536, 8192, 4, 4, 80),
        # Llama-8B head share, 256K tokens in chunks of 64K, backward from stored dS: the largest pass
        "llama_256k": _attn("bf16", 262144, 65536, 8, 2, 128, store_ds=True),
        # the same share with key/value chunks in pinned host memory
        "llama_128k_kv_host": _attn("bf16", 131072, 32768, 8, 2, 128, kv_host=True, store_ds=True),
        # Llama-70B head share (one KV head), key/value chunks and saved activations in pinned host memory
        "llama70b_128k_all_host": _attn("bf16", 131072, 32768, 8, 1, 128, kv_host=True, act_host=True, store_ds=True),
        # block-sparse attention: half of the chunk pairs below the diagonal are kept, K/V fetched from the host
        "sparse_128k_kv_host": _attn("bf16", 131072, 16384, 8, 2, 128, kv_host=True, keep=0.5, mask_seed=7),
        # QKV projection at Llama-8B widths, one GPU's 16K tokens in four chunks
        "qkv_16k": {"kind": "linear", "rows": 16384, "n_in": 4096, "n_out": 6144, "n_chunks": 4},
        # feed-forward block at Llama-8B widths
        "ffn_swiglu_16k": {"kind": "ffn", "act": "swiglu", "rows": 16384, "n_model": 4096, "n_ffn": 14336, "n_chunks": 4},
        # feed-forward block at GPT-2.7B widths on a ragged number of tokens
        "ffn_gelu_ragged": {"kind": "ffn", "act": "gelu", "rows": 3001, "n_model": 2560, "n_ffn": 10240, "n_chunks": 2},
        # the loss over Llama-3's vocabulary in the 2 * vocab / hidden chunks that bound its memory
        "loss_64k": {"kind": "loss", "rows": 65536, "hidden": 4096, "vocab": 128256, "n_chunks": 62},
    }
    return [dict(c, name=n) for n, c in cases.items()]


def _log(rng, lo, hi):
    return lo * (hi / lo) ** rng.random()


def _heads(rng, max_hq=8):
    return rng.choice([h for h in ((2, 2), (4, 4), (8, 8), (8, 2), (8, 1), (4, 2), (2, 1)) if h[0] <= max_hq])


def draw(rng):
    kind = rng.choice(["f32", "fwd", "resident", "resident", "pairs", "sparse", "linear", "ffn", "ffn", "loss"])
    if kind == "f32":
        hq, hkv = _heads(rng, 4)
        chunk = int(_log(rng, 64, 1024))
        return _attn("f32", chunk * rng.randint(1, max(1, min(6, 3072 // chunk))), chunk, hq, hkv, rng.choice([64, 80, 128]))
    if kind == "fwd":
        hq, hkv = _heads(rng)
        top = 65536 // hkv if hkv > 2 else 32768  # what the built-in scratch array holds
        return {"kind": "fwd", "S": 256 * round(_log(rng, 2, top // 256 - 1)), "Hq": hq, "Hkv": hkv, "D": rng.choice([64, 80, 128])}
    if kind == "resident":
        hq, hkv = _heads(rng)
        S = 256 * round(_log(rng, 3, 65536 / 256))
        return _attn("bf16", S, S, hq, hkv, rng.choice([64, 80, 128, 128]))
    if kind in ("pairs", "sparse"):
        hq, hkv = _heads(rng)
        u = rng.randint(2, 8)
        chunk = 256 * round(_log(rng, 8, min(256.0, 196608 / u / 256)))
        act = kind == "pairs" and rng.random() < 0.3
        return _attn("bf16", u * chunk, chunk, hq, hkv, rng.choice([64, 80, 128, 128]), kv_host=act or rng.random() < 0.7,
                     act_host=act, store_ds=rng.random() < 0.6, keep=rng.choice([0.25, 0.5, 0.75]) if kind == "sparse" else 1.0,
                     mask_seed=rng.randint(1, 99) if kind == "sparse" else 0)
    rows = int(_log(rng, 300, 32768))
    if kind == "linear":
        return {"kind": "linear", "rows": rows, "n_in": 8 * round(_log(rng, 64, 640)), "n_out": 8 * round(_log(rng, 64, 1024)),
                "n_chunks": rng.choice([1, 2, 3, 4, 8])}
    if kind == "ffn":
        n_model = 8 * round(_log(rng, 64, 512))
        act = rng.choice(["gelu", "swiglu"])
        n_ffn = 4 * n_model if act == "gelu" else 8 * round(n_model * 3.5 / 8) + rng.choice([0, 0, 8, 1])
        return {"kind": "ffn", "act": act, "rows": min(rows, 16384), "n_model": n_model, "n_ffn": n_ffn, "n_chunks": rng.choice([1, 2, 4, 5, 8])}
    vocab = rng.choice([32000, 50257, 50304, 128256])
    hidden = 128 * rng.randint(8, 32)
    return {"kind": "loss", "rows": rows, "hidden": hidden, "vocab": vocab,
            "n_chunks": max(1, min(rng.choice([4, 16, 2 * vocab // hidden]), rows // 128))}


def _mask(case):
    """Chunk mask of a block-sparse case: every pair below the diagonal with probability `keep`."""
    u, rng = case["S"] // case["chunk"], random.Random(case["mask_seed"])
    return [[1 if i == m or (i < m and rng.random() < case["keep"]) else 0 for i in range(u)] for m in range(u)]


def _bf16(gen, *shape, std=1.0):
    return (torch.randn(*shape, device="cuda", generator=gen) * std).to(torch.bfloat16)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "attn":
        Q, K, V, dO = inputs.make_qkvdo(case["S"], case["Hq"], case["Hkv"], case["D"], case["dtype"], seed, device="cuda")
        flags = (B.FPDT_KV_ON_HOST if case["kv_host"] else 0) | (B.FPDT_ACT_ON_HOST if case["act_host"] else 0)
        flags |= B.FPDT_BWD_STORE_DS if case["store_ds"] else 0
        mask = torch.tensor(_mask(case), dtype=torch.uint8) if case["mask_seed"] else None
        return case, runner.make_buffers(Q, K, V, dO, case["chunk"], case["D"] ** -0.5, flags, chunk_mask=mask)
    if kind == "fwd":
        Q, K, V, _ = inputs.make_qkvdo(case["S"], case["Hq"], case["Hkv"], case["D"], "bf16", seed, device="cuda")
        return case, (Q, K, V, torch.empty_like(Q), torch.empty((case["Hq"], case["S"]), device="cuda"))
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rows, n = case["rows"], case["n_chunks"]
    grad = lambda w: torch.zeros(w.shape, dtype=torch.float32, device="cuda")  # noqa: E731
    if kind == "linear":
        X, W = _bf16(gen, rows, case["n_in"]), _bf16(gen, case["n_out"], case["n_in"], std=case["n_in"] ** -0.5)
        dY = _bf16(gen, rows, case["n_out"])
        return case, (X, W, dY, torch.empty_like(dY), torch.empty_like(X), grad(W))
    if kind == "ffn":
        nm, nf, sw = case["n_model"], case["n_ffn"], case["act"] == "swiglu"
        X, dY = _bf16(gen, rows, nm), _bf16(gen, rows, nm)
        W1, W2 = _bf16(gen, nf, nm, std=nm ** -0.5), _bf16(gen, nm, nf, std=nf ** -0.5)
        W3 = _bf16(gen, nf, nm, std=nm ** -0.5) if sw else None
        code = TW.FPDT_TW_SWIGLU if sw else TW.FPDT_TW_GELU
        ws = torch.empty(TW.fpdt_tw_ffn_workspace_bytes(rows, nm, nf, code, n, True), dtype=torch.uint8, device="cuda")
        return case, (X, W1, W3, W2, dY, torch.empty_like(X), torch.empty_like(X), grad(W1), grad(W3) if sw else None, grad(W2), code, ws)
    hidden, vocab = case["hidden"], case["vocab"]
    H, W = _bf16(gen, rows, hidden), _bf16(gen, vocab, hidden, std=hidden ** -0.5)
    target = torch.randint(0, vocab, (rows,), device="cuda", generator=gen, dtype=torch.int32)
    loss, lse = torch.empty(rows, device="cuda"), torch.empty(rows, device="cuda")
    ws = torch.empty(TW.fpdt_tw_loss_workspace_bytes(rows, hidden, vocab, n), dtype=torch.uint8, device="cuda")
    return case, (H, W, target, loss, lse, torch.empty_like(H), grad(W), ws)


def run(state):
    case, s = state
    kind = case["kind"]
    if kind == "attn":
        runner.forward(s)
        runner.backward(s)
        return s.O, s.LSE, s.dQ, s.dK, s.dV
    if kind == "fwd":
        Q, K, V, O, LSE = s
        B.fpdt_attn_fwd_noalloc(Q, K, V, O, LSE, case["S"], case["D"] ** -0.5)
        return O, LSE
    n = case["n_chunks"]
    # the weight gradients are accumulated into: a training step clears them first
    if kind == "linear":
        X, W, dY, Y, dX, dW = s
        dW.zero_()
        TW.fpdt_tw_linear_fwd(X, W, Y, n)
        TW.fpdt_tw_linear_bwd(X, W, dY, dX, dW, n)
        return Y, dX, dW
    if kind == "ffn":
        X, W1, W3, W2, dY, Y, dX, dW1, dW3, dW2, code, ws = s
        grads = [g for g in (dW1, dW3, dW2) if g is not None]
        for g in grads:
            g.zero_()
        TW.fpdt_tw_ffn_fwd(X, W1, W3, W2, Y, code, n, ws)
        TW.fpdt_tw_ffn_bwd(X, W1, W3, W2, dY, dX, dW1, dW3, dW2, code, n, ws)
        return [Y, dX] + grads
    H, W, target, loss, lse, dH, dW, ws = s
    dW.zero_()
    TW.fpdt_tw_loss_fwd_bwd(H, W, target, 1.0 / case["rows"], loss, lse, dH, dW, n, ws)
    return loss, lse, dH, dW


def work(case):
    kind = case["kind"]
    if kind in ("attn", "fwd"):
        S, Hq, Hkv, D = case["S"], case["Hq"], case["Hkv"], case["D"]
        q, kv, lse = S * Hq * D, S * Hkv * D, 4 * S * Hq
        if kind == "fwd":  # Q, K, V in; O, LSE out
            return {"bytes": 2 * (2 * q + 2 * kv) + lse, "flops": 4.0 * D * Hq * S * (S + 1) / 2}
        C, u = case["chunk"], S // case["chunk"]
        off = sum(map(sum, _mask(case))) - u if case["mask_seed"] else u * (u - 1) // 2
        pairs = off * C * C + u * C * (C + 1) / 2
        # Q, K, V, dO in; O, LSE, dQ, dK, dV out; two products forward, five backward
        return {"bytes": (4 if case["dtype"] == "f32" else 2) * (4 * q + 4 * kv) + lse, "flops": 14.0 * D * Hq * pairs}
    rows = case["rows"]
    if kind == "linear":
        a, b = case["n_in"], case["n_out"]
        return {"bytes": 2 * (2 * rows * a + 2 * rows * b + a * b) + 4 * a * b, "flops": 6.0 * rows * a * b}
    if kind == "ffn":
        a, b, w = case["n_model"], case["n_ffn"], 3 if case["act"] == "swiglu" else 2
        # forward w products; backward 2 w, and those into the hidden layer recomputed (nothing is saved)
        return {"bytes": 2 * (4 * rows * a) + 6 * w * a * b, "flops": 2.0 * rows * a * b * (3 * w + w - 1)}
    a, b = case["hidden"], case["vocab"]
    return {"bytes": 2 * (2 * rows * a + a * b) + 4 * a * b + 12 * rows, "flops": 6.0 * rows * a * b}


def tolerance(case):
    """Four times what the outputs were measured to be off from the same computation in 64 bits (largest over
    the outputs and a few sizes).  bf16 attention: P and dS are rounded to bf16 between the products, so single
    elements of the short rows move by a tenth of the rms."""
    if case["kind"] in ("attn", "fwd"):
        if case.get("dtype") == "f32":
            return {"rel": 4e-6, "max": 1.2e-4}  # measured 8.5e-7, 2.9e-5
        return {"rel": 1e-2, "max": 0.4}  # measured 2.4e-3, 0.1
    return {"linear": {"rel": 7e-3, "max": 1.6e-2},  # measured 1.7e-3, 3.9e-3: the rounding of bf16 outputs
            "ffn": {"rel": 1.4e-2, "max": 8e-2},  # measured 3.6e-3, 2.0e-2: bf16 intermediates
            "loss": {"rel": 9e-3, "max": 2.3e-2}}[case["kind"]]  # measured 2.2e-3, 5.6e-3: bf16 logit gradient
