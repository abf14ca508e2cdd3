"""Products of the token-wise library (csrc/tw_gemm.hip) where their stages, tiles and plans end: every length of k around
the stages of 64, the layouts that plan_launch prefers to plan_product's, and the rows and columns that end within a tile."""
import os
import re
import subprocess
import tempfile

import numpy as np
import pytest
import torch

import launch_rules
from paper_2408_16978_amd import build as lib_build
from paper_2408_16978_amd import tokenwise as TW

# sizes that plan_launch runs otherwise than plan_product, by what it runs
OTHERWISE = [((1630, 2695, 32), (2, 2, "whole")), ((7416, 1816, 250), (2, 2, "whole")), ((591, 680, 694), (2, 2, "divided")),
             ((6234, 2681, 727), (2, 2, "mixed")), ((1428, 5604, 39), (1, 4, "whole")), ((1030, 1215, 952), (1, 4, "divided")),
             ((2434, 1630, 2206), (2, 4, "whole")), ((1501, 2560, 10240), (2, 4, "divided")), ((2544, 3327, 4940), (2, 4, "mixed")),
             ((6144, 4096, 4096), (3, 4, "whole")), ((1462, 1793, 6777), (3, 4, "divided"))]


def test_plans_cover_the_product():
    """Every plan covers all tiles and all of k, in ranges of whole stages none of which is empty, and stands with
    plan_product's where that says whole tiles beside others divided by three or more, or where a side is short."""
    r = np.random.default_rng(3)
    mixed = 0
    for i in range(20000):
        M, N, K = (int(np.exp(r.uniform(np.log(8), np.log(140000)))) for _ in range(3))
        p, q = launch_rules.launched(M, N, K), launch_rules.first_answer(M, N, K)
        assert p["tiles_n"] == -(-N // (64 * p["wnt"])) and p["tiles"] == -(-M // (64 * p["wmt"])) * p["tiles_n"], (M, N, K)
        if p["splits"] == 1:
            assert p["whole"] == p["tiles"], (M, N, K)
        else:
            assert 0 <= p["whole"] < p["tiles"] and p["whole"] % 256 == 0, (M, N, K)
            assert (p["splits"] - 1) * p["split_stages"] < max(K, 32) // 64 <= p["splits"] * p["split_stages"], (M, N, K)
        stands = q["splits"] > 2 and q["whole"] > 0
        mixed += stands
        if stands or min(M, N) < 512:
            assert p == q, (M, N, K)
    assert mixed > 1000


def test_products_that_run_otherwise():
    for size, plan in OTHERWISE:
        assert launch_rules.product(*size) == plan and launch_rules.kind(launch_rules.first_answer(*size)) != plan, size


def test_compiler_moves_no_accumulator():
    """The MFMAs are inline assembly, whose results the compiler does not wait for: between the first of them and the wait
    behind the last one no instruction of its own may touch an accumulation register."""
    with tempfile.TemporaryDirectory() as d:
        out = os.path.join(d, "tw_gemm.s")
        subprocess.run([lib_build.HIPCC] + lib_build.FLAGS + ["-S", "--cuda-device-only", os.path.join(lib_build.SRC_DIR, "tw_gemm.hip"), "-o", out],
                       check=True, capture_output=True)
        with open(out) as f:
            text = f.read()
    kernels = re.findall(r"^_ZN\S*tw_gemm_kernel\S*:.*?s_endpgm", text, re.S | re.M)
    assert len(kernels) == 25
    for k in kernels:
        body = [line.split(";")[0].strip() for line in k.splitlines()]
        first, last = next(i for i, x in enumerate(body) if "v_mfma" in x), next(i for i, x in enumerate(body) if x == "s_nop 15")
        assert not [x for x in body[first:last] if "accvgpr" in x or "scratch" in x], body[0]


def _check(M, N, K):
    """Y = A Bn^T, dX = A Bt, dW += At^T Bt, the fp32 product (the loss's logits, all M rows at once) and the bf16 product that
    adds to another (dX of SwiGLU, hidden width K, whose W1 and W3 products are one each of those).  Against fp64: exact bf16
    products summed in fp32, sqrt(k) 2^-24 of the rms at most, and half an ulp of a bf16 output.  The summand that SwiGLU's
    second product adds to is bf16 as well: where fp32 and fp64 sums round it differently it is off by an ulp, 2^-7 of it."""
    print("[case] product", M, N, K, flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    bf = lambda *s, std=1.0: (torch.randn(*s, device="cuda", generator=g) * std).to(torch.bfloat16)

    def rowwise(name, got, ref, rel=1e-4, more=0.0):
        budget = rel * ref.pow(2).mean(1, keepdim=True).sqrt() + 2.0 ** -8 * ref.abs() + 1e-9 + more
        assert bool(((got.double() - ref).abs() <= budget).all()), (name, M, N, K)

    A, Bn, Bt = bf(M, K), bf(N, K, std=K ** -0.5), bf(K, N, std=K ** -0.5)
    Y = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    TW.fpdt_tw_linear_fwd(A, Bn, Y, 1)
    rowwise("Y", Y, A.double() @ Bn.double().t())
    dX = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    TW.fpdt_tw_linear_bwd(dX, Bt, A, dX, None, 1)
    rowwise("dX", dX, A.double() @ Bt.double())
    At, dW = bf(K, M), torch.ones(M, N, device="cuda")
    TW.fpdt_tw_linear_bwd(Bt, torch.empty(M, N, dtype=torch.bfloat16, device="cuda"), At, None, dW, 1)
    ref = At.double().t() @ Bt.double()
    assert float((dW.double() - 1 - ref).abs().max()) <= 1e-4 * max(1.0, float(ref.abs().max())), ("dW", M, N, K)
    target = torch.randint(0, N, (M,), device="cuda", generator=g, dtype=torch.int32)
    loss, lse = torch.empty(M, device="cuda"), torch.empty(M, device="cuda")
    ws = torch.empty(TW.fpdt_tw_loss_workspace_bytes(M, K, N, 1), dtype=torch.uint8, device="cuda")
    TW.fpdt_tw_loss_fwd_bwd(A, Bn, target, 1.0, loss, lse, None, None, 1, ws)  # fp32 C
    assert float((lse.double() - torch.logsumexp(A.double() @ Bn.double().t(), 1)).abs().max()) <= 2e-5, ("lse", M, N, K)
    X, dY, W1, W3, W2 = bf(M, N), bf(M, N), bf(K, N, std=N ** -0.5), bf(K, N, std=N ** -0.5), bf(N, K, std=K ** -0.5)
    ws = torch.empty(TW.fpdt_tw_ffn_workspace_bytes(M, N, K, TW.FPDT_TW_SWIGLU, 1, True), dtype=torch.uint8, device="cuda")
    TW.fpdt_tw_ffn_bwd(X, W1, W3, W2, dY, dX, None, None, None, TW.FPDT_TW_SWIGLU, 1, ws)
    part = -(-M * K * 2 // 256) * 256  # what the two products read stands in the workspace: [M, K] each, 256-byte aligned
    dA, dB = (ws[i * part:i * part + M * K * 2].view(torch.bfloat16).view(M, K).double() for i in (0, 1))
    first = (dA @ W1.double()).to(torch.bfloat16).double()
    rowwise("SwiGLU dX", dX, first + dB @ W3.double(), more=2.0 ** -7 * first.abs() + 1e-4 * first.pow(2).mean(1, keepdim=True).sqrt())


# one stage or less, the first, second and third stage, each with a rest of one k-step, of more and of none
@pytest.mark.gpu
@pytest.mark.parametrize("K", [1, 7, 8, 31, 32, 33, 56, 63, 64, 65, 72, 96, 97, 127, 128, 129, 160, 191, 192, 193, 232, 256, 320, 385])
def test_gpu_every_end_of_k(K):
    for M, N in ((264, 520), (513, 777), (72, 1288)):
        _check(M, N, K)


@pytest.mark.gpu
@pytest.mark.parametrize("size,plan", OTHERWISE)
def test_gpu_products_that_run_otherwise(size, plan):
    _check(*size)


# columns in pieces of 16 bytes (8 of a bf16 C, 4 of an fp32 one) or not, rows one short of and behind a tile's
@pytest.mark.gpu
@pytest.mark.parametrize("N", [504, 508, 510, 511, 512, 516, 520])
def test_gpu_ends_of_rows(N):
    for M in (255, 256, 257, 1030):
        _check(M, N, 200)
