"""Products of the token-wise library (csrc/tw_gemm.hip) where their stages, tiles and plans end: every length of k around
the stages of 64, the layouts that plan_launch prefers to plan_product's, and the rows and columns that end within a tile."""
import ctypes
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

SHIM = """
#include "tw_plan.h"
extern "C" void launch(int64_t M, int64_t N, int64_t K, int* out)
{
    const int steps = (int)((K < fpdt_tw::SK ? fpdt_tw::SK : K) / fpdt_tw::SK);
    const fpdt_tw::Plan p = fpdt_tw::plan_launch(M, N, steps), q = fpdt_tw::plan_product(M, N, steps);
    const int v[] = {p.wmt, p.wnt, p.u.tiles, p.u.tiles_n, p.u.whole, p.u.splits, p.u.split_stages, q.u.tiles, q.u.splits, q.wmt, q.wnt};
    for (int i = 0; i < 11; ++i) out[i] = v[i];
}
"""


@pytest.fixture(scope="module")
def launch():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "plan.cpp"), os.path.join(d, "plan.so")
        with open(src, "w") as f:
            f.write(SHIM)
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", launch_rules.CSRC, src, "-o", so], check=True)
        L = ctypes.CDLL(so)
    L.launch.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int64, ctypes.POINTER(ctypes.c_int)]

    def plan(M, N, K):
        v = (ctypes.c_int * 11)()
        L.launch(M, N, K, v)
        return list(v)
    return plan


def _kind(p):
    return p[0], p[1], "whole" if p[5] == 1 else "divided" if p[4] == 0 else "mixed"


# sizes that plan_launch runs otherwise than plan_product, by what it runs
OTHERWISE = [((1630, 2695, 32), (2, 2, "whole")), ((7416, 1816, 250), (2, 2, "whole")), ((591, 680, 694), (2, 2, "divided")),
             ((6234, 2681, 727), (2, 2, "mixed")), ((1428, 5604, 39), (1, 4, "whole")), ((1030, 1215, 952), (1, 4, "divided")),
             ((2434, 1630, 2206), (2, 4, "whole")), ((1501, 2560, 10240), (2, 4, "divided")), ((2544, 3327, 4940), (2, 4, "mixed")),
             ((6144, 4096, 4096), (3, 4, "whole")), ((1462, 1793, 6777), (3, 4, "divided"))]


def test_plans_cover_the_product(launch):
    """Every plan covers all tiles and all of k, in ranges of whole stages none of which is empty, and stands with
    plan_product's where that says whole tiles beside others divided by three or more, or where a side is short."""
    r = np.random.default_rng(3)
    for i in range(20000):
        M, N, K = (int(np.exp(r.uniform(np.log(8), np.log(140000)))) for _ in range(3))
        wm, wn, tiles, tiles_n, whole, splits, per, q_tiles, q_splits, q_wm, q_wn = launch(M, N, K)
        assert tiles_n == -(-N // (64 * wn)) and tiles == -(-M // (64 * wm)) * tiles_n, (M, N, K)
        if splits == 1:
            assert whole == tiles, (M, N, K)
        else:
            assert 0 <= whole < tiles and whole % 256 == 0 and (splits - 1) * per < max(K, 32) // 64 <= splits * per, (M, N, K)
        if min(M, N) < 512:
            assert (wm, wn, splits) == (q_wm, q_wn, q_splits), (M, N, K)


def test_products_that_run_otherwise(launch):
    for size, plan in OTHERWISE:
        assert _kind(launch(*size)) == plan and launch_rules.product(*size) != plan, size


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
    """Y = A Bn^T, dX = A Bt, dW += At^T Bt, and the bf16 product that adds to another (dX of SwiGLU, hidden width K, whose
    W1 and W3 products are one each of those).  Against fp64: exact bf16 products summed in fp32, sqrt(k) 2^-24 of the rms at
    most, and half an ulp of a bf16 output."""
    print("[case] product", M, N, K, flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    bf = lambda *s, std=1.0: (torch.randn(*s, device="cuda", generator=g) * std).to(torch.bfloat16)

    def rowwise(name, got, ref, rel=1e-4):
        budget = rel * ref.pow(2).mean(1, keepdim=True).sqrt() + 2.0 ** -8 * ref.abs() + 1e-9
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
