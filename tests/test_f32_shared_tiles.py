"""The fp32 backward with two workgroups per tile (launch_rules.h, f32_bwd_split): which sizes have them, walks of fewer blocks than waves,
ragged last tiles, groups of one to eight heads, and a workspace without room for the sums."""
import ctypes
import os
import subprocess
import tempfile

import pytest
import torch

import launch_rules
from paper_2408_16978_amd import binding as B
from paper_2408_16978_amd import inputs, runner


@pytest.fixture(scope="module")
def shared():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "s.cpp"), os.path.join(d, "s.so")
        with open(src, "w") as f:
            f.write('#include "launch_rules.h"\nextern "C" int split(int64_t S, int Hq, int Hkv) { return fpdt::f32_bwd_split(S, Hq, Hkv); }\n')
        subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", launch_rules.CSRC, src, "-o", so], check=True)
        L = ctypes.CDLL(so)
    L.split.argtypes = [ctypes.c_int64, ctypes.c_int, ctypes.c_int]
    return lambda S, Hq, Hkv: bool(L.split(S, Hq, Hkv))


# (one head a group: measured slower shared up to 192 tokens; many KV heads: up to 1.5 times slower shared)
@pytest.mark.parametrize("S,Hq,Hkv,yes", [(128, 2, 2, False), (192, 2, 2, False), (193, 2, 2, True), (640, 2, 2, True), (641, 2, 2, False), (1024, 2, 2, False),
                                          (2048, 4, 2, True), (2049, 4, 2, False), (4096, 8, 1, True), (4097, 8, 1, False), (4096, 64, 1, True),
                                          (144, 64, 16, False), (256, 32, 16, False), (512, 16, 8, False), (1024, 8, 4, False), (1024, 64, 4, True)])
def test_which_sizes_share(shared, S, Hq, Hkv, yes):
    assert shared(S, Hq, Hkv) == yes
    ws = lambda flags: B.fpdt_attn_workspace_bytes(S, S, Hq, Hkv, 64, B.FPDT_DTYPE_F32, flags, True)  # noqa: E731
    assert (ws(0) > ws(B.FPDT_PAIRWISE)) == yes


def test_a_shared_launch_is_not_too_large(shared):
    """Two workgroups of 512 lanes a tile, in a launch of fewer than 2^32 lanes, with sums of at most 1 GiB (256 * 128 bytes a tile), whatever
    the heads; also where an unshared launch, of up to 2^23 tiles, is one launch."""
    sizes = [S for S in list(range(1, 300, 13)) + [512, 1000, 1024, 2048, 4095, 4096]]
    heads = [(g * h, h) for h in (1, 2, 3, 5, 16) for g in (1, 2, 8, 100, 126, 127, 128, 4096, 16383, 16384, 32766, 100000)]
    for S in sizes:
        for Hq, Hkv in heads:
            if shared(S, Hq, Hkv):
                tiles = (S + 15) // 16 * (Hq + Hkv)
                assert 2 * tiles * 512 < 2 ** 32 and tiles * 256 * 128 <= 2 ** 30, (S, Hq, Hkv)
    assert launch_rules.f32_one_launch(4096, 16384, 1) and not shared(4096, 16384, 1)


def _gradients(Q, K, V, dO, scale):
    """dQ, dK, dV in fp64, by autograd on the definition."""
    S, Hq, _ = Q.shape
    g = Hq // K.shape[1]
    q, k, v = (x.double().requires_grad_() for x in (Q, K, V))
    s = torch.einsum("ihd,jhd->hij", q, k.repeat_interleave(g, 1)) * scale
    s = s.masked_fill(torch.ones(S, S, dtype=torch.bool, device=Q.device).triu(1), float("-inf"))
    o = torch.einsum("hij,jhd->ihd", torch.softmax(s, -1), v.repeat_interleave(g, 1))
    o.backward(dO.double())
    return q.grad, k.grad, v.grad


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 80, 128])
@pytest.mark.parametrize("S,Hq,Hkv", [(129, 1, 1), (193, 1, 1), (145, 8, 1), (250, 3, 3), (512, 2, 2), (640, 2, 1), (1023, 4, 2), (1024, 4, 4)])
def test_gpu_shared_tiles(shared, S, Hq, Hkv, D):
    """Against fp64 within the fp32 tolerance, 1e-4; the same bits on every run; one workgroup per tile where the workspace has no room for
    the sums, within the same tolerance."""
    print("[case] fp32 shared tiles", S, Hq, Hkv, D, flush=True)
    assert shared(S, Hq, Hkv) == (192 < S < 1024 or Hq > Hkv)
    Q, K, V, dO = inputs.make_qkvdo(S, Hq, Hkv, D, "f32", 41, device="cuda")
    b = runner.make_buffers(Q, K, V, dO, S, D ** -0.5, 0)
    runner.forward(b)
    want = _gradients(Q, K, V, dO, D ** -0.5)
    runs = []
    small = torch.empty(B.fpdt_attn_workspace_bytes(S, S, Hq, Hkv, D, B.FPDT_DTYPE_F32, B.FPDT_PAIRWISE, True), dtype=torch.uint8, device="cuda")
    for ws in (b.ws_bwd, b.ws_bwd, small):
        ws.fill_(0xFF)
        for t in (b.dQ, b.dK, b.dV):
            t.fill_(float("nan"))
        b.ws_bwd = ws
        runner.backward(b)
        torch.cuda.synchronize()
        runs.append([t.clone() for t in (b.dQ, b.dK, b.dV)])
        for got, ref in zip(runs[-1], want):
            assert float((got.double() - ref).abs().max()) <= 1e-4
    assert all(torch.equal(x, y) for x, y in zip(runs[0], runs[1]))
