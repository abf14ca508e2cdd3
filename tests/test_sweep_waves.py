"""Workgroups of eight, four and two waves (csrc/launch_rules.h, sweep_waves): the forward with one key group and dQ from
stored dS, for chunk pairs with fewer row tiles than half of the compute units."""
import ctypes
import os
import subprocess
import tempfile

import pytest
import torch

import launch_rules
import parity
from paper_2408_16978_amd import binding as B
from paper_2408_16978_amd import inputs, runner


@pytest.fixture(scope="module")
def waves():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "w.cpp"), os.path.join(d, "w.so")
        with open(src, "w") as f:
            f.write('#include "launch_rules.h"\nextern "C" int waves(int64_t n, int h) { return fpdt::sweep_waves(n, h); }\n')
        subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", launch_rules.CSRC, src, "-o", so], check=True)
        L = ctypes.CDLL(so)
    L.waves.argtypes = [ctypes.c_int64, ctypes.c_int]
    return L.waves


def _run(Q, K, V, dO, chunk, scale, flags):
    b = runner.make_buffers(Q, K, V, dO, chunk, scale, flags)
    runner.forward(b)
    runner.backward(b)
    torch.cuda.synchronize()
    return b


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 80, 128])
@pytest.mark.parametrize("chunk,Hq,Hkv,count", [(256, 64, 8, 2), (512, 64, 16, 4), (1024, 64, 64, 8)])
def test_gpu_forward_bits_do_not_depend_on_the_waves(waves, chunk, Hq, Hkv, count, D):
    """2048 tokens and 64 heads run with one key group: in one launch with eight waves, pair by pair with as many as the
    chunk has row tiles for (four at least).  O and LSE have the same bits; a chunk of 256 has one tile per head."""
    S = 2048
    print("[case] waves of the forward", chunk, Hq, Hkv, D, flush=True)
    assert launch_rules.forward_key_groups(S, Hq) == 1 and waves(S, Hq) == 8 and waves(chunk, Hq) == count
    Q, K, V, dO = inputs.make_qkvdo(S, Hq, Hkv, D, "bf16", 11, device="cuda")
    one = runner.make_buffers(Q, K, V, dO, S, D ** -0.5, 0, bwd=False)
    pairs = runner.make_buffers(Q, K, V, dO, chunk, D ** -0.5, B.FPDT_PAIRWISE, bwd=False)
    runner.forward(one)
    runner.forward(pairs)
    torch.cuda.synchronize()
    assert torch.equal(one.O, pairs.O) and torch.equal(one.LSE, pairs.LSE)


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 80, 128])
@pytest.mark.parametrize("Hq,Hkv,count", [(8, 2, 2), (64, 8, 2), (96, 12, 4), (128, 16, 4), (136, 17, 8)])
def test_gpu_dq_from_stored_ds(waves, Hq, Hkv, count, D):
    S, chunk = 512, 256
    print("[case] waves of dQ from stored dS", Hq, Hkv, D, flush=True)
    assert waves(chunk, Hq) == count
    Q, K, V, dO = inputs.make_qkvdo(S, Hq, Hkv, D, "bf16", 12)
    scale = D ** -0.5
    b = _run(Q, K, V, dO, chunk, scale, B.FPDT_PAIRWISE | B.FPDT_BWD_STORE_DS)
    out = {"O": b.O, "LSE": b.LSE, "dQ": b.dQ, "dK": b.dK, "dV": b.dV}
    print(parity.check_all(out, parity.oracle_full(Q, K, V, dO, scale), True))
