"""Which short forwards read K and V from their tensors (launch_rules.h, sweep_reads_tensors), and the lines that their first
workgroups read ahead: head counts that do not divide 256, more readers than rows of a tile, lengths around the 768 keys from
which they do."""
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
def reads():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "r.cpp"), os.path.join(d, "r.so")
        with open(src, "w") as f:
            f.write('#include "launch_rules.h"\nextern "C" int reads(int64_t S, int Hq, int Hkv, int D, int kg) { return fpdt::sweep_reads_tensors(S, Hq, Hkv, D, kg); }\n')
        subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", launch_rules.CSRC, src, "-o", so], check=True)
        L = ctypes.CDLL(so)
    L.reads.argtypes = [ctypes.c_int64] + [ctypes.c_int] * 4
    return lambda S, Hq, Hkv, D: bool(L.reads(S, Hq, Hkv, D, launch_rules.forward_key_groups(S, Hq)))


# packed: measured 2% to 8% slower otherwise (behind 16K tokens, D = 64 and 128, the same), with the inputs in the caches and without
@pytest.mark.parametrize("S,Hq,Hkv,D", [(6144, 8, 2, 80), (12288, 8, 2, 80), (12288, 4, 1, 80), (9216, 8, 8, 80), (5120, 16, 4, 80), (24576, 2, 1, 80), (49152, 1, 1, 80),
                                        (18432, 2, 1, 64), (40960, 2, 1, 64), (32768, 2, 1, 128)])
def test_packed_where_that_is_faster(reads, S, Hq, Hkv, D):
    assert launch_rules.forward_key_groups(S, Hq) > 1 and not reads(S, Hq, Hkv, D)


# read from the tensors: measured 1% to 22% slower otherwise
@pytest.mark.parametrize("S,Hq,Hkv,D", [(256, 1, 1, 64), (8192, 8, 8, 64), (8192, 4, 1, 64), (2048, 16, 16, 64), (3072, 8, 1, 80), (4096, 4, 1, 80), (1024, 32, 8, 80),
                                        (2048, 8, 2, 128), (4096, 8, 8, 128), (1536, 32, 8, 128), (512, 64, 8, 128), (5120, 8, 8, 64), (5120, 8, 1, 64), (2304, 16, 4, 64),
                                        (2560, 32, 8, 64), (5632, 16, 4, 64), (512, 64, 8, 64), (1536, 32, 8, 64), (10240, 4, 1, 64), (3072, 16, 4, 80), (4096, 8, 2, 80),
                                        (2304, 32, 8, 80), (8192, 4, 4, 80), (16384, 1, 1, 80), (4096, 8, 2, 128), (5120, 4, 4, 128), (6144, 8, 2, 128), (4096, 16, 4, 128),
                                        (8192, 8, 2, 128), (16384, 2, 1, 128)])
def test_read_from_the_tensors_where_that_is_faster(reads, S, Hq, Hkv, D):
    assert launch_rules.forward_key_groups(S, Hq) > 1 and reads(S, Hq, Hkv, D)


def test_one_key_group_is_packed(reads):
    assert not any(reads(S, Hq, Hq, D) for S in range(256, 8449, 256) for Hq in (1, 8, 64) for D in (64, 80, 128)
                   if launch_rules.forward_key_groups(S, Hq) == 1)


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 80, 128])
@pytest.mark.parametrize("S,Hq,Hkv", [(768, 6, 2), (1024, 1, 1), (1024, 7, 7), (1280, 24, 3), (2816, 3, 1), (2048, 12, 4)])
def test_gpu_bits_of_the_packed_forward(reads, S, Hq, Hkv, D):
    print("[case] lines read ahead", S, Hq, Hkv, D, flush=True)
    assert launch_rules.forward_key_groups(S, Hq) == 4 and reads(S, Hq, Hkv, D)
    Q, K, V, dO = inputs.make_qkvdo(S, Hq, Hkv, D, "bf16", 23, device="cuda")
    one = runner.make_buffers(Q, K, V, dO, S, D ** -0.5, 0, bwd=False)
    pairs = runner.make_buffers(Q, K, V, dO, 256, D ** -0.5, B.FPDT_PAIRWISE, bwd=False)
    runner.forward(one)
    runner.forward(pairs)
    torch.cuda.synchronize()
    assert torch.equal(one.O, pairs.O) and torch.equal(one.LSE, pairs.LSE)


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 80, 128])
@pytest.mark.parametrize("S,Hq,Hkv,groups", [(4608, 8, 2, 4), (5120, 8, 8, 2), (10240, 4, 1, 4), (8192, 8, 8, 2), (1536, 32, 8, 2), (16384, 1, 1, 4)])
def test_gpu_bits_of_longer_packed_forwards(reads, S, Hq, Hkv, groups, D):
    """More workgroups than compute units, and tens of tiles, with two and with four key groups."""
    print("[case] longer forwards from tensors", S, Hq, Hkv, D, flush=True)
    assert launch_rules.forward_key_groups(S, Hq) == groups and reads(S, Hq, Hkv, D)
    Q, K, V, dO = inputs.make_qkvdo(S, Hq, Hkv, D, "bf16", 24, device="cuda")
    one = runner.make_buffers(Q, K, V, dO, S, D ** -0.5, 0, bwd=False)
    pairs = runner.make_buffers(Q, K, V, dO, S // 2, D ** -0.5, B.FPDT_PAIRWISE, bwd=False)
    runner.forward(one)
    runner.forward(pairs)
    torch.cuda.synchronize()
    assert torch.equal(one.O, pairs.O) and torch.equal(one.LSE, pairs.LSE)
