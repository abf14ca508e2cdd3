"""How the loss cuts its rows (csrc/tw_plan.h): into groups whose logit gradients are gathered, which the scratch's documented bound
of max(chunk, 2 hidden) rows covers, and those into the rows whose logits are computed at a time."""
import ctypes
import os
import random
import subprocess
import sys
import tempfile

import pytest

import launch_rules

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = """
#include "tw_plan.h"
extern "C" int64_t group(int64_t rows, int64_t c, int64_t hidden) { return fpdt_tw::loss_group(rows, c, hidden); }
extern "C" int64_t step(int64_t n, int64_t full, int64_t vocab, int64_t hidden) { return fpdt_tw::loss_step(n, full, vocab, hidden); }
extern "C" double cost(int64_t n, int64_t step, int64_t vocab, int64_t hidden) { return fpdt_tw::loss_cost(n, step, vocab, hidden); }
"""


@pytest.fixture(scope="module")
def plan():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "loss.cpp"), os.path.join(d, "loss.so")
        with open(src, "w") as f:
            f.write(SHIM)
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", launch_rules.CSRC, src, "-o", so], check=True)
        L = ctypes.CDLL(so)
    L.group.argtypes, L.group.restype = [ctypes.c_int64] * 3, ctypes.c_int64
    L.step.argtypes, L.step.restype = [ctypes.c_int64] * 4, ctypes.c_int64
    L.cost.argtypes, L.cost.restype = [ctypes.c_int64] * 4, ctypes.c_double
    return L


def _sizes(n):
    rng = random.Random(7)
    lg = lambda lo, hi: int(lo * (hi / lo) ** rng.random())  # noqa: E731
    for _ in range(n):
        rows = lg(1, 1 << 20)
        c, vocab = -(-rows // lg(1, rows + 0.5)), lg(1, 300000)
        room, ld = (-(-c * vocab * 4 // 256) * 256 + -(-c * vocab * 2 // 256) * 256) // 4, -(-vocab // 32) * 32  # floats of the workspace
        yield rows, c, lg(1, 16384), room // (ld if c * ld <= room else vocab), vocab


def test_groups_within_their_bound(plan):
    for rows, c, hidden, _, _ in _sizes(20000):
        g = plan.group(rows, c, hidden)
        assert 0 < g <= max(c, 2 * hidden), (rows, c, hidden)
        # no more of them, each a pass over W and dW, than whole chunks would make
        assert -(-rows // g) <= -(-rows // (max(1, 2 * hidden // c) * c)), (rows, c, hidden)


def test_products_of_logits(plan):
    """What has room at once is one product; no more products than the chunks would make, or fewer
    clocks of them (launch_cost) than of as many rows as have room."""
    for rows, c, hidden, full, vocab in _sizes(20000):
        assert full >= c
        step = plan.step(rows, full, vocab, hidden)
        assert 0 < step <= full and (rows > full or step >= rows), (rows, c, hidden, full, vocab)
        assert -(-rows // step) <= -(-rows // c) or \
            plan.cost(rows, step, vocab, hidden) <= plan.cost(rows, full, vocab, hidden) * 16 / 15, (rows, c, hidden, full, vocab)


def test_whole_tiles_where_they_cost_less(plan):
    assert plan.group(65536, 1058, 4096) == 8192 and plan.step(8192, 1587, 128256, 4096) == 1536
    assert plan.step(2075, 390, 50304, 2048) == 256 and plan.step(3396, 1273, 16384, 4096) == 1024 and plan.step(1587, 595, 24000, 2048) == 512
    assert plan.step(1602, 400, 8000, 1024) == 400 and plan.step(300, 450, 8000, 2048) == 450


@pytest.mark.gpu
def test_gpu_scratch_of_a_small_hidden():
    """8 hidden, four million columns, a row a chunk: the gradients of 16 rows, 128 MiB, in the 256 MiB that the scratch starts
    with (256 rows would be 2 GiB)."""
    code = """
import torch
from paper_2408_16978_amd import tokenwise as TW
rows, hidden, vocab = 256, 8, 1 << 22
H = torch.randn(rows, hidden, device="cuda").to(torch.bfloat16)
W = torch.randn(vocab, hidden, device="cuda").to(torch.bfloat16)
t = torch.zeros(rows, dtype=torch.int32, device="cuda")
loss, lse, dH, dW = torch.empty(rows, device="cuda"), torch.empty(rows, device="cuda"), torch.empty_like(H), torch.zeros(vocab, hidden, device="cuda")
ws = torch.empty(TW.fpdt_tw_loss_workspace_bytes(rows, hidden, vocab, rows), dtype=torch.uint8, device="cuda")
torch.cuda.synchronize()
before = torch.cuda.mem_get_info()[0]
TW.fpdt_tw_loss_fwd_bwd(H, W, t, 1.0, loss, lse, dH, dW, rows, ws)
torch.cuda.synchronize()
print("took", (before - torch.cuda.mem_get_info()[0]) >> 20)
"""
    print("[case] scratch of a small hidden", flush=True)
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-2000:]
    assert int(r.stdout.split()[-1]) < 1024, r.stdout
