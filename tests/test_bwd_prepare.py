"""The launch that prepares a backward over the whole sequence (Delta, row statistics, packed operands): the shortest sequence, where every row
has its exact Delta, the first with rows of the other kind, and head counts that leave no power of two.  The pair-by-pair schedule makes the same
with launches of their own."""
import pytest
import torch

import parity
from paper_2408_16978_amd import binding as B
from paper_2408_16978_amd import inputs, runner


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 80, 128])
@pytest.mark.parametrize("S,Hq,Hkv", [(256, 1, 1), (256, 6, 3), (512, 5, 5), (768, 7, 1), (1024, 12, 4)])
def test_gpu_prepared_backward(S, Hq, Hkv, D):
    print("[case] prepared backward", S, Hq, Hkv, D, flush=True)
    Q, K, V, dO = inputs.make_qkvdo(S, Hq, Hkv, D, "bf16", 51)
    scale = D ** -0.5
    ref = parity.oracle_full(Q, K, V, dO, scale)
    for chunk, flags in ((S, 0), (256, B.FPDT_PAIRWISE)):
        b = runner.make_buffers(Q, K, V, dO, chunk, scale, flags)
        b.ws_bwd.fill_(0xFF)
        runner.forward(b)
        runner.backward(b)
        torch.cuda.synchronize()
        print(parity.check_all({"O": b.O, "LSE": b.LSE, "dQ": b.dQ, "dK": b.dK, "dV": b.dV}, ref, True))
