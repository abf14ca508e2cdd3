"""The reference that a row's probabilities are taken against, with one key group (csrc/fwd_bf16.hip): the largest score of the row's first 64
keys, at every head dimension, so that the largest of them has a probability that bf16 holds exactly."""
import math

import pytest
import torch

import launch_rules
from paper_2408_16978_amd import binding as B
from paper_2408_16978_amd import inputs, runner


@pytest.mark.gpu
@pytest.mark.parametrize("first,second", [(5, 40), (0, 63), (31, 32)])
@pytest.mark.parametrize("D", [64, 80, 128])
def test_gpu_reference_of_the_first_64_keys(D, first, second):
    """Two keys count: one of the first 32 and, with a score log(4 / 3) higher, one of the next.  Against the second the first's probability is 3/4
    and P is exact; against the first the second's is 4/3, which bf16 rounds by 1/512, and V is such that O then is half as large again.
    What is left is the rounding of O, 2^-9 of it."""
    S, Hq, Hkv = 512, 160, 20
    print("[case] reference of 64 keys", D, first, second, flush=True)
    assert launch_rules.forward_key_groups(S, Hq) == 1
    Q, K, V, dO = inputs.make_qkvdo(S, Hq, Hkv, D, "bf16", 61)
    Q.zero_(), K.zero_()
    Q[:, :, 0], K[:, :, 0] = 1.0, -1000.0
    K[first, :, 0], K[second, :, 0] = 0.0, 1.0
    V[first], V[second] = -1.328125, 1.0
    scale = math.log(4 / 3)
    want = (0.75 * -1.328125 + 1.0) / 1.75
    for chunk, flags in ((S, 0), (256, B.FPDT_PAIRWISE)):
        b = runner.make_buffers(Q, K, V, dO, chunk, scale, flags, bwd=False)
        runner.forward(b)
        torch.cuda.synchronize()
        assert float((b.O[second:].double() / want - 1).abs().max()) <= 2.0 ** -8
        # (a sum and its logarithm in fp32, values around 1)
        assert float((b.LSE[:, second:].double() - (scale + math.log(1.75))).abs().max()) <= 1e-6
