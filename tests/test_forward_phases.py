"""The forward's two phases per tile (csrc/fwd_bf16.hip): every count of tiles from one on, odd and even, up to where the steady loop takes
most of them, for each number of key groups and both tile heights."""
import pytest
import torch

import launch_rules
import parity
from paper_2408_16978_amd import binding as B
from paper_2408_16978_amd import inputs, runner


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 80, 128])
@pytest.mark.parametrize("S,Hq,Hkv,groups", [(256, 3, 1, 4), (512, 3, 3, 4), (768, 3, 1, 4), (1024, 2, 1, 4), (1280, 2, 2, 4),
                                             (256, 96, 8, 2), (512, 64, 8, 2), (768, 48, 6, 2), (256, 256, 32, 1), (512, 160, 20, 1)])
def test_gpu_every_count_of_tiles(S, Hq, Hkv, groups, D):
    print("[case] forward phases", S, Hq, Hkv, D, flush=True)
    assert launch_rules.forward_key_groups(S, Hq) == groups
    Q, K, V, dO = inputs.make_qkvdo(S, Hq, Hkv, D, "bf16", 31)
    scale = D ** -0.5
    b = runner.make_buffers(Q, K, V, dO, S, scale, 0, bwd=False)
    pairs = runner.make_buffers(Q, K, V, dO, 256, scale, B.FPDT_PAIRWISE, bwd=False)
    runner.forward(b)
    runner.forward(pairs)
    torch.cuda.synchronize()
    assert torch.equal(b.O, pairs.O) and torch.equal(b.LSE, pairs.LSE)
    ref = parity.oracle_full(Q, K, V, dO, scale)
    print(parity.check_all({"O": b.O, "LSE": b.LSE}, ref, True, names=("O", "LSE")))
