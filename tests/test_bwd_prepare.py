"""The launch that prepares a backward over the whole sequence (Delta, row statistics, packed operands): the shortest sequence, where every row
has its exact Delta, the first with rows of the other kind, and head counts that leave no power of two.  The pair-by-pair schedule makes the same
with launches of their own."""
import pytest
import torch

import launch_rules
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


@pytest.mark.parametrize("S,Hq,Hkv,launches", [(256, 1, 1, 1), (2048, 8, 2, 1), (1 << 21, 8, 2, 1), (32 * 41120, 64, 6, 1), (32 * 41152, 64, 6, 2), (1 << 22, 64, 8, 4),
                                               (4096, 13312, 13312, 2)])
def test_launches_of_fewer_than_2_to_the_32_lanes(S, Hq, Hkv, launches):
    """512 lanes a workgroup; every block of Delta, and of the four tensors, once."""
    got = launch_rules.prepare_launches(S, Hq, Hkv)
    assert len(got) == launches and all(512 * n < 2 ** 32 for _, n in got)
    at = 0
    for first, n in got:
        assert first == at and n > 0
        at += n
    assert at == S // 32 * (Hq + 2 * (Hq + Hkv)) < 2 ** 32


@pytest.mark.gpu
def test_gpu_backward_prepared_by_two_launches():
    """13312 heads of 4096 tokens: 64 of them, repeated, so that every repetition has the bits of the first, and these
    what the 64 heads alone give (whose sums are split otherwise: the tolerance of the bf16 gradients)."""
    S, few, times, D = 4096, 64, 208, 64
    print("[case] prepared by two launches", S, few * times, D, flush=True)
    assert len(launch_rules.prepare_launches(S, few * times, few * times)) == 2
    scale = D ** -0.5
    small = runner.make_buffers(*inputs.make_qkvdo(S, few, few, D, "bf16", 52, device="cuda"), S, scale, 0)
    runner.forward(small)
    runner.backward(small)
    b = runner.make_buffers(*(t.repeat(1, times, 1) for t in (small.Q, small.K, small.V, small.dO)), S, scale, 0)
    b.O.copy_(small.O.repeat(1, times, 1))
    b.LSE.copy_(small.LSE.repeat(times, 1))
    runner.backward(b)
    torch.cuda.synchronize()
    for n in ("dQ", "dK", "dV"):
        got, want = getattr(b, n), getattr(small, n)
        for i in range(1, times):
            assert torch.equal(got[:, i * few:(i + 1) * few], got[:, :few]), (n, i)
        rms = want.double().pow(2).mean().sqrt()
        assert float((got[:, :few].double() - want.double()).abs().max() / rms) <= 2e-2 * max(1.0, float(want.double().abs().max() / rms)), n
