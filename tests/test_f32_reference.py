"""The fp32 forward rescales a tile only where one of its rows has a new maximum: scores that climb slowly, by jumps, or
fall, and blocks of -infinity in front of, between and behind the others, must come out alike."""
import pytest
import torch

import parity
from paper_2408_16978_amd import inputs, runner


@pytest.mark.gpu
@pytest.mark.parametrize("S,chunk,Hq,Hkv,D", [(400, 400, 2, 1, 64), (333, 111, 2, 2, 80), (200, 200, 4, 2, 128), (17, 17, 1, 1, 64), (1, 1, 1, 1, 128)])
@pytest.mark.parametrize("slope", [0.05, 0.45, 0.55, 3.0, -1.0])
def test_gpu_f32_climbing_scores(S, chunk, Hq, Hkv, D, slope):
    """score(i, j) = slope j + noise: K grows along the first channel, in which Q is 1.  Against the oracle within the fp32
    tolerance (1e-4) and the rounding of the scores' sums: D additions, each off by 2^-24 of a partial sum, which is at most
    the largest score, delta = D 2^-24 |slope| S.  The LSE moves by that, a weight by twice that of itself, and with |V| <
    4.5 O by less than 9 delta."""
    print("[case] fp32 climbing scores", S, Hq, D, slope, flush=True)
    Q, K, V, dO = inputs.make_qkvdo(S, Hq, Hkv, D, "f32", 3)
    scale = D ** -0.5
    Q, K = Q * 0.5, K * 0.5
    Q[:, :, 0] = 1.0
    K[:, :, 0] = (slope / scale * torch.arange(S, dtype=torch.float32))[:, None]
    b = runner.make_buffers(Q, K, V, dO, chunk, scale, 0, bwd=False)
    runner.forward(b)
    torch.cuda.synchronize()
    ref = parity.oracle_full(Q, K, V, dO, scale)
    delta = D * 2.0 ** -24 * abs(slope) * S
    for name, got, times in (("O", b.O, 9), ("LSE", b.LSE, 1)):
        err = float((got.double().cpu() - torch.from_numpy(ref[name]).reshape(got.shape)).abs().max())
        assert err <= 1e-4 + times * delta, (name, err)


@pytest.mark.gpu
def test_gpu_f32_blocks_of_infinite_scores():
    """Keys whose scores overflow to -infinity, whole blocks of them in front of, between and behind the finite ones: they
    weigh nothing, and a row that has only them is not a number, with an LSE of -infinity."""
    S, D = 300, 64
    Q, K, V, dO = inputs.make_qkvdo(S, 1, 1, D, "f32", 5)
    Q[:, :, 0] = 1e30
    K[:, :, 0] = 0.0
    off = torch.zeros(S, dtype=torch.bool)
    off[:35] = off[100:180] = off[290:] = True
    K[off, :, 0] = -1e30
    b = runner.make_buffers(Q, K, V, dO, S, D ** -0.5, 0, bwd=False)
    runner.forward(b)
    torch.cuda.synchronize()
    O, LSE = b.O[:, 0].double().cpu(), b.LSE[0].double().cpu()
    assert bool(O[:35].isnan().all()) and bool((LSE[:35] == float("-inf")).all())
    s = (Q[:, 0].double() @ K[:, 0].double().t() * D ** -0.5).masked_fill(off[None, :] | torch.ones(S, S, dtype=torch.bool).triu(1), float("-inf"))
    want = torch.softmax(s, -1) @ V[:, 0].double()
    assert float((O - want)[35:].abs().max()) <= 1e-4
    assert float((LSE - torch.logsumexp(s, -1))[35:].abs().max()) <= 1e-4


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 80, 128])
def test_gpu_f32_elements_that_are_not_finite(D):
    """One infinite element of V, or of dO, in a tile of rows that are otherwise finite: it shows in its own channel of the rows
    that attend it, or that it attends, and leaves every other result alone, bit for bit."""
    S, row, d = 150, 70, 5

    def run(V, dO):
        b = runner.make_buffers(Q, K, V, dO, S, D ** -0.5, 0)
        runner.forward(b)
        runner.backward(b)
        torch.cuda.synchronize()
        return b

    print("[case] fp32 elements that are not finite", D, flush=True)
    Q, K, V, dO = inputs.make_qkvdo(S, 2, 1, D, "f32", 6)
    want = run(V, dO)
    others = torch.arange(D) != d
    odd = V.clone()
    odd[row, 0, d] = float("inf")
    O = run(odd, dO).O
    assert torch.equal(O[:row], want.O[:row]) and torch.equal(O[:, :, others], want.O[:, :, others]) and bool((O[row:, :, d] == float("inf")).all())
    odd = dO.clone()
    odd[row, 1, d] = float("inf")
    got = run(V, odd)
    assert torch.equal(got.dV[row + 1:], want.dV[row + 1:]) and torch.equal(got.dV[:, :, others], want.dV[:, :, others])
    assert bool((got.dV[:row + 1, :, d] == float("inf")).all())
    assert torch.equal(got.dK[row + 1:], want.dK[row + 1:]) and torch.equal(got.dQ[:, 0], want.dQ[:, 0])
    rest = torch.arange(S) != row
    assert torch.equal(got.dQ[rest][:, 1], want.dQ[rest][:, 1])
