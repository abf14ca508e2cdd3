"""The loss's row kernel without gradients: the same loss and lse, to the bit, as with them, without a row kept in LDS."""
import pytest
import torch

import kernel_resources
from paper_2408_16978_amd import tokenwise as TW


def test_two_rows_fit_a_compute_unit():
    assert kernel_resources.workgroups_per_cu("tokenwise.hip", "loss_rows_kernel<1024, 0>", 16) == 2
    assert kernel_resources.workgroups_per_cu("tokenwise.hip", "loss_rows_kernel<1024, 32768>", 16) == 1


@pytest.mark.gpu
@pytest.mark.parametrize("vocab", [16383, 16384, 16385, 20000, 32768, 36870])
def test_gpu_same_bits_as_with_gradients(vocab):
    rows, hidden = 33, 64
    print("[case] loss rows without gradients", vocab, flush=True)
    g = torch.Generator(device="cuda").manual_seed(vocab)
    H = torch.randn(rows, hidden, device="cuda", generator=g).to(torch.bfloat16)
    W = (2 * torch.randn(vocab, hidden, device="cuda", generator=g) * hidden ** -0.5).to(torch.bfloat16)
    target = torch.randint(0, vocab, (rows,), device="cuda", generator=g, dtype=torch.int32)
    ws = torch.empty(TW.fpdt_tw_loss_workspace_bytes(rows, hidden, vocab, 1), dtype=torch.uint8, device="cuda")
    out = []
    for grads in (torch.zeros(vocab, hidden, device="cuda"), None):
        ws.fill_(255)
        loss, lse = torch.full((rows,), float("nan"), device="cuda"), torch.full((rows,), float("nan"), device="cuda")
        TW.fpdt_tw_loss_fwd_bwd(H, W, target, 1.0, loss, lse, None, grads, 1, ws)
        out.append((loss, lse))
    want = torch.logsumexp(H.double() @ W.double().t(), 1)
    assert float((out[1][1].double() - want).abs().max()) <= 2e-4  # as in test_loss_rows
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
