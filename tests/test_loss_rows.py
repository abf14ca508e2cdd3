"""The loss's row kernel around its two widths (16384 logits), its trips of 1024 x 16 bytes and its 32768 logits in LDS, with
vocabularies that are not a multiple of 4, and its row groups: logits of other row counts than the chunks', gradients of
several chunks multiplied together."""
import pytest
import torch

from paper_2408_16978_amd import tokenwise as TW


@pytest.mark.gpu
@pytest.mark.parametrize("rows,hidden,vocab,n_chunks", [
    (37, 64, 16380, 1), (37, 64, 16383, 3), (64, 64, 16384, 64), (37, 64, 16385, 37), (40, 64, 32766, 2), (40, 64, 32768, 5),
    (33, 40, 36870, 4), (700, 128, 20001, 2), (1300, 512, 1027, 2), (1300, 256, 1024, 3), (2100, 64, 53, 9), (5, 3, 1, 2)])
def test_gpu_loss_row_groups(rows, hidden, vocab, n_chunks):
    """Against fp64: loss and lse to fp32 round-off of the logits' sums, gradients as in test_tokenwise (a logit gradient
    rounded to bf16 before it is multiplied)."""
    print("[case] loss rows", rows, hidden, vocab, n_chunks, flush=True)
    g = torch.Generator(device="cuda").manual_seed(rows + vocab)
    H = torch.randn(rows, hidden, device="cuda", generator=g).to(torch.bfloat16)
    W = (2 * torch.randn(vocab, hidden, device="cuda", generator=g) * hidden ** -0.5).to(torch.bfloat16)
    target = torch.randint(0, vocab, (rows,), device="cuda", generator=g, dtype=torch.int32)
    target[0], target[rows - 1] = vocab - 1, 0
    logits = H.double() @ W.double().t()
    want_lse = torch.logsumexp(logits, 1)
    want_loss = want_lse - logits.gather(1, target.long()[:, None])[:, 0]
    G = torch.softmax(logits, 1)
    G[torch.arange(rows, device="cuda"), target.long()] -= 1
    G /= rows
    ws = torch.empty(TW.fpdt_tw_loss_workspace_bytes(rows, hidden, vocab, n_chunks), dtype=torch.uint8, device="cuda")
    loss, lse = torch.empty(rows, device="cuda"), torch.empty(rows, device="cuda")
    dH, dW = torch.full_like(H, float("nan")), torch.zeros(vocab, hidden, device="cuda")
    for with_grad in (True, False):
        ws.fill_(255)  # NaN in whatever is read without having been written
        loss.fill_(float("nan"))
        lse.fill_(float("nan"))
        TW.fpdt_tw_loss_fwd_bwd(H, W, target, 1.0 / rows, loss, lse, dH if with_grad else None, dW if with_grad else None, n_chunks, ws)
        assert float((lse.double() - want_lse).abs().max()) <= 2e-4
        assert float((loss.double() - want_loss).abs().max()) <= 2e-4
    for name, got, ref in (("dH", dH, G @ W.double()), ("dW", dW, G.t() @ H.double())):
        budget = 2e-2 * ref.pow(2).mean(1, keepdim=True).sqrt() + 2.0 ** -8 * ref.abs() + 1e-9
        assert bool(((got.double() - ref).abs() <= budget).all()), name
