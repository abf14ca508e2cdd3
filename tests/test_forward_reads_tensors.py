"""The forward that reads K and V from their tensors (launch_rules.h, sweep_reads_tensors): every head dimension with two and
four key groups, several KV heads (a row's pitch), against the pair-by-pair schedule, which packs them; and outputs in the
place of K or V, which have to be packed."""
import pytest
import torch

import launch_rules
from paper_2408_16978_amd import binding as B
from paper_2408_16978_amd import inputs, runner


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 80, 128])
@pytest.mark.parametrize("S,Hq,Hkv,groups", [(256, 1, 1, 4), (768, 6, 3, 4), (1280, 8, 1, 4), (1024, 48, 6, 2), (512, 64, 64, 2)])
def test_gpu_same_bits_as_from_packed_fragments(S, Hq, Hkv, groups, D):
    print("[case] forward from tensors", S, Hq, Hkv, D, flush=True)
    assert launch_rules.forward_key_groups(S, Hq) == groups
    Q, K, V, dO = inputs.make_qkvdo(S, Hq, Hkv, D, "bf16", 21, device="cuda")
    one = runner.make_buffers(Q, K, V, dO, S, D ** -0.5, 0, bwd=False)
    pairs = runner.make_buffers(Q, K, V, dO, 256, D ** -0.5, B.FPDT_PAIRWISE, bwd=False)
    runner.forward(one)
    runner.forward(pairs)
    torch.cuda.synchronize()
    assert torch.equal(one.O, pairs.O) and torch.equal(one.LSE, pairs.LSE)


@pytest.mark.gpu
@pytest.mark.parametrize("place", ["K", "V"])
def test_gpu_output_in_the_place_of_keys_or_values(place):
    S, H, D = 768, 4, 128
    Q, K, V, _ = inputs.make_qkvdo(S, H, H, D, "bf16", 22, device="cuda")
    O, LSE = torch.empty_like(Q), torch.empty(H, S, device="cuda")
    B.fpdt_attn_fwd_noalloc(Q, K, V, O, LSE, S, D ** -0.5)
    k, v, lse = K.clone(), V.clone(), torch.empty_like(LSE)
    out = k if place == "K" else v
    B.fpdt_attn_fwd_noalloc(Q, k, v, out, lse, S, D ** -0.5)
    torch.cuda.synchronize()
    assert torch.equal(out, O) and torch.equal(lse, LSE)
