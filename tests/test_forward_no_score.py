"""bf16 rows whose scores all overflow to -infinity: O is not a number, the LSE -infinity, as in fp32, with every count of key groups and in both
schedules.  Behind such keys a row that also has finite scores is what these make of it."""
import pytest
import torch

import launch_rules
from paper_2408_16978_amd import binding as B
from paper_2408_16978_amd import inputs, runner


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 80, 128])
@pytest.mark.parametrize("S,Hq,Hkv,groups", [(512, 4, 2, 4), (768, 48, 6, 2), (512, 160, 20, 1)])
@pytest.mark.parametrize("empty", [1, 33, 70, 300])
def test_gpu_rows_without_a_finite_score(S, Hq, Hkv, groups, D, empty):
    print("[case] rows without a finite score", S, Hq, Hkv, D, empty, flush=True)
    assert launch_rules.forward_key_groups(S, Hq) == groups
    Q, K, V, _ = inputs.make_qkvdo(S, Hq, Hkv, D, "bf16", 63, device="cuda")
    Q[:, :, 0], K[:, :, 0] = 1e30, 0.0
    K[:empty, :, 0] = -1e30
    scale = D ** -0.5
    q, k, v = (t.double().transpose(0, 1) for t in (Q, K.repeat_interleave(Hq // Hkv, 1), V.repeat_interleave(Hq // Hkv, 1)))
    s = torch.matmul(q, k.transpose(1, 2).contiguous()) * scale
    off = torch.ones(S, S, dtype=torch.bool, device="cuda").triu(1) | (torch.arange(S, device="cuda") < empty)[None]
    s.masked_fill_(off, float("-inf"))
    lse = torch.logsumexp(s, 2)
    o = torch.matmul(torch.softmax(s, 2), v).transpose(0, 1)
    for chunk, flags in ((S, 0), (256, B.FPDT_PAIRWISE)):
        b = runner.make_buffers(Q, K, V, Q, chunk, scale, flags, bwd=False)
        runner.forward(b)
        torch.cuda.synchronize()
        assert bool(b.O[:empty].isnan().all()) and bool((b.LSE[:, :empty] == float("-inf")).all())
        # P and O are rounded to bf16, by 2^-9 each and P's share of the sum of |p v| at most: 2^-7 of the largest value
        assert float((b.O[empty:].double() - o[empty:]).abs().max()) <= 2.0 ** -7 * float(V.abs().max())
        assert float((b.LSE[:, empty:].double() - lse[:, empty:]).abs().max()) <= 1e-4
