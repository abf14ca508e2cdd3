"""bf16 forward: infinities and NaN in keys and values that the causal mask excludes.  Keys leave every row that does not see them alone; a value
that is not finite reaches the rows of its own block of 32 at most (0 times it is not a number), whatever the key groups, the blocks of a tile and
where K and V are read from."""
import pytest
import torch

import launch_rules
from paper_2408_16978_amd import binding as B
from paper_2408_16978_amd import inputs, runner


def _forward(Q, K, V, chunk, flags):
    b = runner.make_buffers(Q, K, V, Q, chunk, Q.shape[2] ** -0.5, flags, bwd=False)
    runner.forward(b)
    torch.cuda.synchronize()
    return b.O, b.LSE


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 80, 128])
@pytest.mark.parametrize("S,Hq,Hkv,groups", [(512, 4, 2, 4), (768, 48, 6, 2), (512, 64, 64, 2), (512, 160, 20, 1), (2048, 64, 8, 1)])
def test_gpu_later_keys_and_values_may_hold_anything(S, Hq, Hkv, groups, D):
    print("[case] values that are not finite", S, Hq, Hkv, D, flush=True)
    assert launch_rules.forward_key_groups(S, Hq) == groups
    Q, K, V, _ = inputs.make_qkvdo(S, Hq, Hkv, D, "bf16", 62, device="cuda")
    for chunk, flags in ((S, 0), (256, B.FPDT_PAIRWISE)):
        O, LSE = _forward(Q, K, V, chunk, flags)
        for key in (32, 63, 96, 97, 224, S - 32):
            for bad in (float("inf"), float("nan")):
                k, v = K.clone(), V.clone()
                k[key], v[key] = bad, bad
                rows = key // 32 * 32
                # (a wave whose later rows see such a key takes new references for all of its 32 rows: P is rounded elsewhere, by 2^-9 of it
                # on either side, and so is O)
                o, lse = _forward(Q, k, V, chunk, flags)
                assert torch.equal(o[:rows], O[:rows]) and torch.equal(lse[:, :rows], LSE[:, :rows]), (key, bad)
                if key > rows:
                    assert float((o[rows:key].double() - O[rows:key].double()).abs().max()) <= 2.0 ** -7 * float(V[:key].abs().max()), (key, bad)
                    assert float((lse[:, rows:key] - LSE[:, rows:key]).abs().max()) <= 1e-5, (key, bad)
                o, lse = _forward(Q, K, v, chunk, flags)
                assert torch.equal(o[:rows], O[:rows]) and torch.equal(lse, LSE), (key, bad)
                assert not bool(o[key:].isfinite().any())
