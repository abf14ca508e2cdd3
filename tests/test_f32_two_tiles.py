"""The fp32 forward with two workgroups on a compute unit at D = 64 and 80, and the order of its tiles around 256 and 512 of them,
where the second half starts with the shortest."""
import pytest
import torch

import kernel_resources
from paper_2408_16978_amd import inputs, runner


@pytest.mark.parametrize("D", [64, 80])
def test_two_workgroups_fit_a_compute_unit(D):
    assert kernel_resources.workgroups_per_cu("f32_path.hip", "f32_fwd_kernel<%d>" % D, 8) >= 2


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 80, 128])
@pytest.mark.parametrize("S,Hq,Hkv", [(4096, 1, 1), (4097, 1, 1), (1030, 4, 2), (2720, 3, 1), (8176, 1, 1), (2048, 4, 4), (2049, 4, 1)])
def test_gpu_every_tile_runs(S, Hq, Hkv, D):
    """255 .. 516 tiles of 16 rows.  Against fp64 within the fp32 tolerance, 1e-4."""
    print("[case] fp32 tiles", S, Hq, Hkv, D, flush=True)
    Q, K, V, dO = inputs.make_qkvdo(S, Hq, Hkv, D, "f32", 31, device="cuda")
    b = runner.make_buffers(Q, K, V, dO, S, D ** -0.5, 0, bwd=False)
    b.O.fill_(float("nan"))
    b.LSE.fill_(float("nan"))
    runner.forward(b)
    mask = torch.ones(S, S, dtype=torch.bool, device="cuda").triu(1)
    for h in range(Hq):
        s = (Q[:, h].double() @ K[:, h * Hkv // Hq].double().t() * D ** -0.5).masked_fill(mask, float("-inf"))
        assert float((b.LSE[h].double() - torch.logsumexp(s, 1)).abs().max()) <= 1e-4
        assert float((b.O[:, h].double() - torch.softmax(s, 1) @ V[:, h * Hkv // Hq].double()).abs().max()) <= 1e-4
