"""The loops of the attention kernels keep everything in registers: none of these kernels has scratch memory."""
import pytest

import kernel_resources


@pytest.mark.parametrize("source,kernel,count", [("fwd_bf16.hip", "fwd_sweep_kernel", 18), ("bwd_bf16.hip", "bwd_dq_kernel", 9), ("bwd_bf16.hip", "bwd_dq_ds_kernel", 9),
                                                 ("f32_path.hip", "f32_fwd_kernel", 3), ("f32_path.hip", "f32_bwd_kernel", 6)])
def test_no_scratch_memory(source, kernel, count):
    found = {n: v for n, v in kernel_resources.kernels(source).items() if n.split("<")[0] == kernel}
    assert len(found) == count and not [n for n, v in found.items() if v[2]], found
