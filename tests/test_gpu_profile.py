"""Per-kernel times of a prefill: a kernel that a plan does not launch takes no time."""
import pytest
import torch

from paper_2501_02573_amd import workloads as W

pytestmark = pytest.mark.gpu


# launched: pre-pass, scan, walk
@pytest.mark.parametrize("dtype,B,H,N,d,segments,launched", [
    ("f32", 1, 1, 256, 64, 1, (False, False, True)),
    ("f32", 1, 1, 256, 64, 4, (True, False, True)),     # three states of 16 KB: the walk combines them
    ("f32", 2, 8, 2048, 64, 0, (True, False, True)),    # fifteen of them
    ("f32", 1, 2, 256, 128, 4, (True, False, True)),    # three of 64 KB
    ("f32", 1, 2, 512, 128, 8, (True, True, True)),     # seven of 64 KB: the scan does
    ("f32", 1, 2, 2048, 64, 32, (True, True, True)),
    ("bf16", 1, 2, 2048, 64, 4, (True, True, True)),
])
def test_kernels_that_are_not_launched_take_no_time(dtype, B, H, N, d, segments, launched):
    from paper_2501_02573_amd import binding
    q, k, v, gamma = (t.cuda() for t in W.make_custom_forward_inputs(B, H, N, d, dtype, seed=1))
    out, ms = binding.leet_attn_forward_profile(q, k, v, gamma, segments=segments)
    assert tuple(t > 0 for t in ms) == launched, ms
    assert torch.equal(out, binding.leet_attn_forward_ex(q, k, v, gamma, segments=segments))
