"""What the binding hands out and refuses, whatever the layout and type of its arguments."""
import pytest
import torch

from paper_2501_02573_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2501_02573_amd import binding
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return binding


def _entry_points(B, q, k, v, gamma):
    """The outputs of every entry point that makes its own (decode steps if there is one token)."""
    b, h, n, d = q.shape
    S = torch.zeros((b, h, d, d), device="cuda")
    yield B.leet_attn_forward(q, k, v, gamma)
    yield B.leet_attn_forward_ex(q, k, v, gamma)
    yield B.leet_attn_forward_v2(q, k, v, gamma)
    yield B.leet_attn_forward_v2(q, k, v, gamma, out_dtype=q.dtype)
    yield B.leet_attn_forward_rd(q, k, v, gamma)
    yield B.leet_attn_forward_v3(q, k, v, gamma)
    yield B.leet_attn_forward_recurrent(q, k, v, gamma)
    yield B.leet_attn_forward_recurrent_rd(q, k, v, gamma)
    yield B.leet_attn_forward_fleet(q, k, v, gamma)
    yield B.leet_attn_forward_profile(q, k, v, gamma)[0]
    if n == 1:
        q, k, v = (t.select(2, 0) for t in (q, k, v))
        yield B.leet_attn_decode_step(q, k, v, gamma, S)
        yield B.leet_attn_decode_step_ex(q, k, v, gamma, S)
        yield B.leet_attn_decode_step_v2(q, k, v, gamma, S)
        yield B.leet_attn_decode_step_rd(q, k, v, gamma, S)


def _standard_strides(t):
    return torch.empty(t.shape, device="meta").stride()


def test_outputs_have_the_strides_of_a_fresh_tensor(B):
    # one head, seen through a transpose: contiguous, with another stride in the dimension of size one
    x = [torch.randn((2, 5, 1, 64), device="cuda").bfloat16()[:1].transpose(1, 2) for _ in range(3)]
    gamma = torch.full((1,), 0.9, device="cuda")
    assert x[0].is_contiguous() and x[0].stride() != _standard_strides(x[0])
    for n, out in enumerate(_entry_points(B, *x, gamma)):
        assert out.stride() == _standard_strides(out), n
    x = [torch.randn((2, 1, 64), device="cuda").bfloat16().as_strided((2, 1, 1, 64), (64, 7, 9, 1)) for _ in range(3)]
    for n, out in enumerate(_entry_points(B, *x, gamma)):
        assert out.stride() == _standard_strides(out), n


def test_outputs_are_plain_tensors(B):
    class Named(torch.Tensor):
        pass

    x = [torch.randn((2, 1, 1, 64), device="cuda").bfloat16().as_subclass(Named) for _ in range(3)]
    for n, out in enumerate(_entry_points(B, *x, torch.full((1,), 0.9, device="cuda"))):
        assert type(out) is torch.Tensor, n


@pytest.mark.parametrize("stream", ["0", 0.0, 1.5, b"0"])
def test_a_prepared_call_takes_a_stream_handle_only(B, stream):
    q, k, v, gamma = (t.cuda() for t in W.make_custom_forward_inputs(1, 1, 8, 64, "bf16", seed=1))
    out = torch.empty((1, 1, 8, 64), device="cuda")
    with pytest.raises(TypeError):
        B.PreparedForward(q, k, v, gamma, out, stream=stream)


def test_a_prepared_call_runs_on_the_stream_it_was_given(B):
    q, k, v, gamma = (t.cuda() for t in W.make_custom_forward_inputs(1, 4, 300, 64, "bf16", seed=2))
    want = B.leet_attn_forward(q, k, v, gamma)
    stream = torch.cuda.Stream()
    for handle in (stream.cuda_stream, 0):
        out = torch.zeros_like(want)
        torch.cuda.synchronize()
        B.PreparedForward(q, k, v, gamma, out, stream=handle)()
        torch.cuda.synchronize()
        assert torch.equal(out, want)
