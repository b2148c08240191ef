"""The fp32 chunk walks at the edges of their tiles (32 tokens at width 128, 64 at width 64), against the fp64 oracle,
exponents that move by powers of two, and non-finite tokens kept from earlier ones.  What lies outside the range
of three-term operands is in test_gpu_f32_range.py."""
import numpy as np
import pytest
import torch

import oracle
from helpers import max_rel_err
from paper_2501_02573_amd import workloads as W

pytestmark = pytest.mark.gpu

# Products round at 2^-24 (test_gpu_f32_products.py); an output is the sum of two fp32 contractions (128 and 32 terms a
# tile, fewer than 64 roundings at full size between them) of operands that carry as many again.  With random
# signs that is sqrt(128) * 2^-25 = 3.4e-7 of the head's largest value; six of that.  A partial product
# left out (2^-16 to 2^-17 of a term) shows as 4e-6 and more.
TOL = 2e-6


@pytest.fixture(scope="module")
def B():
    from paper_2501_02573_amd import binding
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return binding


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N,segments", [(1, 0), (2, 0), (31, 0), (32, 0), (33, 0), (63, 1), (64, 0), (65, 2), (95, 1),
                                        (97, 2), (128, 2), (191, 3), (450, 0), (600, 5), (1100, 17)])
def test_tile_edges_with_state_in_place(B, d, N, segments):
    q, k, v, gamma = W.make_custom_forward_inputs(2, 3, N, d, "f32", seed=1000 + N + d)
    state = torch.randn((2, 3, d, d), generator=torch.Generator().manual_seed(N)) * 0.1
    ref, s_ref = oracle.recurrent(*(W.to_f64(t) for t in (q, k, v, gamma)), W.to_f64(state))
    S = state.cuda()
    out = B.leet_attn_forward_v2(q.cuda(), k.cuda(), v.cuda(), gamma.cuda(), state_in=S, state_out=S, segments=segments)
    errs = max_rel_err(out.cpu().numpy(), ref), max_rel_err(S.cpu().numpy(), s_ref)
    print(f"  N {N} d {d} segments {segments}: out {errs[0]:.2e} state {errs[1]:.2e}", flush=True)
    assert max(errs) <= TOL


@pytest.mark.parametrize("tile", [0, 1, 6, 7, 8, 15, 16, 21])
def test_width_128_finds_an_infinity_in_any_tile(B, tile):
    # the walk looks up every second tile whether it has to be taken again, and at its end
    N, col = 700, 77
    q, k, v, gamma = W.make_custom_forward_inputs(1, 2, N, 128, "f32", seed=40 + tile)
    tok = 32 * tile + 16  # the first of a sixteen: earlier tokens of its sixteen would meet it with a weight of zero
    ref, _ = oracle.recurrent(*(W.to_f64(t) for t in (q, k, v, gamma)))
    v[0, 1, tok, col] = float("inf")
    out = B.leet_attn_forward_v2(q.cuda(), k.cuda(), v.cuda(), gamma.cuda(), segments=1).cpu().numpy()
    # infinite, or, once the state's infinities of both signs are summed, NaN
    assert not np.any(np.isfinite(out[0, 1, tok:, col]))
    out[0, 1, tok:, col] = ref[0, 1, tok:, col]
    assert np.all(np.isfinite(out))
    assert max_rel_err(out, ref) <= TOL


@pytest.mark.parametrize("d", [64, 128])
def test_powers_of_two_pass_through_exactly(B, d):
    q, k, v, gamma = (t.cuda() for t in W.make_custom_forward_inputs(1, 2, 300, d, "f32", seed=7))
    out = B.leet_attn_forward(q, k, v, gamma)
    scaled = B.leet_attn_forward(q * 2.0 ** 60, k * 2.0 ** -40, v * 2.0 ** 30, gamma)
    assert torch.equal(scaled, out * 2.0 ** 50)


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), 3.4e38])
def test_large_and_non_finite_tokens_do_not_reach_earlier_sixteens(B, bad):
    q, k, v, gamma = (t.cuda() for t in W.make_custom_forward_inputs(1, 1, 200, 64, "f32", seed=8))
    clean = B.leet_attn_forward(q, k, v, gamma)
    for t, x in (("k", k), ("v", v), ("q", q)):
        y = x.clone()
        y[0, 0, 117] = bad
        out = B.leet_attn_forward(y if t == "q" else q, y if t == "k" else k, y if t == "v" else v, gamma)
        first = 117 if t == "q" else 112
        assert torch.equal(out[0, 0, :first], clean[0, 0, :first]), t
        assert t != "q" or torch.equal(out[0, 0, 118:], clean[0, 0, 118:])
        if not np.isfinite(bad):
            assert not torch.isfinite(out[0, 0, 117]).any(), t
