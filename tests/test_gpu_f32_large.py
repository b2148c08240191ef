"""fp32 prefills that the small cases do not reach: inputs beyond the last-level cache (loaded nontemporally by an
instance of the kernels of its own), and segment states combined by the walk on grids that do not fit the device
at once, with the state handed on in place."""
import numpy as np
import pytest
import torch

import oracle
from helpers import max_rel_err
from paper_2501_02573_amd import workloads as W

pytestmark = pytest.mark.gpu

# fp32 sums of up to some thousand terms in tiles of 32 and 64, as in the cases at the tiles' edges
TOL = 2e-6


@pytest.fixture(scope="module")
def B():
    from paper_2501_02573_amd import binding
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return binding


def _check(B, b, h, N, d, gamma, segments, seed):
    q, k, v, gamma = W.make_custom_forward_inputs(b, h, N, d, "f32", seed=seed, gamma=gamma)
    state = torch.randn((b, h, d, d), generator=torch.Generator().manual_seed(seed)) * 0.1
    ref, s_ref = oracle.recurrent(*(W.to_f64(t) for t in (q, k, v, gamma)), W.to_f64(state))
    S = state.cuda()
    out = B.leet_attn_forward_v2(q.cuda(), k.cuda(), v.cuda(), gamma.cuda(), state_in=S, state_out=S, segments=segments)
    errs = max_rel_err(out.cpu().numpy(), ref), max_rel_err(S.cpu().numpy(), s_ref)
    print(f"  B {b} H {h} N {N} d {d} segments {segments}: out {errs[0]:.2e} state {errs[1]:.2e}", flush=True)
    assert max(errs) <= TOL


@pytest.mark.parametrize("h,N,d,segments", [(9, 19555, 128, 0), (9, 19555, 128, 2), (24, 7401, 128, 1), (13, 27001, 64, 0)])
def test_inputs_beyond_the_last_level_cache(B, h, N, d, segments):
    assert h * N * 3 * d * 4 > 256 << 20
    gamma = W.make_gamma("pow2:4:9", h)
    gamma[1] = 0.3  # width 128: a head that runs on the fp32 matrix instructions
    _check(B, 1, h, N, d, gamma, segments, seed=h)


@pytest.mark.parametrize("b,h,N,d,segments", [(25, 12, 250, 128, 4), (40, 10, 129, 128, 3), (20, 16, 1020, 64, 16), (50, 16, 250, 64, 4)])
def test_combined_states_in_place_on_a_grid_of_several_rounds(B, b, h, N, d, segments):
    nseg, _ = B.query_plan(b, h, N, d, B.LEET_F32, segments)
    # the walk combines: no finer pre-pass segments, and at most 240 KB of states before a segment
    assert nseg == segments and B.workspace_bytes(b, h, N, d, B.LEET_F32, segments) == b * h * nseg * d * d * 4
    assert (nseg - 1) * d * d * 4 <= 240 << 10 and b * h * nseg > 4 * 256
    _check(B, b, h, N, d, W.make_gamma("pow2:4:9", h), segments, seed=N)
