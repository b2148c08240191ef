"""The fp32 kernel outside the range in which its 16-bit terms hold an operand exactly: infinities,
overflow, magnitudes near both ends of fp32.  Results there are those of fp32 products."""
import numpy as np
import pytest
import torch

import oracle
from helpers import max_rel_err
from paper_2501_02573_amd import workloads as W

pytestmark = pytest.mark.gpu

INF = float("inf")


@pytest.fixture(scope="module")
def B():
    from paper_2501_02573_amd import binding
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return binding


def _positive(N, d, seed):
    """q, k, v > 0: an infinity then reaches every output that depends on it with a known sign."""
    q, k, v, gamma = W.make_custom_forward_inputs(1, 2, N, d, "f32", seed=seed)
    return q.abs() + 2.0 ** -10, k.abs() + 2.0 ** -10, v.abs() + 2.0 ** -10, gamma


def _run(B, q, k, v, gamma, state=None, segments=0):
    s_out = torch.empty((*q.shape[:2], q.shape[3], q.shape[3]), device="cuda")
    out = B.leet_attn_forward_v2(q.cuda(), k.cuda(), v.cuda(), gamma.cuda(), state_in=None if state is None else state.cuda(),
                                 state_out=s_out, segments=segments)
    return out.cpu().numpy(), s_out.cpu().numpy()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("segments", [1, 3])
@pytest.mark.parametrize("where", ["q", "k", "v", "state"])
def test_an_infinity_reaches_what_it_should_as_an_infinity(B, d, segments, where):
    # entry (token 75, element 21) of head 1; the tokens of its own sixteen before it (64..74) are left out:
    # a product of tiles adds 0 * inf there
    N, t, e = 200, 75, 21
    q, k, v, gamma = _positive(N, d, seed=20 + d)
    state = torch.rand((1, 2, d, d), generator=torch.Generator().manual_seed(d)) * 0.1
    clean, s_clean = _run(B, q, k, v, gamma, state, segments)
    if where == "state":
        state[0, 1, 9, e] = INF
    else:
        {"q": q, "k": k, "v": v}[where][0, 1, t, e] = INF
    out, s = _run(B, q, k, v, gamma, state, segments)
    want, s_want = clean.copy(), s_clean.copy()
    if where == "q":
        want[0, 1, t] = INF
    elif where == "k":
        want[0, 1, t:] = INF
        s_want[0, 1, e] = INF
    elif where == "v":
        want[0, 1, t:, e] = INF
        s_want[0, 1, :, e] = INF
    else:
        want[0, 1, :, e] = INF
        s_want[0, 1, 9, e] = INF
    tokens = np.ones(N, dtype=bool)
    if where in "kv":
        tokens[64:75] = False
    for got, ref in ((out[:, :, tokens], want[:, :, tokens]), (s, s_want)):
        assert np.array_equal(np.isinf(got), np.isinf(ref)) and not np.isnan(got).any()
        assert (got[np.isinf(ref)] > 0).all()
        fin = np.isfinite(ref)
        # both results are within this of the exact ones (fp32 sums of up to 128 + 32 terms a tile)
        assert np.abs(got[fin] - ref[fin]).max() <= 4e-6 * np.abs(ref[fin]).max()


@pytest.mark.parametrize("d", [64, 128])
def test_values_next_to_the_largest_float(B, d):
    # o = (q . k) v with one-hot rows: 1 * v is v, 2 * v overflows; nothing else of the job is touched
    N, big = 70, 3.4e38
    q, k, v = torch.zeros(3, 1, 1, N, d).unbind(0)
    gamma = torch.ones(1)
    q[..., 3], k[0, 0, 20, 3], v[0, 0, 20, 5] = 1.0, 1.0, big
    q[0, 0, 40, 3] = 2.0
    out, s = _run(B, q, k, v, gamma)
    want = np.zeros((1, 1, N, d), dtype=np.float32)
    want[0, 0, 20:, 5] = big
    want[0, 0, 40, 5] = INF
    assert np.array_equal(out, want)
    want_s = np.zeros((1, 1, d, d), dtype=np.float32)
    want_s[0, 0, 3, 5] = big
    assert np.array_equal(s, want_s)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("scales", [(-60, -60, 104), (-118, 60, 50), (40, -112, 60), (60, 56, -118), (0, 0, -116)])
def test_small_operands_keep_their_bits(B, d, scales):
    # powers of two move the exponents only; the same bound as at the usual sizes.  Nothing underflows: the
    # smallest scores, states and outputs stay above 2^-126 / 2^-24 of their largest.
    q, k, v, gamma = W.make_custom_forward_inputs(1, 2, 150, d, "f32", seed=d)
    q, k, v = (t * 2.0 ** s for t, s in zip((q, k, v), scales))
    ref, s_ref = oracle.recurrent(*(W.to_f64(t) for t in (q, k, v, gamma)))
    out, s = _run(B, q, k, v, gamma)
    errs = max_rel_err(out, ref), max_rel_err(s, s_ref)
    print(f"  d {d} scales {scales}: out {errs[0]:.2e} state {errs[1]:.2e}", flush=True)
    assert max(errs) <= 2e-6


@pytest.mark.parametrize("how", ["fast decay", "one small value", "one large value"])
@pytest.mark.parametrize("N,segments", [(1, 1), (31, 1), (32, 1), (33, 1), (63, 1), (65, 2), (97, 2), (200, 4), (700, 1), (700, 0),
                                        (1100, 17), (2304, 9)])
def test_width_128_on_fp32_matrix_instructions(B, N, segments, how):
    """Every shape of the walk that width 128 falls back to: edges of the 32-token tiles, one and several segments
    (whose states the walk combines itself, or the scan), the state handed on in place."""
    gamma = torch.tensor([0.3, 0.0, 0.02]) if how == "fast decay" else torch.tensor([0.875, 0.97, 1.0])
    q, k, v, gamma = W.make_custom_forward_inputs(2, 3, N, 128, "f32", seed=3000 + N, gamma=gamma)
    state = torch.randn((2, 3, 128, 128), generator=torch.Generator().manual_seed(N)) * 0.1
    if how == "one small value":
        v[:, :, [0, N - 1], 77] = 2.0 ** -100
    elif how == "one large value":  # the sum of the outputs' magnitudes overflows, no output does
        v[:, :, N // 2, 77], k[:, :, N // 2], q[:, :, N // 2:, :] = 3e38, 0.25, 0.0
        q[:, :, N // 2:, 5], k[:, :, N // 2, 5] = 1.0, 1.0
    ref, s_ref = oracle.recurrent(*(W.to_f64(t) for t in (q, k, v, gamma)), W.to_f64(state))
    S = state.cuda()
    out = B.leet_attn_forward_v2(q.cuda(), k.cuda(), v.cuda(), gamma.cuda(), state_in=S, state_out=S, segments=segments)
    if how == "one large value":  # column 77 by itself, the others by theirs
        out, ref, S, s_ref = (np.swapaxes(np.asarray(t.cpu() if torch.is_tensor(t) else t, dtype=np.float64), 1, 3)
                              for t in (out, ref, S, s_ref))
        out, ref, S, s_ref = (t.reshape(t.shape[0], 128, -1) for t in (out, ref, S, s_ref))
        errs = max_rel_err(out, ref), max_rel_err(S, s_ref)
    else:
        errs = max_rel_err(out.cpu().numpy(), ref), max_rel_err(S.cpu().numpy(), s_ref)
    print(f"  N {N} segments {segments} {how}: out {errs[0]:.2e} state {errs[1]:.2e}", flush=True)
    assert max(errs) <= 2e-6


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("segments", [1, 5])
def test_a_state_that_decays_away(B, d, segments):
    # 200 tokens, then k = v = 0 for long: the state passes every magnitude down to zero, and rows of q that meet it
    # must give it back.  Every entry is positive, so an output errs by what its state does: one rounding (2^-24) a tile of 32
    # tokens, and half a unit of gamma^32 as it enters each of them, over 122 tiles; a few more at the end.
    N = 3900
    q, k, v, gamma = W.make_custom_forward_inputs(1, 2, N, d, "f32", seed=40 + d, gamma=torch.tensor([0.97, 0.985]))
    q, k, v = (t.abs() + 2.0 ** -10 for t in (q, k, v))
    k[:, :, 200:], v[:, :, 200:] = 0.0, 0.0
    q[:, :, 2000:2100] = 0.0
    ref, s_ref = oracle.recurrent(*(W.to_f64(t) for t in (q, k, v, gamma)))
    out, s = _run(B, q, k, v, gamma, segments=segments)
    big = ref > 2.0 ** -118
    err = np.abs(out[big] / ref[big] - 1).max()
    print(f"  d {d} segments {segments}: {err:.2e} down to {ref[big].min():.1e}", flush=True)
    assert big.mean() > 0.5 and err <= (1.5 * N / 32 + 8) * 2.0 ** -24
    assert (out[:, :, 2000:2100] == 0).all() and np.abs(out[~big] - ref[~big]).max() <= 2.0 ** -118


def test_data_out_of_range_is_found_in_the_first_tiles(B):
    # Ten tiles a sequence: walked again after the second of them a call takes 1.4 times as long as on ordinary data, after
    # the eighth 1.9 times.
    q, k, v, gamma = (t.cuda() for t in W.make_custom_forward_inputs(16, 32, 300, 128, "f32", seed=77))
    small = [t * 2.0 ** e for t, e in ((q, -60), (k, -60), (v, 104))]
    out = torch.empty_like(v)

    def us(args):
        times = []
        for _ in range(40):
            start, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            start.record()
            B.leet_attn_forward(*args, gamma, out=out)
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end) * 1e3)
        return float(np.median(times))

    us((q, k, v))
    ordinary, outside = us((q, k, v)), us(small)
    print(f"  ordinary {ordinary:.1f} us, out of range {outside:.1f} us", flush=True)
    assert outside <= 1.6 * ordinary
