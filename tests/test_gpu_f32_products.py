"""One product at a time through the fp32 kernel: with one-hot q and k nothing averages out, so an
output shows how exact the products are that the kernel builds from 16-bit terms."""
import numpy as np
import pytest
import torch

from paper_2501_02573_amd import workloads as W

pytestmark = pytest.mark.gpu

ULP = 2.0 ** -24  # relative rounding error of fp32


@pytest.fixture(scope="module")
def B():
    from paper_2501_02573_amd import binding
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return binding


def _one_hot(shape, gen):
    """Rows with one entry of magnitude 1..2 (the sizes at which a relative error is largest)."""
    x = torch.zeros(shape, dtype=torch.float32)
    idx = torch.randint(shape[-1], shape[:-1] + (1,), generator=gen)
    val = (1 + torch.rand(shape[:-1] + (1,), generator=gen)) * (torch.randint(0, 2, shape[:-1] + (1,), generator=gen) * 2 - 1)
    return x.scatter_(-1, idx, val), idx


def _dense(shape, gen):
    return (1 + torch.rand(shape, generator=gen)) * (torch.randint(0, 2, shape, generator=gen) * 2 - 1)


def _worst(got, ref):
    got = got.cpu().numpy().astype(np.float64)
    nz = ref != 0
    assert np.array_equal(got[~nz], ref[~nz])
    return float(np.abs(got[nz] / ref[nz] - 1).max())


@pytest.mark.parametrize("d", [64, 128])
def test_single_products_are_rounded_like_fp32_products(B, d):
    # 2048 heads of one token: S' = k^T v is one product; o = (q . k) v two, q S' none more (chunked form);
    # with an entering state and k = 0, o = q S is one.  A product of exact three-term operands, summed as
    # leading term plus lower terms, is rounded once at full size; the sums of the lower terms round at
    # 2^-6 of it, seven times.  One part in six more than the roundings at full size covers those.
    gen = torch.Generator().manual_seed(5 + d)
    shape = (64, 32, 1, d)
    v = _dense(shape, gen)
    q, iq = _one_hot(shape, gen)
    k = torch.zeros(shape).scatter_(-1, iq, _dense(shape[:-1] + (1,), gen))  # the same index as q
    s_out = torch.empty((64, 32, d, d), device="cuda")
    out = B.leet_attn_forward_v2(q.cuda(), k.cuda(), v.cuda(), None, state_out=s_out, mask=B.LEET_MASK_CAUSAL)
    q64, k64, v64 = (W.to_f64(t) for t in (q, k, v))
    errs = {"(q k) v": (_worst(out, (q64 * k64).sum(-1, keepdims=True) * v64), 2),
            "k^T v": (_worst(s_out, np.swapaxes(k64, 2, 3) * v64), 1)}
    S = _dense((64, 32, d, d), gen)
    out = B.leet_attn_forward_v2(q.cuda(), torch.zeros_like(k).cuda(), v.cuda(), None, state_in=S.cuda(),
                                 mask=B.LEET_MASK_CAUSAL)
    errs["q S"] = _worst(out, np.matmul(q64, W.to_f64(S))), 1
    print("  " + ", ".join(f"{n}: {e:.3e} of {m * ULP:.3e}" for n, (e, m) in errs.items()), flush=True)
    for name, (e, m) in errs.items():
        assert e <= m * ULP * 7 / 6, name
