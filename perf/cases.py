"""The work that users of this library have it do, as timed cases.

A case is one call of the public binding (``paper_2501_02573_amd.binding``): a prefill of B x H
sequences of N tokens, with or without a state handed in and on, or one decode step.  The sizes
are the repository's benchmark configurations (``workloads.py``), its usage-example and
batch shapes (``latency_table.py``) and generic ragged ones.

Fields of a case: ``kind`` "prefill" | "decode"; ``B``, ``H``, ``N`` (prefill only); ``r`` (width of q
and k), ``dv`` (width of v and out); ``dtype`` of q, k, v; ``out`` "f32" | "in" (the input type);
``mask`` "decay" | "causal"; ``state`` "none" | "out" | "in_out" (prefill only); ``gamma`` (see
``workloads.make_gamma``).
"""
import math

import torch

from paper_2501_02573_amd import binding, workloads

CHUNK = 64  # the chunk size that the flop count of the chunked form is quoted at


def _prefill(name, B, H, N, r, dv, dtype, out="f32", mask="decay", state="none", gamma="pow2:5:10"):
    return {"name": name, "kind": "prefill", "B": B, "H": H, "N": N, "r": r, "dv": dv, "dtype": dtype,
            "out": out, "mask": mask, "state": state, "gamma": gamma}


def _decode(name, B, H, r, dv, dtype, mask="decay", gamma="pow2:5:10"):
    return {"name": name, "kind": "decode", "B": B, "H": H, "r": r, "dv": dv, "dtype": dtype, "mask": mask,
            "gamma": gamma}


def listed():
    c1, c2, c3, c4, c5 = (workloads.CONFIG1, workloads.CONFIG2, workloads.CONFIG3, workloads.CONFIG4,
                          workloads.CONFIG5)
    return [
        # the next token of one user: 32 heads, a state of 2 MiB; latency and host time are all of it
        _decode("decode_one_user", 1, 32, 128, 128, "bf16"),
        # the next token of a full batch: 128 MiB of state read and written
        _decode("decode_batch64", c5.B, c5.H, c5.d, c5.d, "bf16", gamma=c5.gamma_kind),
        # a small batch at rank 128, value width 256 in fp16 (the usage example's widths): 32 MiB of state
        _decode("decode_wide_value", 8, 32, 128, 256, "f16"),
        # the smallest prefill: one fp32 head of 256 tokens
        _prefill("prefill_tiny_f32", c1.B, c1.H, c1.N, c1.d, c1.d, "f32", gamma=c1.gamma_kind),
        # a small fp32 job of eight heads
        _prefill("prefill_small_f32", c2.B, c2.H, c2.N, c2.d, c2.d, "f32", gamma=c2.gamma_kind),
        # the headline shape in fp32, as a user runs it who needs fp32 throughout
        _prefill("prefill_mid_f32", c3.B, c3.H, c3.N, c3.d, c3.d, "f32", gamma=c3.gamma_kind),
        # the headline workload: a mid-sized batch of prompts in bf16
        _prefill("prefill_mid_bf16", c3.B, c3.H, c3.N, c3.d, c3.d, "bf16", gamma=c3.gamma_kind),
        # one long document
        _prefill("prefill_long_bf16", c4.B, c4.H, c4.N, c4.d, c4.d, "bf16", gamma=c4.gamma_kind),
        # the next turn of a conversation: a short ragged prompt that continues from a state and hands one on
        _prefill("prefill_turn_bf16", 1, 32, 777, 128, 128, "bf16", state="in_out"),
        # one prompt at the usage example's widths, fp16 in and out, the state kept for decoding
        _prefill("prefill_wide_value_f16", 1, 32, 2000, 128, 256, "f16", out="in", state="out"),
        # a batch of prompts at width 64 without decay (0/1 causal mask), fp16 in and out
        _prefill("prefill_causal_d64_f16", 8, 16, 4000, 64, 64, "f16", out="in", mask="causal", state="out"),
        # a few tokens at once for a batch of users (drafted tokens being checked): the state in and out is
        # nearly all of the traffic
        _prefill("few_tokens_bf16", 16, 32, 5, 128, 128, "bf16", state="in_out"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: decode steps of 1 to 64 users, prefills of 1 to 32768 tokens."""
    while True:
        r, dv = rng.choice(((64, 64), (128, 128), (128, 128), (128, 256)))
        dtype = rng.choice(("bf16", "bf16", "f16", "f32") if dv != 256 else ("bf16", "f16"))
        H = rng.choice((1, 2, 3, 4, 8, 12, 16, 24, 32, 32))
        mask = rng.choice(("decay", "decay", "decay", "causal"))
        if rng.random() < 0.25:
            case = _decode("", _log_int(rng, 1, 64), H, r, dv, dtype, mask=mask)
        else:
            out = "f32" if dtype == "f32" else rng.choice(("f32", "f32", "in"))
            case = _prefill("", _log_int(rng, 1, 16), H, _log_int(rng, 2, 32768), r, dv, dtype, out=out, mask=mask,
                            state=rng.choice(("none", "out", "in_out")))
        del case["name"]
        # no more than the largest listed case asks for: 1.34 GB, and in fp32 the headline shape's 537 MB
        if work(case)["bytes"] <= (0.53e9 if dtype == "f32" and case["kind"] == "prefill" else 1.3e9):
            return case


def _isz(dtype):
    return 4 if dtype == "f32" else 2


def work(case):
    BH, r, dv, isz = case["B"] * case["H"], case["r"], case["dv"], _isz(case["dtype"])
    if case["kind"] == "decode":
        # the state in and out, q, k, v in, fp32 out; gamma S + k v, then q S: 5 operations an entry
        return {"bytes": BH * (2 * r * dv * 4 + (2 * r + dv) * isz + dv * 4) + 4 * case["H"],
                "flops": BH * 5 * r * dv}
    osz = 4 if case["out"] == "f32" else isz
    states = {"none": 0, "out": 1, "in_out": 2}[case["state"]]
    tokens = BH * case["N"]
    # per token: q S and k v against the r x dv state, and half of a chunk's scores and their products with v
    return {"bytes": tokens * ((2 * r + dv) * isz + dv * osz) + states * BH * r * dv * 4 + 4 * case["H"],
            "flops": tokens * (4 * r * dv + min(CHUNK, case["N"]) * (r + dv))}


def tolerance(case):
    # About four times the largest differences to the same recurrence in 64 bits over the listed cases
    # and forty drawn ones: decode steps 1.1e-7 (2-norm) and 7.6e-7 (single elements); fp32 prefill,
    # 32-bit products and sums in another order, 3.2e-7 and 3.0e-6; fp16 prefill, which rounds the
    # scores, the state and the weighted values to the input type once each, 3.5e-4 and 3.0e-3; bf16,
    # with three bits fewer, 2.7e-3 and 2.4e-2.
    if case["kind"] == "decode":
        return {"rel": 5e-7, "max": 4e-6}
    if case["dtype"] == "f32":
        return {"rel": 1.5e-6, "max": 1.5e-5}
    if case["dtype"] == "f16":
        return {"rel": 1.5e-3, "max": 1.2e-2}
    return {"rel": 1e-2, "max": 9e-2}


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(seed)
    B, H, r, dv = case["B"], case["H"], case["r"], case["dv"]
    dt = workloads.torch_dtype(case["dtype"])
    lead = (B, H) if case["kind"] == "decode" else (B, H, case["N"])

    def normal(shape, sigma, dtype):
        return torch.randn(shape, device=dev, generator=gen, dtype=torch.float32).mul_(sigma).to(dtype)

    st = {"case": case,
          "q": normal(lead + (r,), r ** -0.5, dt),
          "k": normal(lead + (r,), r ** -0.5, dt),
          "v": normal(lead + (dv,), dv ** -0.5, dt),
          "gamma": workloads.make_gamma(case["gamma"], H).to(dev) if case["mask"] == "decay" else None}
    if case["kind"] == "decode" or case["state"] == "in_out":
        # the state that earlier tokens have left
        st["state"] = normal((B, H, r, dv), 0.1, torch.float32)
    if case["kind"] == "prefill" and case["state"] != "none":
        # where the state goes (apart from the entering one, which other continuations may start from)
        st["state_out"] = torch.zeros((B, H, r, dv), dtype=torch.float32, device=dev)
    return st


def run(st):
    case = st["case"]
    q, k, v, gamma = st["q"], st["k"], st["v"], st["gamma"]
    mask = binding.LEET_MASK_CAUSAL if case["mask"] == "causal" else binding.LEET_MASK_DECAY
    square = case["r"] == case["dv"]
    if case["kind"] == "decode":
        if not square:
            out = binding.leet_attn_decode_step_rd(q, k, v, gamma, st["state"], mask=mask)
        elif case["dtype"] == "bf16" and case["mask"] == "decay":
            out = binding.leet_attn_decode_step(q, k, v, gamma, st["state"])
        else:
            out = binding.leet_attn_decode_step_v2(q, k, v, gamma, st["state"], mask=mask)
        return out, st["state"]
    if square and case["out"] == "f32" and case["mask"] == "decay" and case["state"] == "none" and case["dtype"] != "f16":
        return binding.leet_attn_forward(q, k, v, gamma)
    fwd = binding.leet_attn_forward_v2 if square else binding.leet_attn_forward_rd
    out = fwd(q, k, v, gamma, state_in=st.get("state"), state_out=st.get("state_out"),
              out_dtype=q.dtype if case["out"] == "in" else torch.float32, mask=mask)
    return (out, st["state_out"]) if "state_out" in st else out
