"""Calls of several shapes from several threads and streams, and across changes of the process-wide kernel choice: a
thread keeps the plan of its last call, which must serve that call's shape and choice only."""
import threading

import pytest
import torch

from paper_2501_02573_amd import workloads as W

pytestmark = pytest.mark.gpu

# (B, H, N, r, dv, dtype): one and several segments, every kernel
JOBS = [(1, 4, 300, 64, 64, "f32"), (1, 4, 700, 128, 128, "f32"), (1, 2, 4100, 128, 128, "bf16"), (1, 2, 4100, 64, 64, "f16"),
        (1, 2, 1000, 128, 256, "f16"), (2, 2, 4100, 128, 128, "bf16")]


@pytest.fixture(scope="module")
def B():
    from paper_2501_02573_amd import binding
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return binding


def _inputs(job, seed):
    b, h, N, r, dv, dtype = job
    return [t.cuda() for t in W.make_rd_forward_inputs(b, h, N, r, dv, dtype, seed=seed)]


def _workspace(B, job, kernel=-1):
    b, h, N, r, dv, dtype = job
    code = {"f32": B.LEET_F32, "bf16": B.LEET_BF16, "f16": B.LEET_F16}[dtype]
    return torch.empty(max(B.workspace_bytes_v3(b, h, N, r, dv, code, 0, kernel), 256), dtype=torch.uint8, device="cuda")


def test_threads_with_streams_of_their_own(B):
    want = {job: B.leet_attn_forward_v3(*_inputs(job, seed=1)) for job in JOBS}
    torch.cuda.synchronize()
    failures = []

    def work(first):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                jobs = [JOBS[(first + i) % len(JOBS)] for i in range(len(JOBS))]
                mine = {job: (_inputs(job, seed=1), _workspace(B, job)) for job in jobs}
                for repeat in range(3):
                    for job in jobs:
                        x, ws = mine[job]
                        for _ in range(repeat + 1):  # the same shape again, and another one next
                            out = B.leet_attn_forward_v3(*x, workspace=ws)
                        stream.synchronize()
                        if not torch.equal(out, want[job]):
                            failures.append((first, job))
        except Exception as e:  # a thread's exception would be lost
            failures.append((first, repr(e)))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failures, failures


@pytest.mark.parametrize("job", JOBS[2:])
def test_kernel_choice_between_calls_of_one_shape(B, job):
    x = _inputs(job, seed=2)
    choices = (B.KERNEL_WIDE, B.KERNEL_COLUMN_SPLIT, B.KERNEL_AUTO)
    want = {c: B.leet_attn_forward_v3(*x, kernel=c) for c in choices}
    before = B.get_bf16_kernel()
    try:
        for c in choices + choices[::-1]:
            B.set_bf16_kernel(c)
            for _ in range(2):  # with just the workspace that this choice asks for
                assert torch.equal(B.leet_attn_forward_rd(*x, workspace=_workspace(B, job)), want[c]), c
            other = choices[(c + 1) % 3]
            assert torch.equal(B.leet_attn_forward_v3(*x, workspace=_workspace(B, job, other), kernel=other), want[other])
    finally:
        B.set_bf16_kernel(before)
