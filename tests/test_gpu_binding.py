"""The CPython extension as the rest of a Python program sees it."""
import sys
import threading
import time

import pytest
import torch

pytestmark = pytest.mark.gpu


def call_of(name):
    """One per-step call of the extension, its tensors and workspaces made and used once."""
    from paper_2506_03206_amd import rdk
    N, n, B, C = 1300, 300, 4, 2
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    p = torch.softmax(torch.randn((B, N), generator=g, device="cuda"), 1)
    kept = torch.arange(0, 4 * n, 4, dtype=torch.int32, device="cuda")
    q = p[:, kept.long()].contiguous()
    kern = rdk.rdk_build_kernel(N, kept, rdk.IDENTITY)
    o, m = rdk.VerifyOutputs(B, N, 2, "cuda"), rdk.MultiOutputs(B, C, "cuda")
    qp = torch.empty((B, N), device="cuda")
    ids, qd = torch.empty(B, dtype=torch.int32, device="cuda"), torch.empty(B, device="cuda")
    child = torch.full((2, 2, C), -1, dtype=torch.int32, device="cuda")
    f = getattr(rdk.native(), name)
    args = {
        "redistribute_verify": (kern, rdk.LINEAR_TAYLOR, p, q, 1, 0, 2, "prob", "prob", True, o, None),
        "verify_sample": (p, p, 1, 0, 2, "prob", True, o, True),
        "redistribute_exact": (kern, q, "prob", qp),
        "redistribute_linear": (kern, rdk.LINEAR_TAYLOR, q, "prob", p, "prob", qp),
        "sample_draft": (kern, q, 1, 0, "prob", qp, ids, qd),
        "verify_multi": (p, p, C, 1, 0, "prob", True, m),
        "tree_walk": (child, m.accepted, m.token),
    }[name]
    status = f(*args)
    assert (status[0] if isinstance(status, tuple) else status) == rdk.OK
    torch.cuda.synchronize()
    return lambda: f(*args)


@pytest.mark.parametrize("name", ["redistribute_verify", "verify_sample", "redistribute_exact", "redistribute_linear", "sample_draft",
                                  "verify_multi", "tree_walk"])
def test_other_threads_run_during_a_call(name):
    """With the interpreter's own switching out of the way another thread advances only while a call gives it the lock."""
    call = call_of(name)
    ticks, stop = [0], [False]

    def tick():
        while not stop[0]:
            ticks[0] += 1
            time.sleep(0)

    interval = sys.getswitchinterval()
    sys.setswitchinterval(600.0)
    t = threading.Thread(target=tick, daemon=True)
    try:
        t.start()
        before = ticks[0]
        for _ in range(2000):
            call()
            if ticks[0] != before:
                break
        advanced = ticks[0] != before
    finally:
        stop[0] = True
        sys.setswitchinterval(interval)
    t.join(30)
    assert advanced
    torch.cuda.synchronize()


def test_out_of_memory_is_raised_as_torch_raises_it():
    """A workspace that the allocator refuses (a limit set for this process; nothing is launched)."""
    from paper_2506_03206_amd import rdk
    N, n, B = 40000, 16000, 1 << 14
    kept = torch.arange(n, dtype=torch.int32, device="cuda")
    kern = rdk.rdk_build_kernel(N, kept, rdk.SPARSE_TOPK, k=0, embeddings=torch.ones((N, 4), device="cuda"))
    q = torch.ones((1, n), device="cuda").expand(B, n)          # the workspace is asked for before the stride is looked at
    out = torch.ones((1, N), device="cuda")
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    try:
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (64 << 20)) / total)
        with pytest.raises(torch.OutOfMemoryError):
            rdk.rdk_redistribute_linear(kern, rdk.LINEAR_SPARSE, q, out=out)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    with pytest.raises(rdk.RdkError):
        rdk.rdk_redistribute_linear(kern, rdk.LINEAR_SPARSE, q, out=out)
