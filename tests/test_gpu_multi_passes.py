"""The passes of a position that rejects several candidates: the blocks that the wavefronts keep (fewer blocks than wavefronts, as
many, one more) and the others in both directions, ends inside a block, rows at odd strides -- against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from parity_util import check_multi

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["prob", "logit"])
@pytest.mark.parametrize("N", [9, 1024, 15 * 1024 + 1, 16 * 1024, 16 * 1024 + 3, 35 * 1024 - 1])
def test_passes_of_several_rejections(N, kind):
    from paper_2506_03206_amd import rdk
    B, C, seed, offset = 6, 5, 12, 3
    rng = np.random.default_rng(N)
    z = (rng.normal(size=(B, N)) * 2).astype(np.float32)
    p64 = oracle.probs_from(z, "logit")
    p32 = p64.astype(np.float32)
    qp32 = oracle.probs_from(z + rng.normal(size=(B, N)) * 1.5, "logit").astype(np.float32)
    p64 = p32.astype(np.float64) if kind == "prob" else p64
    q64 = qp32.astype(np.float64)
    cand = np.full((B, C), N + 7, np.int32)            # never kept: every round a pass
    cand[1, 2] = int(np.argmax(p32[1]))                # rounds, and a candidate that may be kept
    cand[2, 3:] = -1                                   # a list that ends
    ref = oracle.verify_multi_batch(p64, q64, C, seed, offset, cand_ids=cand)
    wide = lambda a: torch.nn.functional.pad(torch.from_numpy(np.ascontiguousarray(a)).cuda(), (0, 1), value=float("nan"))[:, :-1]
    o = rdk.rdk_verify_multi(wide(p32 if kind == "prob" else z), wide(qp32), C, seed, offset, kind,
                             cand_ids=torch.from_numpy(cand).cuda())
    check_multi(o, ref, p64, q64, seed, offset, C, min_exact=0.8)
    even = rdk.rdk_verify_multi(torch.from_numpy(p32 if kind == "prob" else z).cuda(), torch.from_numpy(qp32).cuda(), C, seed, offset,
                                kind, cand_ids=torch.from_numpy(cand).cuda())
    check_multi(even, ref, p64, q64, seed, offset, C, min_exact=0.8)


# Long rows: a launch a round up to 256 positions, one block a wavefront up to 32, two beyond.  Ends inside a block, the fewest ids for
# one and for four candidates, one block in the last workgroup.
@pytest.mark.parametrize("kind", ["prob", "logit"])
@pytest.mark.parametrize("N,C", [(40000, 1), (60001, 2), (99999, 3), (100000, 4), (127 * 1024 + 1, 4)])
def test_a_launch_a_round(N, C, kind):
    from paper_2506_03206_amd import rdk
    B, seed, offset = 257, 5, 9
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N + C)
    z = torch.randn((B, N), generator=gen, device="cuda").mul_(2)
    qp = torch.softmax(z + torch.randn((B, N), generator=gen, device="cuda"), 1)
    p = torch.softmax(z, 1) if kind == "prob" else z
    cand = np.full((B, C), N + 7, np.int32)            # never kept: every round a pass
    best = torch.softmax(z, 1).argmax(1).cpu().numpy()
    cand[1::4, C - 1] = best[1::4]                     # rounds, and a candidate that may be kept
    cand[2::4, C // 2:] = -1                           # a list that ends, from the start for C = 1
    cand[3::4, 0] = best[3::4]
    cand[4] = -1                                       # a leaf
    cd = torch.from_numpy(cand).cuda()
    whole = rdk.rdk_verify_multi(p, qp, C, seed, offset, kind, cand_ids=cd)          # a workgroup a position
    for m in (32, 33, 128, 129, 256):
        part = rdk.rdk_verify_multi(p[:m], qp[:m], C, seed, offset, kind, cand_ids=cd[:m].contiguous())
        assert torch.equal(whole.accepted[:m], part.accepted) and torch.equal(whole.token[:m], part.token)
        # the same blocks in the same order, but for the statistics of logit rows, which are cut by the size of the batch
        torch.testing.assert_close(part.resid_mass, whole.resid_mass[:m], rtol=0 if kind == "prob" else 1e-5, atol=0)
    n = 6
    p64 = p[:n].cpu().numpy().astype(np.float64) if kind == "prob" else oracle.probs_from(z[:n].cpu().numpy(), "logit")
    q64 = qp[:n].cpu().numpy().astype(np.float64)
    ref = oracle.verify_multi_batch(p64, q64, C, seed, offset, cand_ids=cand[:n])
    few = rdk.rdk_verify_multi(p[:n], qp[:n], C, seed, offset, kind, cand_ids=cd[:n].contiguous())
    check_multi(few, ref, p64, q64, seed, offset, C, min_exact=0.8)


def test_rounds_in_a_graph():
    """Replays on other candidates, with eager calls between them, against the eager call."""
    from paper_2506_03206_amd import rdk
    N, C, B = 60001, 2, 40
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    z = torch.randn((B, N), generator=gen, device="cuda").mul_(2)
    p, qp = torch.softmax(z, 1), torch.softmax(z + torch.randn((B, N), generator=gen, device="cuda"), 1)
    cand = torch.randint(0, N, (B, C), generator=gen, device="cuda", dtype=torch.int32)
    o = rdk.MultiOutputs(B, C, "cuda")
    rdk.rdk_verify_multi(p, qp, C, 5, 9, cand_ids=cand, outputs=o)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rdk.rdk_verify_multi(p, qp, C, 5, 9, cand_ids=cand, outputs=o)
    for rep in range(3):
        cand.copy_(torch.topk(qp, C + rep, dim=1).indices[:, rep:].int())
        cand[rep::5, 1:] = -1
        cand[rep + 1::7] = -1
        o.token.fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        ref = rdk.rdk_verify_multi(p, qp, C, 5, 9, cand_ids=cand)
        for name in ("accepted", "token", "resid_mass"):
            assert torch.equal(getattr(o, name), getattr(ref, name)), name


@pytest.mark.parametrize("kind", ["prob", "logit"])
def test_least_workspace_gives_the_same_results(kind):
    """A shape that goes a launch a round, with the workspace for that and with the least that the call accepts."""
    import ctypes
    from paper_2506_03206_amd import rdk
    B, N, C, seed, offset = 6, 70001, 2, 11, 2
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    z = torch.randn((B, N), generator=gen, device="cuda").mul_(2)
    qp = torch.softmax(z + torch.randn((B, N), generator=gen, device="cuda"), 1)
    p = torch.softmax(z, 1) if kind == "prob" else z
    cand = torch.topk(qp, C, dim=1).indices.int()
    cand[1], cand[2, 1:], cand[3] = N, -1, -1
    full = rdk.rdk_verify_multi(p, qp, C, seed, offset, kind, cand_ids=cand)
    o = rdk.MultiOutputs(B, C, "cuda")
    o.cand_ids.copy_(cand)
    code = rdk.PROB_F32 if kind == "prob" else rdk.LOGIT_F32
    d = rdk.MultiDesc(B=B, N=N, C=C, seed=seed, offset=offset, sample_candidates=1)
    asked, least = ctypes.c_size_t(), ctypes.c_size_t()
    assert rdk.lib().rdk_verify_multi_workspace_bytes(ctypes.byref(d), code, ctypes.byref(least)) == rdk.OK   # no rounds where they are drawn
    d.sample_candidates = 0
    assert rdk.lib().rdk_verify_multi_workspace_bytes(ctypes.byref(d), code, ctypes.byref(asked)) == rdk.OK
    assert least.value < asked.value
    ws = torch.empty(asked.value, dtype=torch.uint8, device="cuda")
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())
    call = lambda size: rdk.lib().rdk_verify_multi(ctypes.byref(d), ptr(p), code, N, ptr(qp), N, ptr(o.cand_ids), ptr(o.accepted), ptr(o.token),
                                                   ptr(o.resid_mass), ptr(ws), size, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    slack = 256                                        # which the query adds and the call does not need
    assert call(least.value - slack - 1) == 6          # RDK_ERR_WORKSPACE
    for size, kernel in ((least.value - slack, "verify_multi_kernel"), (asked.value - slack - 1, "verify_multi_kernel"),
                         (asked.value - slack, "verify_multi_round_kernel")):
        for t in (o.accepted, o.token, o.resid_mass):
            t.fill_(-7)
        rdk.rdk_timing_select(kernel)
        assert call(size) == rdk.OK
        torch.cuda.synchronize()
        rdk.rdk_timing_select(None)
        assert rdk.rdk_timing_read(kernel)[0] == (1 if kernel == "verify_multi_kernel" else C + 1)
        assert torch.equal(o.accepted, full.accepted) and torch.equal(o.token, full.token) and torch.equal(o.resid_mass, full.resid_mass)
