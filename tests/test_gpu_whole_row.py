"""Eq. 3 with q' written by one workgroup per row where it can go wrong: ends inside a quad and on a chunk, a second chunk for one
wavefront and for all, the last quads of the drafter row, chunks without kept ids and with nothing but, rows at odd strides, both
sides of the lines to the two passes -- against the oracle, and the fused call against the one that only writes."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_03206_amd import synth
from parity_util import check_verify_outputs

pytestmark = pytest.mark.gpu

SHAPES = [  # N, n, B, gamma, which ids are kept, one launch
    (4, 4, 2, 1, "any", True),
    (5, 3, 2, 1, "any", False),              # a drafter row without a whole quad
    (1023, 5, 3, 3, "tail", True),
    (1025, 1024, 3, 3, "first", True),       # every id of the first chunk, none of the second
    (3001, 2999, 260, 4, "any", True),
    (16 * 1024, 4001, 4, 2, "any", True),
    (16 * 1024 + 1, 5003, 4, 2, "tail", True),
    (24 * 1024, 6001, 63, 1, "any", True),
    (24 * 1024 + 1, 6001, 63, 1, "any", False),
    (24 * 1024 + 1, 6002, 64, 4, "tail", True),
    (32 * 1024, 9001, 64, 2, "any", True),
    (32 * 1024 + 1, 9001, 64, 2, "any", False),
    (700, 130, 1024, 4, "any", True),
    (700, 130, 1025, 5, "any", True),        # beyond one row for every place on the chip
    (700, 130, 2049, 3, "any", False),
    (2048, 500, 2049, 3, "any", True),
]


@pytest.mark.parametrize("kinds", ["prob prob", "logit logit", "bf16 bf16", "prob bf16", "bf16 prob"])
@pytest.mark.parametrize("shape", SHAPES)
def test_rows_written_in_one_launch(shape, kinds):
    from paper_2506_03206_amd import rdk
    N, n, B, gamma, where, one = shape
    rng = np.random.default_rng(N + n)
    if where == "first":
        kept = np.arange(n)
    elif where == "tail":                    # runs that end with the drafter row, one slot and two in the last quads
        kept = np.concatenate([np.sort(rng.choice(N - 8, size=n - 3, replace=False)), [N - 6, N - 2, N - 1]])
    else:
        kept = np.sort(rng.choice(N, size=n, replace=False))
    kept = kept.astype(np.int32)
    zp = (rng.normal(size=(B, N)) * 2).astype(np.float32)
    zq = (zp + rng.normal(size=(B, N)).astype(np.float32))[:, kept]
    if N > 3072:
        zp[0, 1024:2048] = -np.inf           # a chunk of masked ids
    zp[1, : N // 2] = np.finfo(np.float32).min
    rows, p64, dev = [], [], []
    for z, kind in zip((zp, zq), kinds.split()):
        if kind == "bf16":
            z = synth.bf16_round(np.maximum(z, -1e38))
        if kind == "prob":
            z = oracle.probs_from(z, "logit").astype(np.float32)
        rows.append("prob" if kind == "prob" else "logit")
        p64.append(oracle.probs_from(z, rows[-1]))
        t = torch.from_numpy(np.ascontiguousarray(z)).cuda().to(torch.bfloat16 if kind == "bf16" else torch.float32)
        dev.append(torch.nn.functional.pad(t, (0, 1), value=float("nan"))[:, :-1])
    kern = rdk.rdk_build_kernel(N, torch.from_numpy(kept).cuda(), rdk.IDENTITY)
    held = torch.full((B, N + 3), 7.0, device="cuda")
    rdk.rdk_timing_select("*")
    rdk.rdk_redistribute_linear(kern, rdk.LINEAR_TAYLOR, dev[1], rows[1], p=dev[0], p_kind=rows[0], out=held[:, :N])
    torch.cuda.synchronize()
    rdk.rdk_timing_select(None)
    launches = {name: rdk.rdk_timing_read(name)[0] for name in ("taylor_whole_kernel", "taylor_stats_kernel", "taylor_write_kernel", "row_stats_kernel")}
    assert launches["taylor_whole_kernel"] == (1 if one else 0) and launches["taylor_stats_kernel"] == (0 if one else 1)
    assert not one or launches["row_stats_kernel"] == 0
    assert bool((held[:, N:] == 7.0).all())  # nothing behind a row is written
    got = held[:, :N].cpu().numpy().astype(np.float64)
    ref = oracle.redistribute_batch("taylor", p64[1], kept, N, p=p64[0])
    # fp32 terms and sums of at most 2**15 terms in a tree; a softmax term carries its logit's rounding (2**-24 of a difference of 15)
    assert (np.abs(got - ref) <= 1e-5 * np.abs(ref) + 1e-7).all()
    qp = torch.empty((B, N), device="cuda")
    out = rdk.rdk_redistribute_verify(kern, rdk.LINEAR_TAYLOR, dev[0], dev[1], 9, 4, gamma, rows[0], rows[1], q_prime=qp)
    assert torch.equal(qp, held[:, :N])      # the same bits in both calls
    want = oracle.verify_batch(p64[0], ref, 9, 4, gamma=gamma)
    check_verify_outputs(out, want, p64[0], ref, 9, 4, gamma, rows[0], min_exact=0.6)


# The fused call without q': both sides of the lines to the kernel that keeps the kept values in LDS (the shapes that a kernel of one
# launch for probabilities and for logits takes are named).
WHOLE, ROW = "taylor_whole_kernel", "taylor_row_kernel"


@pytest.mark.parametrize("kind", ["prob", "logit", "bf16"])
@pytest.mark.parametrize("N,n,B,gamma,takes", [
    (1001, 1000, 5, 1, (WHOLE, WHOLE)), (1023, 131, 1026, 3, (WHOLE, WHOLE)), (1025, 131, 1026, 3, (WHOLE, WHOLE)),
    (4096, 900, 257, 1, (WHOLE, WHOLE)), (4097, 900, 257, 1, (WHOLE, WHOLE)), (8192, 2000, 256, 4, (WHOLE, WHOLE)),
    (8193, 2000, 6, 3, (WHOLE, WHOLE)), (8192, 2000, 513, 3, (WHOLE, ROW)), (8193, 2000, 257, 1, (ROW, ROW)),
    (12288, 3000, 5, 1, (WHOLE, WHOLE)), (12289, 3000, 256, 2, (WHOLE, ROW)), (32768, 8000, 3, 3, (WHOLE, ROW)),
    (600, 200, 1024, 4, (WHOLE, WHOLE)), (3001, 700, 1026, 2, (WHOLE, WHOLE))])
def test_rows_finished_in_one_launch(N, n, B, gamma, takes, kind):
    from paper_2506_03206_amd import rdk
    rng = np.random.default_rng(N + B)
    kept = np.sort(rng.choice(N, size=n, replace=False)).astype(np.int32)
    zp = (rng.normal(size=(B, N)) * 2).astype(np.float32)
    zq = np.ascontiguousarray((zp + rng.normal(size=(B, N)).astype(np.float32))[:, kept])
    zp[0, : N // 2], zp[1], zq[2] = -np.inf, 1.5, -2.0             # masked ids, uniform rows
    if kind == "bf16":
        zp, zq = synth.bf16_round(zp), synth.bf16_round(zq)
    pk = "prob" if kind == "prob" else "logit"
    if kind == "prob":
        zp, zq = [oracle.probs_from(x, "logit").astype(np.float32) for x in (zp, zq)]
    dt = torch.bfloat16 if kind == "bf16" else torch.float32
    wide = lambda a: torch.nn.functional.pad(torch.from_numpy(np.ascontiguousarray(a)).cuda().to(dt), (0, 1), value=float("nan"))[:, :-1]
    kern = rdk.rdk_build_kernel(N, torch.from_numpy(kept).cuda(), rdk.IDENTITY)
    p64, q64 = oracle.probs_from(zp, pk), oracle.probs_from(zq, pk)
    ref = oracle.redistribute_batch("taylor", q64, kept, N, p=p64)
    want = oracle.verify_batch(p64, ref, 9, 4, gamma=gamma)
    rdk.rdk_timing_select(takes[kind != "prob"])
    for _ in range(2):                       # the records of the scan are as they were after a call
        out = rdk.rdk_redistribute_verify(kern, rdk.LINEAR_TAYLOR, wide(zp), wide(zq), 9, 4, gamma, pk, pk)
        check_verify_outputs(out, want, p64, ref, 9, 4, gamma, pk, min_exact=0.6)
    rdk.rdk_timing_select(None)
    assert rdk.rdk_timing_read(takes[kind != "prob"])[0] == 2


# Rows by one workgroup, and (probabilities, or q' written; the last also for logits) in two passes.
@pytest.mark.parametrize("N", [3000, 8000, 40000, 60000])
@pytest.mark.parametrize("keep", [False, True])
def test_rows_without_mass_and_with_nan(N, keep):
    """A drafter row of masked ids (or of zeros) drafts nothing and leaves the whole target row; NaN stays visible, whether q' is
    written or not."""
    from paper_2506_03206_amd import rdk
    kern = rdk.rdk_build_kernel(N, torch.arange(0, N, 4, dtype=torch.int32, device="cuda"), rdk.IDENTITY)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N)
    z = torch.randn((6, N), generator=gen, device="cuda")
    for kind in ("logit", "prob"):
        p, q = (z, z[:, ::4]) if kind == "logit" else (torch.softmax(z, 1), torch.softmax(z, 1)[:, ::4])
        p, q = p.clone(), q.clone().contiguous()
        q[1] = -float("inf") if kind == "logit" else 0.0
        p[2, 7] = float("nan")
        q[3, 5] = float("nan")
        p[4, 9] = float("inf")
        qp = torch.empty((6, N), device="cuda") if keep else None
        o = rdk.rdk_redistribute_verify(kern, rdk.LINEAR_TAYLOR, p, q, 3, 0, 3, kind, kind, q_prime=qp)
        assert int(o.draft_ids[1]) == -1 and float(o.alpha[1]) == 0.0 and int(o.resid_ids[1]) >= 0
        assert abs(float(o.resid_mass[1]) - 1.0) < 1e-5        # fp32 sum of a row that adds up to one
        assert (o.draft_ids[2:5] == -1).all() and (o.draft_ids[[0, 5]] >= 0).all()
        if keep:
            assert not qp[1].any() and qp[2:5].isnan().any(1).all()
        assert o.alpha[2:5].isnan().all() and o.resid_mass[2:5].isnan().all() and (o.resid_ids[2:5] == -1).all()


@pytest.mark.parametrize("N,B,keep", [(3000, 20, False), (3000, 20, True), (20001, 640, True), (8000, 512, False), (3000, 1100, False), (3000, 1100, True)])
def test_graph_replays_of_rows_in_one_launch(N, B, keep):
    """Replays on other rows, with eager calls between them, against the eager call; every sequence is scanned."""
    from paper_2506_03206_amd import rdk
    kern = rdk.rdk_build_kernel(N, torch.arange(1, N, 3, dtype=torch.int32, device="cuda"), rdk.IDENTITY)
    gamma = 4

    def rows(seed):
        gen = torch.Generator(device="cuda")
        gen.manual_seed(seed)
        z = torch.randn((B, N), generator=gen, device="cuda")
        return torch.softmax(2 * z, 1), torch.softmax(2 * z + torch.randn((B, N), generator=gen, device="cuda"), 1)[:, 1::3].contiguous()
    p, q = rows(0)
    o, qp = rdk.VerifyOutputs(B, N, gamma, "cuda"), torch.empty((B, N), device="cuda") if keep else None
    call = lambda out, held: rdk.rdk_redistribute_verify(kern, rdk.LINEAR_TAYLOR, p, q, 5, 0, gamma, q_prime=held, outputs=out)
    call(o, qp)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(o, qp)
    for rep in range(3):
        p2, q2 = rows(10 + rep)
        p.copy_(p2)
        q.copy_(q2)
        o.n_accepted.fill_(-7)
        o.out_tokens.fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        ref, held = rdk.VerifyOutputs(B, N, gamma, "cuda"), torch.empty((B, N), device="cuda") if keep else None
        call(ref, held)
        for name in ("draft_ids", "accept", "alpha", "resid_mass", "resid_ids", "n_accepted", "out_tokens"):
            assert torch.equal(getattr(o, name), getattr(ref, name)), name
        assert (o.n_accepted >= 0).all() and (not keep or torch.equal(qp, held))


@pytest.mark.parametrize("N", [4000, 8003])
def test_rounding_that_the_ids_of_a_row_share(N):
    """Errors of the normaliser, of its reciprocal and of the factor between a wavefront's weights and the row's move every id of a row
    alike, and alpha and the residual mass with them.  Their mean relative error over 512 rows of logits is 3.9e-8 to 4.4e-8 where these
    are carried along and 5.4e-8 to 5.8e-8 where they are rounded; a mean over 1024 values of that spread is good to 2e-9."""
    from paper_2506_03206_amd import rdk
    rng = np.random.default_rng(N)
    B, n = 512, N // 4
    kept = np.sort(rng.choice(N, size=n, replace=False)).astype(np.int32)
    zp = (rng.normal(size=(B, N)) * 2.0 - np.log1p(rng.permutation(N))).astype(np.float32)
    zq = np.ascontiguousarray((zp + rng.normal(size=(B, N)).astype(np.float32))[:, kept])
    kern = rdk.rdk_build_kernel(N, torch.from_numpy(kept).cuda(), rdk.IDENTITY)
    p, q = oracle.probs_from(zp, "logit"), np.zeros((B, N))
    q[:, kept] = oracle.probs_from(zq, "logit")
    pt = (N * q + (p * q).sum(1, keepdims=True) * p) / (N + p)
    qp = pt / pt.sum(1, keepdims=True)
    o = rdk.rdk_redistribute_verify(kern, rdk.LINEAR_TAYLOR, torch.from_numpy(zp).cuda(), torch.from_numpy(zq).cuda(), 3, 0, 0, "logit", "logit")
    alpha, resid = np.minimum(p, qp).sum(1), np.maximum(p - qp, 0).sum(1)
    off = lambda got, ref: np.abs(got.cpu().numpy().astype(np.float64) / ref - 1).mean()
    assert (off(o.alpha, alpha) + off(o.resid_mass, resid)) / 2 < 4.9e-8
