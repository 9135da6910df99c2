"""The sparse product out of LDS where it can go wrong: one workgroup per row and several, both tile widths, the largest slab,
rounds beyond the first sixteen neighbours, vocabularies without pruned ids, rows at odd strides -- against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_03206_amd import synth
from parity_util import assert_close, check_verify_outputs, stochastic_topk_kernel

pytestmark = pytest.mark.gpu

SHAPES = [  # N, n, k, B, gamma
    (3840, 961, 16, 6, 3),      # tiles of 64 ids
    (4097, 2, 1, 2, 1),         # tiles of 256 ids, two kept ids
    (5000, 5000, 0, 4, 2),      # every id kept
    (9001, 2303, 33, 5, 5),     # three rounds per id, several workgroups per row
    (40000, 36003, 5, 3, 3),    # a slab that fills LDS
]


@pytest.mark.parametrize("kind", ["prob", "logit"])
@pytest.mark.parametrize("shape", SHAPES)
def test_slab_against_oracle(shape, kind):
    from paper_2506_03206_amd import rdk
    N, n, k, B, gamma = shape
    rng = np.random.default_rng(N + k)
    kept = np.sort(rng.choice(N, size=n, replace=False)).astype(np.int32)
    idx, w, sw = stochastic_topk_kernel(rng, N, kept, k)
    idx, w, sw = idx.astype(np.int32), w.astype(np.float32), sw.astype(np.float32)
    zp = (rng.normal(size=(B, N)) * 2).astype(np.float32)
    zq = (zp + rng.normal(size=(B, N)).astype(np.float32))[:, kept]
    p_in, q_in = zp, np.ascontiguousarray(zq)
    if kind == "prob":
        p_in, q_in = [oracle.probs_from(x, "logit").astype(np.float32) for x in (zp, q_in)]
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    wide = lambda a: torch.nn.functional.pad(d(a), (0, 1), value=float("nan"))[:, :-1]   # an odd row stride
    kern = rdk.rdk_build_kernel(N, d(kept), rdk.SPARSE_TOPK, k=k, sparse=(d(idx), d(w), d(sw)))
    p64 = oracle.probs_from(p_in, kind)
    q64 = oracle.probs_from(q_in, kind)
    ref_qp = oracle.redistribute_batch("sparse", q64, kept, N, sparse=(idx, w.astype(np.float64), sw.astype(np.float64)))
    qp = torch.full((B, N + 3), -1.0, device="cuda")[:, :N]
    out = rdk.rdk_redistribute_verify(kern, rdk.LINEAR_SPARSE, wide(p_in), wide(q_in), 9, 4, gamma, kind, kind, q_prime=qp)
    assert_close(qp.cpu().numpy(), ref_qp, what="q'")
    ref = oracle.verify_batch(p64, ref_qp, 9, 4, gamma=gamma)
    check_verify_outputs(out, ref, p64, ref_qp, 9, 4, gamma, kind, min_exact=0.6)
    alone = rdk.rdk_redistribute_linear(kern, rdk.LINEAR_SPARSE, d(q_in), kind)
    assert torch.equal(alone, qp)
    ids, qd = rdk.rdk_sample_draft(kern, d(q_in), 9, 4, kind)
    assert torch.equal(ids, out.draft_ids)
    assert_close(qd.cpu().numpy(), ref_qp[np.arange(B), ids.cpu().numpy()], what="q' at the draft")


@pytest.mark.parametrize("N", [32513, 65281, 65793, 131073, 163585, 164097, 262400])
def test_draws_at_the_edges_of_the_held_block_sums(N):
    """Rows whose block sums just fit, or just miss, what a lane of the finish holds in registers: the draws follow the
    prefix sums of q' and of max(0, p - q') as the two-call path writes q'."""
    from paper_2506_03206_amd import rdk
    n, B, k = 4000, 3, 4
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    kept = torch.sort(torch.randperm(N, generator=g, device="cuda")[:n]).values.to(torch.int32)
    kern = rdk.rdk_build_kernel(N, kept, rdk.SPARSE_TOPK, embeddings=torch.randn((N, 8), generator=g, device="cuda"), tau=0.1, k=k)
    p = torch.softmax(torch.randn((B, N), generator=g, device="cuda"), 1)
    q = torch.softmax(torch.randn((B, n), generator=g, device="cuda"), 1)
    qp = rdk.rdk_redistribute_linear(kern, rdk.LINEAR_SPARSE, q)
    out = rdk.rdk_redistribute_verify(kern, rdk.LINEAR_SPARSE, p, q, 11, 0, 1, "prob", "prob")
    ids, qd = rdk.rdk_sample_draft(kern, q, 11, 0)
    p64, q64 = p.double().cpu().numpy(), qp.double().cpu().numpy()
    assert torch.equal(ids, out.draft_ids)
    for b in range(B):
        u = oracle.uniforms(11, b)
        for ids_, w, x in ((out.draft_ids, q64[b], u[0]), (out.resid_ids, np.maximum(p64[b] - q64[b], 0), u[2])):
            c, j = np.cumsum(w), int(ids_[b])
            tol = 1e-6 * c[-1]                          # fp32 block sums of an fp64 search
            assert w[j] > 0 and c[j] - w[j] - tol <= x * c[-1] <= c[j] + tol


@pytest.mark.parametrize("n", [1001, 16384, 16385])
def test_finish_reads_short_bf16_rows_themselves(n):
    """Batches beyond the product out of LDS: the finish takes drafter weights from a short bf16 row or from the position-minor
    copy; the draws follow the prefix sums of q' and of max(0, p - q') as the two-call path writes q'."""
    from paper_2506_03206_amd import rdk
    N, k, gamma = n + 19003, 32, 2
    B = 66                                              # two position blocks and two rows; 66 x 4.9 MB of table
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    kept = torch.sort(torch.randperm(N, generator=g, device="cuda")[:n]).values.to(torch.int32)
    kern = rdk.rdk_build_kernel(N, kept, rdk.SPARSE_TOPK, embeddings=torch.randn((N, 8), generator=g, device="cuda"), tau=0.1, k=k)
    wide = lambda z: torch.nn.functional.pad(z.to(torch.bfloat16), (0, 1), value=float("nan"))[:, :-1]
    zp = wide(torch.randn((B, N), generator=g, device="cuda") * 2)
    zq = wide(torch.randn((B, n), generator=g, device="cuda") * 2)
    qp = rdk.rdk_redistribute_linear(kern, rdk.LINEAR_SPARSE, zq, "logit")
    out = rdk.rdk_redistribute_verify(kern, rdk.LINEAR_SPARSE, zp, zq, 11, 0, gamma, "logit", "logit")
    ids, qd = rdk.rdk_sample_draft(kern, zq, 11, 0, "logit")
    p64, q64 = torch.softmax(zp.double(), 1).cpu().numpy(), qp.double().cpu().numpy()
    assert torch.equal(ids, out.draft_ids)
    np.testing.assert_allclose(qd.cpu().numpy(), q64[np.arange(B), ids.cpu().numpy()], rtol=1e-5)
    for b in range(B):
        u = oracle.uniforms(11, b)
        for ids_, w, x in ((out.draft_ids, q64[b], u[0]), (out.resid_ids, np.maximum(p64[b] - q64[b], 0), u[2])):
            c, j = np.cumsum(w), int(ids_[b])
            tol = 1e-5 * c[-1]                          # a residual is a difference of fp32 softmax outputs
            assert w[j] > 0 and c[j] - w[j] - tol <= x * c[-1] <= c[j] + tol
