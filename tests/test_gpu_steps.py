"""The sparse product several positions at a time out of LDS (larger batches, drafter rows of up to 20320 slots) where it can go
wrong: batches that are no multiple of the positions held together, the edges of the row lengths at which their number changes,
neighbour counts around the eight entries of a unit, stretches of kept ids, the last row of ids, rows at odd strides."""
import numpy as np
import pytest
import torch

import oracle
from parity_util import assert_close, check_verify_outputs, stochastic_topk_kernel

pytestmark = pytest.mark.gpu

TABLE_MB = 290          # beyond the rule that takes the call to this form, whatever the shape


def batch_for(N, n, k, gamma, extra):
    """The smallest batch of whole sequences whose table reads exceed the line, and a few sequences more."""
    per = (N - n) * ((k + 15) // 16 * 16) * 8
    return ((TABLE_MB << 20) // per // gamma + 1 + extra) * gamma


SHAPES = [  # N, n, k, gamma, additional sequences, kept ids
    (4102, 1021, 16, 3, 0, "spread"),
    (4096, 64, 1, 1, 1, "spread"),
    (5003, 1500, 9, 1, 2, "first"),        # whole rows of kept ids before the first pruned one
    (9001, 2303, 33, 5, 0, "spread"),      # five units per id
    (6000, 4, 4, 1, 0, "spread"),          # the shortest row
    (12000, 10144, 16, 1, 1, "spread"),    # four positions together at most
    (12000, 10145, 8, 1, 0, "spread"),     # two
    (30000, 20288, 64, 1, 0, "last"),      # a row that ends with a round of banks
    (30000, 20289, 16, 1, 0, "spread"),    # one slot in the last round of banks
    (30000, 20320, 64, 1, 0, "last"),      # the longest row, the most neighbours
    (30000, 20321, 16, 1, 0, "spread"),    # one slot too many: no table, one of the other forms
]


@pytest.mark.parametrize("kind", ["prob", "logit"])
@pytest.mark.parametrize("shape", SHAPES)
def test_steps_against_oracle(shape, kind):
    from paper_2506_03206_amd import rdk
    N, n, k, gamma, extra, where = shape
    B = batch_for(N, n, k, gamma, extra)
    rng = np.random.default_rng(N + n + k)
    kept = {"spread": lambda: np.sort(rng.choice(N, size=n, replace=False)), "first": lambda: np.arange(n),
            "last": lambda: np.arange(N - n, N)}[where]().astype(np.int32)
    idx, w, sw = stochastic_topk_kernel(rng, N, kept, k)
    idx, w, sw = idx.astype(np.int32), w.astype(np.float32), sw.astype(np.float32)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    kern = rdk.rdk_build_kernel(N, d(kept), rdk.SPARSE_TOPK, k=k, sparse=(d(idx), d(w), d(sw)))
    # a kernel that has this form holds its table beside the pairs
    table, pairs = 48 * ((N + 255) // 256 * 256) * ((k + 7) // 8 + 0.5), (N - n) * ((k + 15) // 16 * 16) * 8
    assert (kern.storage.numel() > pairs + table) == (n <= 20320)
    g = torch.Generator(device="cuda")
    g.manual_seed(N)
    wide = lambda x: torch.nn.functional.pad(x, (0, 1), value=float("nan"))[:, :-1]   # an odd row stride
    z = torch.randn((B, N), generator=g, device="cuda") * 2
    zq = (z + torch.randn((B, N), generator=g, device="cuda"))[:, d(kept).long()]
    if kind == "prob":
        p_in, q_in = wide(torch.softmax(z, 1)), wide(torch.softmax(zq, 1) * 0.7)
    else:
        p_in, q_in = wide(z.to(torch.bfloat16)), wide(zq.to(torch.bfloat16))
    del z, zq
    qp = torch.full((B, N + 3), -1.0, device="cuda")[:, :N]
    out = rdk.rdk_redistribute_verify(kern, rdk.LINEAR_SPARSE, p_in, q_in, 9, 4, gamma, kind, kind, q_prime=qp)
    # the first and the last sequences against the oracle
    rows = np.r_[0:gamma, B - gamma:B] if B > gamma else np.arange(B)
    t = torch.from_numpy(rows).cuda()
    p64 = oracle.probs_from(p_in[t].float().cpu().numpy(), kind)
    q64 = oracle.probs_from(q_in[t].float().cpu().numpy(), kind)
    ref_qp = oracle.redistribute_batch("sparse", q64, kept, N, sparse=(idx, w.astype(np.float64), sw.astype(np.float64)))
    assert_close(qp[t].cpu().numpy(), ref_qp, what="q'")
    for lo, first in ((0, 0), (gamma, B - gamma))[:1 if B == gamma else 2]:
        part = slice(lo, lo + gamma)
        ref = oracle.verify_batch(p64[part], ref_qp[part], 9, 4 + first, gamma=gamma)
        got = rdk.VerifyOutputs(gamma, N, gamma, torch.device("cuda"))
        for name in ("draft_ids", "accept", "alpha", "resid_mass", "resid_ids"):
            setattr(got, name, getattr(out, name)[first:first + gamma])
        s = first // gamma
        got.n_accepted, got.out_tokens = out.n_accepted[s:s + 1], out.out_tokens[s:s + 1]
        check_verify_outputs(got, ref, p64[part], ref_qp[part], 9, 4 + first, gamma, kind, min_exact=0.6)
    # the whole batch against the same positions a few at a time, which take the other forms
    for b in range(0, B, max(1, B // 7)):
        few = rdk.rdk_redistribute_linear(kern, rdk.LINEAR_SPARSE, q_in[b:b + 1].clone(), kind)
        assert_close(qp[b:b + 1].cpu().numpy(), few.cpu().numpy(), what="q' of position %d" % b)
    # the other calls on the same batch: the same q', the same drafts
    assert torch.equal(rdk.rdk_redistribute_linear(kern, rdk.LINEAR_SPARSE, q_in, kind), qp)
    ids, qd = rdk.rdk_sample_draft(kern, q_in, 9, 4, kind)
    assert torch.equal(ids, out.draft_ids)
    assert_close(qd[t].cpu().numpy(), ref_qp[np.arange(len(rows)), ids[t].cpu().numpy()], what="q' at the draft")
    again = rdk.rdk_redistribute_verify(kern, rdk.LINEAR_SPARSE, p_in, q_in, 9, 4, gamma, kind, kind)
    for name in ("draft_ids", "accept", "alpha", "resid_mass", "resid_ids", "n_accepted", "out_tokens"):
        assert torch.equal(getattr(again, name), getattr(out, name)), name


def test_steps_rows_without_mass():
    """A drafter row of zeros gives the zero row, an accept of nothing and a residual draw from p, beside ordinary rows."""
    from paper_2506_03206_amd import rdk
    N, n, k = 4102, 1021, 16
    B = batch_for(N, n, k, 1, 0)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    kept = torch.sort(torch.randperm(N, generator=g, device="cuda")[:n]).values.to(torch.int32)
    kern = rdk.rdk_build_kernel(N, kept, rdk.SPARSE_TOPK, embeddings=torch.randn((N, 8), generator=g, device="cuda"), tau=0.1, k=k)
    p = torch.softmax(torch.randn((B, N), generator=g, device="cuda"), 1)
    q = torch.softmax(torch.randn((B, n), generator=g, device="cuda"), 1)
    q[1::3] = 0
    out = rdk.rdk_redistribute_verify(kern, rdk.LINEAR_SPARSE, p, q, 5, 0, 1, "prob", "prob")
    empty = torch.arange(B, device="cuda") % 3 == 1
    assert (out.draft_ids[empty] == -1).all() and (out.accept[empty] == 0).all() and (out.alpha[empty] == 0).all()
    assert (out.resid_ids[empty] >= 0).all() and (out.draft_ids[~empty] >= 0).all()
    torch.testing.assert_close(out.resid_mass[empty], p[empty].sum(1), rtol=1e-5, atol=1e-6)
