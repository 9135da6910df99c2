"""Verification in one launch, where a workgroup holds a position: the smallest rows, ends inside a quad, both sides of the
sizes at which the split form takes over, more rows than compute units, a masked chunk, rows at odd strides -- against the
oracle; and the two forms against each other."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_03206_amd import synth
from parity_util import check_verify_outputs

pytestmark = pytest.mark.gpu

SHAPES = [  # N, B, gamma, one launch with probabilities / with logits
    (3, 6, 3, False, False),
    (4, 6, 3, True, True),
    (5, 6, 2, True, True),
    (1023, 3, 1, True, True),
    (1026, 258, 2, True, True),      # more rows than compute units
    (1025, 514, 2, False, True),     # more than two per compute unit
    (8193, 6, 3, True, True),
    (24576, 2, 2, True, True),
    (24577, 2, 1, False, False),
    (32767, 48, 4, True, True),
    (33797, 128, 8, False, True),
]


@pytest.mark.parametrize("kind", ["prob", "logit", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_verify_against_oracle(shape, kind):
    from paper_2506_03206_amd import rdk
    N, B, gamma, one_p, one_l = shape
    rng = np.random.default_rng(N + B)
    zp = (rng.normal(size=(B, N)) * 2).astype(np.float32)
    zq = zp + rng.normal(size=(B, N)).astype(np.float32)
    if N > 3072:
        zp[0, 1024:2048] = -np.inf
    if kind == "bf16":
        zp = synth.bf16_round(zp)
    q = oracle.probs_from(zq, "logit").astype(np.float32)
    pk = "prob" if kind == "prob" else "logit"
    if kind == "prob":
        zp = oracle.probs_from(zp, "logit").astype(np.float32)
    wide = lambda a, dt: torch.nn.functional.pad(torch.from_numpy(a).cuda().to(dt), (0, 1), value=float("nan"))[:, :-1]
    p64 = oracle.probs_from(zp, pk)
    ref = oracle.verify_batch(p64, q.astype(np.float64), 9, 4, gamma=gamma)
    rdk.rdk_timing_select("verify_finalize_kernel")
    out = rdk.rdk_verify_sample(wide(zp, torch.bfloat16 if kind == "bf16" else torch.float32), wide(q, torch.float32), seed=9, offset=4,
                                gamma=gamma, p_kind=pk)
    torch.cuda.synchronize()
    rdk.rdk_timing_select(None)
    assert rdk.rdk_timing_read("verify_finalize_kernel")[0] == (0 if (one_p if kind == "prob" else one_l) else 1)
    check_verify_outputs(out, ref, p64, q.astype(np.float64), 9, 4, gamma, pk)


def test_both_forms_agree_bit_for_bit():
    """Rows of probabilities: the block sums have the same order in both forms, so a row's outputs do not depend on how many
    others are verified with it."""
    from paper_2506_03206_amd import rdk
    N, B, gamma = 9001, 514, 2
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    p = torch.softmax(torch.randn((B, N), generator=g, device="cuda") * 2, 1)
    q = torch.softmax(torch.randn((B, N), generator=g, device="cuda") * 2, 1)
    a = rdk.rdk_verify_sample(p, q, seed=3, offset=0, gamma=gamma)            # split
    b = rdk.rdk_verify_sample(p[:258], q[:258], seed=3, offset=0, gamma=gamma)  # one launch, 512 threads
    c = rdk.rdk_verify_sample(p[:34], q[:34], seed=3, offset=0, gamma=gamma)    # one launch, 1024 threads
    for name in ("draft_ids", "accept", "alpha", "resid_mass", "resid_ids"):
        for o, rows in ((b, 258), (c, 34)):
            assert torch.equal(getattr(a, name)[:rows], getattr(o, name)), name
    assert torch.equal(a.out_tokens[:129], b.out_tokens) and torch.equal(a.n_accepted[:17], c.n_accepted)
