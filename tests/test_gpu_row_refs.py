"""Eq. 3 in one pass where a wavefront's reference for its weights has to move: logits that rise along the row by more than a
float's exponentials hold, that start masked, that fall, and runs of kept ids longer than what is fetched ahead -- against the
oracle, with both sizes of workgroup."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_03206_amd import synth
from parity_util import check_verify_outputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["logit", "bf16"])
@pytest.mark.parametrize("N,n,B", [(40001, 5000, 6), (40001, 5000, 260), (4096, 1500, 4), (2050, 700, 4)])
def test_moving_references_against_oracle(N, n, B, kind):
    from paper_2506_03206_amd import rdk
    rng = np.random.default_rng(N + B)
    last = (N - 1) // 1024 * 1024
    dense = np.arange(last - 1024, last - 1024 + min(1024, n // 2))        # a chunk that keeps all, or most, of its ids
    others = np.setdiff1d(np.arange(N), dense)
    kept = np.sort(np.concatenate([dense, rng.choice(others, size=n - dense.size, replace=False)])).astype(np.int32)
    zp = (rng.normal(size=(B, N)) * 2).astype(np.float32)
    zq = (zp + rng.normal(size=(B, N)).astype(np.float32))[:, kept]
    chunk = np.arange(N) // 1024
    zp[0] += 40.0 * chunk                              # e^40 from one chunk to the next: the last one holds the mass
    zp[1] -= 40.0 * chunk
    zp[2, chunk < chunk[-1]] = -np.inf                 # nothing but the last chunk
    zq[3] += 40.0 * chunk[kept]
    zq[1] -= 40.0 * chunk[kept]
    zq[2, : n // 2] = -np.inf
    zp[3, last:] += 15.5                               # just beyond the weights that are taken as they are
    if kind == "bf16":
        zp, zq = synth.bf16_round(zp), synth.bf16_round(zq)
    kern = rdk.rdk_build_kernel(N, torch.from_numpy(kept).cuda(), rdk.IDENTITY)
    p64, q64 = oracle.probs_from(zp, "logit"), oracle.probs_from(zq, "logit")
    ref_qp = oracle.redistribute_batch("taylor", q64, kept, N, p=p64)
    ref = oracle.verify_batch(p64, ref_qp, 9, 4, gamma=2)
    dt = torch.bfloat16 if kind == "bf16" else torch.float32
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda().to(dt)
    rdk.rdk_timing_select("taylor_row_kernel")
    out = rdk.rdk_redistribute_verify(kern, rdk.LINEAR_TAYLOR, t(zp), t(zq), 9, 4, 2, "logit", "logit")
    torch.cuda.synchronize()
    rdk.rdk_timing_select(None)
    assert rdk.rdk_timing_read("taylor_row_kernel")[0] == 1
    check_verify_outputs(out, ref, p64, ref_qp, 9, 4, 2, "logit", min_exact=0.6)
