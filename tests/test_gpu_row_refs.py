"""Eq. 3 in one pass where the largest logits of a row's chunks, which their weights are taken relative to, lie far apart: logits
that rise along the row by more than a float's exponentials hold, that start masked, that fall, and runs of kept ids longer than
what is fetched ahead -- against the oracle, with both sizes of workgroup.  And how finely the weights are rounded."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_03206_amd import synth
from parity_util import check_verify_outputs

pytestmark = pytest.mark.gpu

ROW, WHOLE = "taylor_row_kernel", "taylor_whole_kernel"   # one pass, and out of registers where the rows are short


@pytest.mark.parametrize("kind", ["logit", "bf16"])
@pytest.mark.parametrize("N,n,B,kernel", [(40001, 5000, 6, ROW), (40001, 5000, 260, ROW), (12300, 1500, 4, ROW), (4100, 1500, 514, ROW),
                                          (4096, 1500, 4, WHOLE), (2050, 700, 4, WHOLE)])
def test_moving_references_against_oracle(N, n, B, kernel, kind):
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
    rdk.rdk_timing_select(kernel)
    out = rdk.rdk_redistribute_verify(kern, rdk.LINEAR_TAYLOR, t(zp), t(zq), 9, 4, 2, "logit", "logit")
    torch.cuda.synchronize()
    rdk.rdk_timing_select(None)
    assert rdk.rdk_timing_read(kernel)[0] == 1
    check_verify_outputs(out, ref, p64, ref_qp, 9, 4, 2, "logit", min_exact=0.6)


def test_the_largest_weights_of_a_chunk_are_not_rounded():
    """A row's mass in two chunks, hundreds of ids at logit 0 in one and four ids at a = 4.5 .. 5.5 in a later one.  Relative to its
    own chunk every weight is 1, and the factor between the chunks carries the rounding of a * log2(e) along.  Rows whose product
    rounds up against rows where it rounds down: a weight taken relative to the other chunk is off by the rounding, 3.1e-7 of it
    between the two sets, which moves alpha (about the mass f of the four ids) by f (1 - f) of that, 7e-8.  What other roundings a
    row has (1e-7 of alpha at most, of either sign) average out over 64 rows a set: 1.5e-8 is allowed."""
    from paper_2506_03206_amd import rdk
    N, B, K, far = 40001, 64, 4, 16 * 1024
    rng = np.random.default_rng(5)
    kept = np.concatenate([[5], far + 4 * np.arange(K)]).astype(np.int32)
    kern = rdk.rdk_build_kernel(N, torch.from_numpy(kept).cuda(), rdk.IDENTITY)
    a = rng.uniform(4.5, 5.5, 20000).astype(np.float32)
    off = (a * np.float32(np.log2(np.e))).astype(np.float64) - a.astype(np.float64) * np.log2(np.e)
    shift = []
    for some in (a[off > 1.3e-7][:B], a[off < -3.2e-7][:B]):
        zp = np.full((B, N), -np.inf, np.float32)
        for b in range(B):
            zp[b, : rng.integers(350, 1000)] = 0
        zp[:, kept[1:]] = some[:, None]
        zq = np.zeros((B, K + 1), np.float32)
        p64, q64 = oracle.probs_from(zp, "logit"), oracle.probs_from(zq, "logit")
        ref_qp = oracle.redistribute_batch("taylor", q64, kept, N, p=p64)
        out = rdk.rdk_redistribute_verify(kern, rdk.LINEAR_TAYLOR, torch.from_numpy(zp).cuda(), torch.from_numpy(zq).cuda(), 9, 4, 1,
                                          "logit", "logit")
        shift.append(np.mean(out.alpha.cpu().numpy().astype(np.float64).ravel() - np.minimum(p64, ref_qp).sum(1)))
    assert abs(shift[0] - shift[1]) < 1.5e-8, shift
