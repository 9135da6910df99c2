"""The entry point that allocates nothing (rdk_verify_sample_static): its outputs against rdk_verify_sample's on the
same inputs, bit for bit, on two calls in a row of which the second is smaller (the scratch array keeps the first
call's contents), the largest batches it takes, and the refusal of a batch beyond the fixed scratch size."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_03206_amd import synth
from parity_util import check_verify_outputs

pytestmark = pytest.mark.gpu

FIELDS = ("draft_ids", "accept", "alpha", "resid_mass", "resid_ids", "n_accepted", "out_tokens")


def inputs(N, B, seed, logits):
    rng = np.random.default_rng(seed)
    z = rng.normal(0, 3, size=(2, B, N)).astype(np.float32)
    e = np.exp(z.astype(np.float64) - z.max(2, keepdims=True))
    p, q = [(x / x.sum(2 if x.ndim == 3 else 1, keepdims=True)) for x in (e[0], e[1])]
    p_in = z[0] if logits else p.astype(np.float32)
    return p_in, q.astype(np.float32)


def test_static_scratch_entry_point_matches_workspace_entry_point():
    from paper_2506_03206_amd import rdk
    rdk.lib()
    assert torch.cuda.is_available()
    dev = torch.device("cuda:0")
    # first a batch of 5000-id rows (5 block sums per row), then a smaller one that leaves most of the scratch stale
    for (N, B, gamma, logits, seed) in ((5000, 24, 4, True, 1), (1300, 6, 3, False, 2)):
        p_in, q = inputs(N, B, seed, logits)
        kind = "logit" if logits else "prob"
        p_d, q_d = torch.from_numpy(p_in).to(dev), torch.from_numpy(q).to(dev)
        ref = rdk.rdk_verify_sample(p_d, q_d, seed=11, offset=3, gamma=gamma, p_kind=kind)
        out = rdk.VerifyOutputs(B, N, gamma, dev)
        torch.cuda.synchronize()
        before = torch.cuda.memory_allocated()
        rdk.rdk_verify_sample_static(p_d, q_d, seed=11, offset=3, gamma=gamma, p_kind=kind, outputs=out)
        torch.cuda.synchronize()
        assert torch.cuda.memory_allocated() == before
        for name in FIELDS:
            assert torch.equal(getattr(out, name), getattr(ref, name)), (name, N, B)
        # and both agree with the oracle
        p64 = oracle.probs_from(p_in, kind)
        q64 = q.astype(np.float64)
        check_verify_outputs(out, oracle.verify_batch(p64, q64, 11, 3, gamma=gamma), p64, q64, 11, 3, gamma, kind, min_exact=0.9)
    # the bonus draw (no drafter row) through the same entry point
    p_in, _ = inputs(1300, 6, 3, False)
    p_d = torch.from_numpy(p_in).to(dev)
    ref = rdk.rdk_verify_sample(p_d, None, seed=5)
    out = rdk.VerifyOutputs(6, 1300, 0, dev)
    rdk.rdk_verify_sample_static(p_d, None, seed=5, outputs=out)
    assert torch.equal(out.resid_ids, ref.resid_ids) and torch.equal(out.resid_mass, ref.resid_mass)


def test_static_scratch_entry_point_refuses_large_batches():
    from paper_2506_03206_amd import rdk
    dev = torch.device("cuda:0")
    N, B = 1024 * 40, 4096                       # 3 * 4 * B * 40 bytes of block sums = 1.9 MB ... doubled below
    p = torch.zeros((2, N), dtype=torch.float32, device=dev)
    # the size check happens on the host before anything is launched: rows are never read, so a 2-row tensor with a
    # declared batch of 3 * B positions (5.9 MB of block sums) is enough to ask for too much
    import ctypes
    d = rdk.VerifyDesc(B=3 * B, N=N, gamma=0, sample_draft=1, seed=0, offset=0)
    ids = torch.zeros(3 * B, dtype=torch.int32, device=dev)
    acc = torch.zeros(3 * B, dtype=torch.uint8, device=dev)
    rc = rdk.lib().rdk_verify_sample_static(ctypes.byref(d), ctypes.c_void_p(p.data_ptr()), rdk.PROB_F32, N,
                                            ctypes.c_void_p(p.data_ptr()), N, ctypes.c_void_p(ids.data_ptr()),
                                            ctypes.c_void_p(acc.data_ptr()), None, None, ctypes.c_void_p(ids.data_ptr()),
                                            None, None, None)
    assert rc == 6                               # RDK_ERR_WORKSPACE


@pytest.mark.parametrize("N,B,gamma", [(4, 209696, 4), (4, 209696, 0), (4, 116484, 4), (128256, 2759, 1)])
def test_scratch_limit_is_that_of_the_block_sums(N, B, gamma):
    """The largest batches the 4 MiB hold: 12 bytes per row and 1024 ids and the statistics partials, with a per-sequence scan
    as without.  A workspace sized for gamma = 0 serves a scan too."""
    import ctypes
    from paper_2506_03206_amd import rdk
    dev = torch.device("cuda:0")
    g = torch.Generator(device=dev)
    g.manual_seed(N + B)
    p = torch.softmax(torch.randn((B, N), generator=g, device=dev), 1)
    q = torch.softmax(torch.randn((B, N), generator=g, device=dev), 1)
    ref = rdk.rdk_verify_sample(p, q, seed=11, offset=3, gamma=gamma)
    out = rdk.VerifyOutputs(B, N, gamma, dev)
    rdk.rdk_verify_sample_static(p, q, seed=11, offset=3, gamma=gamma, outputs=out)
    small = rdk.VerifyOutputs(B, N, gamma, dev)
    d = rdk.VerifyDesc(B=B, N=N, gamma=0, sample_draft=1, seed=0, offset=0)
    need = ctypes.c_size_t()
    assert rdk.lib().rdk_verify_workspace_bytes(ctypes.byref(d), ctypes.byref(need)) == 0
    assert need.value - 256 <= 4 << 20
    small.ws = torch.empty(need.value, dtype=torch.uint8, device=dev)
    rdk.rdk_verify_sample(p, q, seed=11, offset=3, gamma=gamma, outputs=small)
    for name in FIELDS[: None if gamma else 5]:
        assert torch.equal(getattr(out, name), getattr(ref, name)), name
        assert torch.equal(getattr(small, name), getattr(ref, name)), name
    if B != 116484:                                    # (there the records would not fit beside the sums)
        d.B += 1                                       # one row more and the sums do not fit
        assert rdk.lib().rdk_verify_workspace_bytes(ctypes.byref(d), ctypes.byref(need)) == 0 and need.value - 256 > 4 << 20
