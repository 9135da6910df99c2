"""Eq. 3 without q' where it can go wrong, in one pass, out of registers and in two passes: the smallest vocabularies of each, ends
inside a quad, runs of one slot at the end of the row, chunks without kept ids or without any target mass, two
workgroups on a compute unit, rows at odd strides -- against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2506_03206_amd import synth
from parity_util import check_verify_outputs

pytestmark = pytest.mark.gpu

ROW, WHOLE, TWO = "taylor_row_kernel", "taylor_whole_kernel", "taylor_write_kernel"   # one pass, out of registers, two passes

SHAPES = [  # N, n, B, gamma, which ids are kept, what takes probabilities, logits
    (5, 4, 6, 3, "any", WHOLE, WHOLE),
    (1023, 130, 3, 1, "any", WHOLE, WHOLE),
    (1025, 131, 3, 3, "any", WHOLE, WHOLE),
    (4095, 900, 258, 2, "any", WHOLE, WHOLE),     # more rows than compute units
    (4099, 1030, 4, 2, "tail", WHOLE, WHOLE),     # the last three runs hold one slot each
    (4097, 900, 514, 2, "any", WHOLE, ROW),       # the shortest logit rows in one pass
    (8193, 2000, 257, 1, "any", ROW, ROW),        # the shortest rows of probabilities
    (8195, 1030, 300, 2, "tail", ROW, ROW),
    (9001, 700, 260, 4, "first", ROW, ROW),       # the kept ids in one chunk
    (12289, 1001, 3, 3, "tail", WHOLE, ROW),
    (12291, 12291, 300, 1, "any", ROW, ROW),      # every id is kept
    (24576, 6001, 2, 2, "any", WHOLE, ROW),
    (32769, 4, 88, 4, "any", ROW, ROW),           # one quad of slots, in at most four chunks
    (33003, 8190, 90, 3, "any", ROW, ROW),
    (49152, 9999, 2, 1, "tail", TWO, ROW),
]


@pytest.mark.parametrize("kind", ["prob", "logit", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_one_pass_rows_against_oracle(shape, kind):
    from paper_2506_03206_amd import rdk
    N, n, B, gamma, where, *takes = shape
    kernel = takes[kind != "prob"]
    rng = np.random.default_rng(N + n)
    if where == "first":
        kept = np.sort(rng.choice(1000, size=n, replace=False))
    elif where == "tail":
        last = (N - 1) // 1024 * 1024                  # first id of the last chunk
        kept = np.concatenate([np.sort(rng.choice(last - 2048, size=n - 3, replace=False)), [last - 1500, last - 7, N - 1]])
    else:
        kept = np.sort(rng.choice(N, size=n, replace=False))
    kept = kept.astype(np.int32)
    zp = (rng.normal(size=(B, N)) * 2).astype(np.float32)
    zq = (zp + rng.normal(size=(B, N)).astype(np.float32))[:, kept]
    if kind == "bf16":
        zp, zq = synth.bf16_round(zp), synth.bf16_round(zq)
    if N > 3072:
        zp[0, 1024:2048] = -np.inf                     # a chunk of masked ids
    pk = "prob" if kind == "prob" else "logit"
    if kind == "prob":
        zp, zq = [oracle.probs_from(x, "logit").astype(np.float32) for x in (zp, zq)]
    dt = torch.bfloat16 if kind == "bf16" else torch.float32
    wide = lambda a: torch.nn.functional.pad(torch.from_numpy(np.ascontiguousarray(a)).cuda().to(dt), (0, 1), value=float("nan"))[:, :-1]
    kern = rdk.rdk_build_kernel(N, torch.from_numpy(kept).cuda(), rdk.IDENTITY)
    p64, q64 = oracle.probs_from(zp, pk), oracle.probs_from(zq, pk)
    ref_qp = oracle.redistribute_batch("taylor", q64, kept, N, p=p64)
    rdk.rdk_timing_select(kernel)
    out = rdk.rdk_redistribute_verify(kern, rdk.LINEAR_TAYLOR, wide(zp), wide(zq), 9, 4, gamma, pk, pk)
    torch.cuda.synchronize()
    rdk.rdk_timing_select(None)
    assert rdk.rdk_timing_read(kernel)[0] == 1
    ref = oracle.verify_batch(p64, ref_qp, 9, 4, gamma=gamma)
    check_verify_outputs(out, ref, p64, ref_qp, 9, 4, gamma, pk, min_exact=0.6)


@pytest.mark.parametrize("kind", ["logit", "bf16"])
@pytest.mark.parametrize("N,B,kernel", [(4099, 6, WHOLE), (4099, 260, WHOLE), (4099, 514, ROW), (12301, 6, ROW), (60001, 66, ROW), (60001, 6, TWO)])
def test_rows_masked_with_the_lowest_finite_value(N, B, kernel, kind):
    """Masks of finfo.min instead of -inf, over part of a row and over all of it (a uniform row then), out of registers, in one pass and
    split over workgroups; a logit near the largest finite value beside them."""
    from paper_2506_03206_amd import rdk
    rng = np.random.default_rng(N + B)
    kept = np.sort(rng.choice(N, size=N // 5, replace=False)).astype(np.int32)
    zp = (rng.normal(size=(B, N)) * 2).astype(np.float32)
    zq = (zp + rng.normal(size=(B, N)).astype(np.float32))[:, kept]
    dt = torch.bfloat16 if kind == "bf16" else torch.float32
    if kind == "bf16":
        zp, zq = synth.bf16_round(zp), synth.bf16_round(zq)
    low = np.float32(torch.finfo(dt).min)
    zq[0] = low                                        # the whole drafter row
    zq[1, : kept.size // 2] = low                      # half of it: chunks whose kept ids are all masked
    zp[2] = low                                        # the whole target row
    zp[3, 1024:2048] = low                             # one chunk of it
    zp[4, 100] = np.float32(torch.finfo(dt).max)       # a one-hot row whose differences leave the range of a float
    zp[5], zq[5] = low, low
    kern = rdk.rdk_build_kernel(N, torch.from_numpy(kept).cuda(), rdk.IDENTITY)
    p64, q64 = oracle.probs_from(zp, "logit"), oracle.probs_from(zq, "logit")
    ref_qp = oracle.redistribute_batch("taylor", q64, kept, N, p=p64)
    ref = oracle.verify_batch(p64, ref_qp, 9, 4, gamma=2)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda().to(dt)
    rdk.rdk_timing_select(kernel)
    out = rdk.rdk_redistribute_verify(kern, rdk.LINEAR_TAYLOR, t(zp), t(zq), 9, 4, 2, "logit", "logit")
    torch.cuda.synchronize()
    rdk.rdk_timing_select(None)
    assert rdk.rdk_timing_read(kernel)[0] == 1
    check_verify_outputs(out, ref, p64, ref_qp, 9, 4, 2, "logit", min_exact=0.6)


@pytest.mark.parametrize("N,B", [(60001, 6), (33001, 70)])
def test_two_passes_over_chunks_of_masked_ids(N, B):
    """q' of rows in which a wavefront's first chunk, and every chunk of one, is masked with -inf."""
    from paper_2506_03206_amd import rdk
    rng = np.random.default_rng(N)
    kept = np.sort(rng.choice(N, size=N // 4, replace=False)).astype(np.int32)
    zp = (rng.normal(size=(B, N)) * 2).astype(np.float32)
    zq = np.ascontiguousarray((zp + rng.normal(size=(B, N)).astype(np.float32))[:, kept])
    zp[0, :3072] = -np.inf
    zp[1, 1024:] = -np.inf
    kern = rdk.rdk_build_kernel(N, torch.from_numpy(kept).cuda(), rdk.IDENTITY)
    got = rdk.rdk_redistribute_linear(kern, rdk.LINEAR_TAYLOR, torch.from_numpy(zq).cuda(), "logit", p=torch.from_numpy(zp).cuda(),
                                      p_kind="logit").cpu().numpy().astype(np.float64)
    ref = oracle.redistribute_batch("taylor", oracle.probs_from(zq, "logit"), kept, N, p=oracle.probs_from(zp, "logit"))
    assert (np.abs(got - ref) <= 1e-5 * np.abs(ref) + 1e-7).all()
