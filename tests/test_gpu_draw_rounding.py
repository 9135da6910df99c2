"""Draws whose threshold lies on a step of the prefix sums, where fp64 sums taken in another order differ by an ulp: the block and
the id that are picked carry mass and lie in the row."""
import numpy as np
import pytest
import torch

import oracle

N = 16384
ULP = 2.0 ** -52                                 # of a double in [1, 2)
BLOCK = {"draft": 1024, "residual": 1024, "bonus": 1024, "tree": 1024, "fused": 64}   # ids per block sum of each call's finish


def uniform(call, seed):
    """The uniform that decides the call's draw at position 0."""
    if call == "tree":
        return oracle.multi_uniform(seed, 0, 2)
    return float(oracle.uniforms(seed, 0)[{"draft": 0, "residual": 2, "bonus": 3, "fused": 2}[call]])


def with_rest(row, block, rest):
    """The rest of the total, with the blocks of three other lanes, in floats that add up to it exactly."""
    for i in range(3):
        f = np.float32(rest)
        f = np.nextafter(f, np.float32(0)) if float(f) > rest else f
        row[(4 + 4 * i) * block] = f
        rest -= float(f)
    assert rest == 0.0
    return row


def row_between_blocks(u, block):
    """A lane owns four blocks, of sums 1, 0, 3/4 ulp and 1/2 ulp, and the threshold u * total is 1 + ulp: added up one after the
    other they are 1 + 2 ulp, a scan over the lanes has reached 1 + ulp at the last of them, and 1 + 2 ulp three lanes later, where
    the lane has no block.  The row and the ids that may be drawn, or None where no total has that threshold."""
    thr = 1.0 + ULP
    total = next((float(t) for t in (thr / u, np.nextafter(thr / u, 0), np.nextafter(thr / u, 4)) if u * t == thr), 0.0)
    if not 1.01 < total < 1.99:
        return None
    row = np.zeros(N, np.float32)
    row[0], row[2 * block + 5], row[3 * block + 9] = 1.0, 0.75 * ULP, 0.5 * ULP
    return with_rest(row, block, total - (1.0 + 2 * ULP)), [2 * block + 5, 3 * block + 9]


def rows(call, make, count):
    """The first seeds whose uniform allows the construction, with their rows and the ids that may be drawn."""
    out = []
    for seed in range(1000):
        made = make(uniform(call, seed), BLOCK[call])
        if made is not None:
            out.append((seed,) + made)
        if len(out) == count:
            return out
    raise AssertionError("no seed")


def draw(call, row, seed):
    from paper_2506_03206_amd import rdk
    x = torch.from_numpy(row)[None].cuda()
    zero = torch.zeros_like(x)
    if call == "draft":
        return int(rdk.rdk_verify_sample(x, x, seed).draft_ids[0])
    if call == "residual":
        return int(rdk.rdk_verify_sample(x, zero, seed).resid_ids[0])
    if call == "bonus":
        return int(rdk.rdk_verify_sample(x, None, seed).resid_ids[0])
    if call == "tree":
        none = torch.full((1, 1), -1, dtype=torch.int32, device="cuda")
        return int(rdk.rdk_verify_multi(x, zero, 1, seed, cand_ids=none).token[0])
    kept = torch.arange(0, N, 16, dtype=torch.int32, device="cuda")
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    kern = rdk.rdk_build_kernel(N, kept, rdk.SPARSE_TOPK, embeddings=torch.randn((N, 16), generator=gen, device="cuda"), k=4)
    q = torch.zeros((1, kept.numel()), device="cuda")    # no drafter mass: the token is drawn from the target row
    return int(rdk.rdk_redistribute_verify(kern, rdk.LINEAR_SPARSE, x, q, seed).resid_ids[0])


@pytest.mark.gpu
@pytest.mark.parametrize("call", list(BLOCK))
def test_threshold_between_two_orders_of_the_block_sums(call):
    for seed, row, ids in rows(call, row_between_blocks, 3):
        assert draw(call, row, seed) in ids


def row_between_ids(u, block):
    """Ids 0, 4, 8 and 12 (0 to 3 in blocks of 64) of the first block weigh 1 and three times 1/4 ulp, and the threshold is 1: their
    own prefixes are rounded to 1, those of the empty places that follow to 1 + ulp.  The next id with a weight is drawn, or, with
    sums that don't round, the second."""
    step = 1 if block == 64 else 4
    total = next((float(t) for t in (1.0 / u, np.nextafter(1.0 / u, 0), np.nextafter(1.0 / u, 4)) if u * t == 1.0), 0.0)
    if not 1.01 < total < 1.99:
        return None
    row = np.zeros(N, np.float32)
    row[0], row[step], row[2 * step], row[3 * step] = 1.0, 0.25 * ULP, 0.25 * ULP, 0.25 * ULP
    row[50 * step + 1 if step > 1 else 50] = 2.0 ** -8
    return with_rest(row, block, total - (1.0 + 2.0 ** -8)), [step, 2 * step, 3 * step, 50 * step + 1 if step > 1 else 50]


@pytest.mark.gpu
@pytest.mark.parametrize("call", list(BLOCK))
def test_threshold_between_two_orders_of_a_block(call):
    for seed, row, ids in rows(call, row_between_ids, 3):
        assert draw(call, row, seed) in ids
