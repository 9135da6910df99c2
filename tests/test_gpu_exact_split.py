"""The exact product with its slots split over workgroups: even and uneven splits, every workgroup shape, output rows at odd
strides, ragged ends of the slots -- against fp64 on the kernel as stored."""
import numpy as np
import pytest
import torch

from parity_util import assert_close

pytestmark = pytest.mark.gpu

SHAPES = [  # N, n, B
    (130, 3, 2),         # one turn of stages: not split
    (515, 500, 5),       # two turns
    (1003, 1000, 129),   # three turns, two rows of workgroups
    (8033, 2500, 3),     # seven turns in four splits, the last one shorter
    (8033, 2500, 513),   # five rows of the smallest workgroups
    (9001, 1537, 200),
    (9001, 1537, 300),
    (16500, 400, 6),     # column groups enough: not split
    (4500, 4097, 3),     # rows long enough for statistics of their own (fp32 path)
    (4500, 4096, 3),
]


@pytest.mark.parametrize("kind", ["prob", "logit"])
@pytest.mark.parametrize("fmt", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES)
def test_split_product(shape, fmt, kind):
    check_product(shape, fmt, kind)


# The fp32 path's wavefronts (128 ids), workgroups (512 ids, dealt out eight at a time), turns (48 slots) and row groups (64
# positions) at their edges.
@pytest.mark.parametrize("shape", [(127, 47, 64), (512, 48, 65), (513, 49, 128), (4095, 96, 1), (4097, 97, 129), (1400, 290, 193)])
def test_fp32_edges(shape):
    check_product(shape, "f32", "prob")


# Drafter rows brought into operand form by a workgroup each and by a thread per record: both sides of the line (2048 slots of
# probabilities, 4096 of logits), ends inside eight slots, one chunk of 1024 and a single slot more.
@pytest.mark.parametrize("kind", ["prob", "logit"])
@pytest.mark.parametrize("shape", [(700, 2048, 65), (700, 2049, 65), (513, 3077, 1), (700, 4096, 33), (700, 4097, 129)])
def test_fp32_drafter_rows(shape, kind):
    N, n, B = shape
    check_product((N + n, n, B), "f32", kind)


# Column groups (128 ids) beyond whole rounds of the chip (256 workgroups, 768 of the smallest ones, 512 of the next, or those and 256
# more) have their slots split: one group and a ragged one, 128 groups (the most that are split), one more, a single turn of slots (nothing to split), and the batches
# at which the workgroup changes.
@pytest.mark.parametrize("shape", [(98305, 800, 3), (98500, 400, 64), (98305, 800, 65), (98500, 400, 128), (65537, 800, 65), (81900, 800, 100), (32897, 1153, 129),
                                   (33001, 1200, 256), (49152, 800, 300), (49153, 800, 260), (33001, 384, 200), (33030, 3100, 512)])
def test_bf16_tail(shape):
    check_product(shape, "bf16", "prob")


def check_product(shape, fmt, kind):
    from paper_2506_03206_amd import rdk
    N, n, B = shape
    rng = np.random.default_rng(N + B)
    kept = np.sort(rng.choice(N, size=n, replace=False)).astype(np.int32)
    M = rng.random((n, N)).astype(np.float32) ** 4
    M /= M.sum(1, keepdims=True)
    kern = rdk.rdk_build_kernel(N, torch.from_numpy(kept).cuda(), rdk.DENSE_F32 if fmt == "f32" else rdk.DENSE_BF16,
                                dense_M=torch.from_numpy(M).cuda())
    Ms = M.astype(np.float64) if fmt == "f32" else rdk.rdk_kernel_get_dense(kern).cpu().numpy().astype(np.float64)
    x = (rng.normal(size=(B, n)) * 2).astype(np.float32)
    if kind == "prob":
        x = np.exp(x)
        x = (x / x.sum(1, keepdims=True) * 0.75).astype(np.float32)
    q = x.astype(np.float64) if kind == "prob" else np.exp(x.astype(np.float64))
    q /= q.sum(1, keepdims=True)
    out = torch.full((B, N + 1), -7.0, device="cuda")
    rdk.rdk_redistribute_exact(kern, torch.from_numpy(x).cuda(), kind, out=out[:, :N])
    ref = q @ Ms
    ref /= ref.sum(1, keepdims=True) if fmt == "bf16" else 1.0
    # 16-bit: a drafter weight is rounded by at most 2^-12 of itself, which moves a sum of positive terms by as much, and the
    # mass of the row that it is divided by too: 2^-11, and the rounding of the fp32 sums.  fp32: the latter alone
    assert_close(out[:, :N].cpu().numpy(), ref, rtol=2.0 ** -11 + 1e-5 if fmt == "bf16" else 1e-5, atol=1e-9, what="exact product")
    assert (out[:, N] == -7.0).all()
