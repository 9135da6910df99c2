"""Rows that start at any multiple of their element's size: every path on rows at odd strides gives what it gives on rows at a stride
of eight elements, bit for bit (the order of its sums does not depend on where a row starts); the latter are held against the
oracle elsewhere.  N and n end inside a quad, a chunk of 1024 ids and a tile of 256."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def at_stride(x, stride):
    return torch.full((x.shape[0], stride), float("nan"), device="cuda", dtype=x.dtype)[:, :x.shape[1]].copy_(x)


def same(a, b):
    for x, y in zip(a, b):
        assert torch.equal(x, y)


@pytest.mark.parametrize("kind", ["prob", "logit", "logit_bf16"])
@pytest.mark.parametrize("N,n,B", [(515, 130, 5), (5121, 1027, 12), (30723, 3001, 66), (90002, 21001, 40)])
def test_rows_at_odd_strides(N, n, B, kind):
    from paper_2506_03206_amd import rdk
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N + B)
    kept = torch.sort(torch.randperm(N, generator=gen, device="cuda")[:n]).values.to(torch.int32)
    z = torch.randn((B, N), generator=gen, device="cuda") * 2
    p, q = z, (z + torch.randn((B, N), generator=gen, device="cuda"))[:, kept.long()]
    if kind == "prob":
        p, q = torch.softmax(p, 1), torch.softmax(q, 1) * 0.75
    elif kind == "logit_bf16":
        p, q = p.to(torch.bfloat16), q.to(torch.bfloat16)
    k = "prob" if kind == "prob" else "logit"
    E = torch.randn((N, 16), generator=gen, device="cuda")
    kern = rdk.rdk_build_kernel(N, kept, rdk.SPARSE_TOPK, embeddings=E, tau=0.1, k=9)
    cand = torch.randint(0, N, (B, 3), generator=gen, device="cuda", dtype=torch.int32)
    cand[:, 2] = N + 5                       # never kept: every position that comes so far takes another pass
    got = []
    for odd in (0, 1):
        ps, qs = (at_stride(x, (x.shape[1] + 15) // 8 * 8 + odd) for x in (p, q))
        out = torch.zeros((B, (N + 15) // 8 * 8 + odd), device="cuda")[:, :N]
        res = []
        for mode in (rdk.LINEAR_SPARSE, rdk.LINEAR_TAYLOR):
            o = rdk.rdk_redistribute_verify(kern, mode, ps, qs, seed=7, offset=0, gamma=1, p_kind=k, q_kind=k)
            qp = rdk.rdk_redistribute_linear(kern, mode, qs, k, p=ps if mode == rdk.LINEAR_TAYLOR else None, p_kind=k, out=out)
            v = rdk.rdk_verify_sample(ps, qp, seed=7, offset=0, gamma=1, p_kind=k)
            res += [o.draft_ids, o.alpha, o.resid_mass, o.resid_ids, o.out_tokens, qp.clone(), v.draft_ids, v.alpha, v.resid_mass, v.resid_ids]
        res += list(rdk.rdk_sample_draft(kern, qs, 7, 0, k))
        m = rdk.rdk_verify_multi(ps, qp, 3, 7, 0, k, cand_ids=cand.clone())
        res += [m.accepted, m.token, m.resid_mass]
        got.append(res)
    same(*got)


@pytest.mark.parametrize("fmt", ["f32", "bf16"])
def test_exact_rows_at_odd_strides(fmt):
    from paper_2506_03206_amd import rdk
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    N, n, B = 1031, 257, 70
    kept = torch.sort(torch.randperm(N, generator=gen, device="cuda")[:n]).values.to(torch.int32)
    M = torch.softmax(torch.randn((n, N), generator=gen, device="cuda"), 1)
    kern = rdk.rdk_build_kernel(N, kept, rdk.DENSE_F32 if fmt == "f32" else rdk.DENSE_BF16, dense_M=M)
    q = torch.randn((B, n), generator=gen, device="cuda")
    outs = [rdk.rdk_redistribute_exact(kern, at_stride(q, 264 + odd), "logit", out=torch.zeros((B, 1040 + odd), device="cuda")[:, :N])
            for odd in (0, 1)]
    same([outs[0]], [outs[1]])
