"""A drafter row of logits whose ids are all masked with -inf has no mass: every redistribution returns the zero row for it, and its
neighbours are as they are beside an ordinary row."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def kernel(form, N, n, k):
    from paper_2506_03206_amd import rdk
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N + n)
    kept = torch.sort(torch.randperm(N, generator=gen, device="cuda")[:n]).values.to(torch.int32)
    if form in ("taylor", "identity"):
        return rdk.rdk_build_kernel(N, kept, rdk.IDENTITY)
    fmt = {"sparse": rdk.SPARSE_TOPK, "exact_f32": rdk.DENSE_F32, "exact_bf16": rdk.DENSE_BF16}[form]
    return rdk.rdk_build_kernel(N, kept, fmt, embeddings=torch.randn((N, 16), generator=gen, device="cuda"), k=k)


# Every kernel that forms drafter weights: rows of Eq. 3 by one workgroup and in two passes (statistics of the target row before or
# in the first of them), positions out of LDS one and several at a time and thirty-two at a time, operands of the dense products
# written a row at a time and in their own order.
CASES = [("taylor", 3000, 700, 0, 5), ("taylor", 40000, 9000, 0, 5), ("taylor", 900, 300, 0, 1200), ("identity", 3000, 700, 0, 5),
         ("sparse", 3000, 700, 8, 5), ("sparse", 60000, 30000, 8, 5), ("sparse", 20000, 5000, 32, 200), ("sparse", 40000, 24000, 32, 80),
         ("exact_f32", 3000, 700, 0, 5), ("exact_f32", 6000, 4500, 0, 5), ("exact_bf16", 3000, 700, 0, 5)]


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("p_kind", ["logit", "prob"])
@pytest.mark.parametrize("form,N,n,k,B", CASES)
def test_masked_drafter_row(form, N, n, k, B, p_kind, bf16):
    from paper_2506_03206_amd import rdk
    kern = kernel(form, N, n, k)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(B)
    dt = torch.bfloat16 if bf16 else torch.float32
    zp = torch.randn((B, N), generator=gen, device="cuda") * 2
    p = torch.softmax(zp, 1) if p_kind == "prob" else zp.to(dt)
    whole = (torch.randn((B, n), generator=gen, device="cuda") * 2).to(dt)
    masked = whole.clone()
    gone = B // 2
    masked[gone] = -float("inf")
    others = torch.arange(B, device="cuda") != gone
    mode = rdk.LINEAR_TAYLOR if form == "taylor" else rdk.LINEAR_SPARSE
    if form in ("taylor", "sparse"):
        run = lambda q: rdk.rdk_redistribute_linear(kern, mode, q, "logit", p=p if form == "taylor" else None, p_kind=p_kind)
    else:
        run = lambda q: rdk.rdk_redistribute_exact(kern, q, "logit")
    got, beside = run(masked), run(whole)
    assert not got[gone].any() and torch.equal(got[others], beside[others])
    if form == "sparse":
        ids, qd = rdk.rdk_sample_draft(kern, masked, 5, 0, "logit")
        assert int(ids[gone]) == -1 and float(qd[gone]) == 0.0 and (ids[others] >= 0).all()
    if form in ("taylor", "sparse"):
        for keep in (False, True):
            held = torch.empty((B, N), device="cuda") if keep else None
            o = rdk.rdk_redistribute_verify(kern, mode, p, masked, 5, 0, 0, p_kind, "logit", q_prime=held)
            assert int(o.draft_ids[gone]) == -1 and int(o.accept[gone]) == 0 and float(o.alpha[gone]) == 0.0
            assert int(o.resid_ids[gone]) >= 0 and abs(float(o.resid_mass[gone]) - 1.0) < 1e-5   # fp32 sum of a row that adds up to one
            assert (o.draft_ids[others] >= 0).all() and (o.alpha[others] > 0).all()
            assert not keep or not held[gone].any()
