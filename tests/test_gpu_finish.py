"""The per-sequence scan that runs inside the finish of the rows (Alg. 4, steps 4-10): its outputs follow from the rows' own
accept flags and ids, call after call on the same workspace and in replays of a HIP graph, up to and beyond the longest
sequence that one wavefront scans."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def rows(N, B, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    z = torch.randn((B, N), generator=g, device="cuda") * 2
    return torch.softmax(z, 1), torch.softmax(z + 0.7 * torch.randn((B, N), generator=g, device="cuda"), 1)


def check_scan(o, gamma):
    acc, d, r = o.accept.cpu().numpy().reshape(-1, gamma), o.draft_ids.cpu().numpy().reshape(-1, gamma), o.resid_ids.cpu().numpy().reshape(-1, gamma)
    n, tok = o.n_accepted.cpu().numpy(), o.out_tokens.cpu().numpy()
    for s in range(acc.shape[0]):
        j = gamma if acc[s].all() else int(np.argmin(acc[s]))
        want = np.full(gamma + 1, -1)
        want[:j] = d[s, :j]
        if j < gamma:
            want[j] = r[s, j]
        assert n[s] == j and np.array_equal(tok[s], want)


@pytest.mark.parametrize("gamma", [1, 2, 63, 64])
def test_scan_follows_from_the_rows(gamma):
    from paper_2506_03206_amd import rdk
    N, S = 1300, 5
    o = rdk.VerifyOutputs(S * gamma, N, gamma, "cuda")
    for rep in range(3):                                   # the workspace keeps what the call before left in it
        p, q = rows(N, S * gamma, rep)
        rdk.rdk_verify_sample(p, q, seed=5, offset=rep, gamma=gamma, outputs=o)
        check_scan(o, gamma)


def test_scan_in_graph_replays():
    from paper_2506_03206_amd import rdk
    N, S, gamma = 1300, 7, 5
    p, q = rows(N, S * gamma, 0)
    o = rdk.VerifyOutputs(S * gamma, N, gamma, "cuda")
    rdk.rdk_verify_sample(p, q, seed=5, offset=0, gamma=gamma, outputs=o)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rdk.rdk_verify_sample(p, q, seed=5, offset=0, gamma=gamma, outputs=o)
    for rep in range(3):
        p2, q2 = rows(N, S * gamma, 10 + rep)
        p.copy_(p2)
        q.copy_(q2)
        o.n_accepted.fill_(-7)
        o.out_tokens.fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        check_scan(o, gamma)
        ref = rdk.rdk_verify_sample(p, q, seed=5, offset=0, gamma=gamma)
        assert torch.equal(ref.out_tokens, o.out_tokens) and torch.equal(ref.n_accepted, o.n_accepted)


@pytest.mark.parametrize("N,B,gamma,kind", [(1300, 1024, 8, "prob"), (1300, 1024, 4, "logit"), (30000, 256, 2, "prob"), (1300, 512, 32, "prob")])
def test_every_sequence_of_a_large_batch_is_scanned(N, B, gamma, kind):
    """Rows of a sequence on many compute units at once, forty calls on one workspace: no sequence is left without its scan."""
    from paper_2506_03206_amd import rdk
    p, q = rows(N, B, 3)
    if kind == "logit":
        p = torch.log(p)
    o = rdk.VerifyOutputs(B, N, gamma, "cuda")
    at = torch.arange(gamma + 1, device="cuda")
    for rep in range(40):
        o.n_accepted.fill_(-7)
        o.out_tokens.fill_(-7)
        rdk.rdk_verify_sample(p, q, seed=9, offset=rep * B, gamma=gamma, p_kind=kind, outputs=o)
        acc = o.accept.reshape(-1, gamma).to(torch.int32)
        n = torch.cumprod(acc, 1).sum(1)
        pad = lambda t: torch.nn.functional.pad(t.reshape(-1, gamma), (0, 1), value=-1)
        want = torch.where(at < n[:, None], pad(o.draft_ids), torch.where(at == n[:, None], pad(o.resid_ids), -1))
        assert torch.equal(n.to(torch.int32), o.n_accepted) and torch.equal(want.to(torch.int32), o.out_tokens), rep
