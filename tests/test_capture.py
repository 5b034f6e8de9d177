"""Calls under stream capture: a call that the workspace of an earlier one can serve is captured, whatever it could have
used beyond that, and replays give the eager result."""
import numpy as np
import pytest

EPS = 1e-16


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", [(1001, 1003, 40), (700, 300, 12)])
def test_a_longer_run_is_captured_after_a_short_one(m, n, k):
    """1001 x 1003 at 40 factors: one iteration runs on a copy of A, several would take A^T as well."""
    import torch

    import paper_2202_09518_amd as nmf
    g = torch.Generator(device="cuda")
    g.manual_seed(m + n)
    A, W, H = (torch.rand(s, generator=g, device="cuda") for s in ((m, n), (m, k), (k, n)))
    torch.cuda.synchronize()
    nmf.nmf_mu_release()
    Wd, Hd = W.clone(), H.clone()
    nmf.nmf_mu_dense(A, m, n, k, Wd, Hd, 1, EPS)       # the only call that may allocate
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        Wd.copy_(W)
        Hd.copy_(H)
        nmf.nmf_mu_dense(A, m, n, k, Wd, Hd, 3, EPS)
    results = []
    for _ in range(3):
        Wd.zero_()
        Hd.zero_()
        graph.replay()
        torch.cuda.synchronize()
        results.append((Wd.clone(), Hd.clone()))
        torch.cuda.synchronize()
    We, He = W.clone(), H.clone()
    nmf.nmf_mu_dense(A, m, n, k, We, He, 3, EPS)       # free to take the larger plan
    torch.cuda.synchronize()
    for Wg, Hg in results:
        assert torch.equal(Wg, results[0][0]) and torch.equal(Hg, results[0][1])
        # three iterations on either plan: a few roundings of 2^-24 apart
        assert ((Wg - We).norm() / We.norm()).item() < 2e-6
        assert ((Hg - He).norm() / He.norm()).item() < 2e-6
    del graph
