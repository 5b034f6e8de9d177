"""Runs of several ranks on one matrix: stacks of up to 32 factors take the plan without a transposed copy of A, larger
ones the plan that reads it, in any order and also where the workspace has no room for the stacks."""
import numpy as np
import pytest

from oracle import nmf_oracle as orc

EPS = 1e-16


@pytest.mark.gpu
@pytest.mark.parametrize("ranks", [[16, 64], [20, 60, 5], [50, 20, 50], [64, 16, 64]])
@pytest.mark.parametrize("kind", [3, 0])     # room for the stacks; for the runs one by one only
def test_ranks_on_one_matrix(ranks, kind):
    import torch

    import paper_2202_09518_amd as nmf
    m, n, iters = 300, 260, 2
    r = np.random.default_rng(sum(ranks))
    A = r.random((m, n), dtype=np.float32)
    W = [r.random((m, k), dtype=np.float32) for k in ranks]
    H = [r.random((k, n), dtype=np.float32) for k in ranks]
    Ad = torch.from_numpy(A).cuda()
    Wd, Hd = [torch.from_numpy(x).cuda() for x in W], [torch.from_numpy(x).cuda() for x in H]
    # 0.75 in every float of it: nothing that an earlier call left in the workspace can stand in for A^T
    ws = torch.full((nmf.nmf_mu_workspace_bytes(kind, m, n, 0, max(ranks), 0),), 0x3f, dtype=torch.uint8, device="cuda")
    nmf.nmf_mu_set_workspace(ws)
    try:
        nmf.nmf_mu_dense_batched(len(ranks), [Ad] * len(ranks), m, n, ranks, Wd, Hd, iters, EPS)
        torch.cuda.synchronize()
    finally:
        nmf.nmf_mu_set_workspace(None)
    for i in range(len(ranks)):
        Wr, Hr = orc.mu_dense(A, W[i], H[i], iters, float(np.float32(EPS)))
        # two updates of each factor, sums of one sign: a few roundings of 2^-24 per sum
        assert orc.rel_fro(Wd[i].cpu().numpy(), Wr) < 2e-6, i
        assert orc.rel_fro(Hd[i].cpu().numpy(), Hr) < 2e-6, i
