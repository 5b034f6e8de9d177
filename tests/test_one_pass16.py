"""The one-pass kernel for up to 16 factors, at row counts that the resident plan does not take: column counts that leave
waves without columns or with a few, rests of row blocks, more than 8 blocks a workgroup, against the oracle; a run cut in
two; the objective of every iteration."""
import numpy as np
import pytest

from oracle import nmf_oracle as orc

EPS = 1e-16


@pytest.mark.gpu
@pytest.mark.parametrize("m,n", [(16385, 4), (16417, 36), (20001, 100), (8257, 260), (33000, 484), (270001, 132), (140001, 512)])
@pytest.mark.parametrize("k", [3, 16])
def test_iterations(m, n, k):
    import torch

    import paper_2202_09518_amd as nmf
    r = np.random.default_rng(m + n + k)
    A, W, H = (r.random(s, dtype=np.float32) for s in ((m, n), (m, k), (k, n)))
    Ad, eps = torch.from_numpy(A).cuda(), float(np.float32(EPS))
    Wd, Hd = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
    nmf.nmf_mu_dense(Ad, m, n, k, Wd, Hd, 3, EPS)
    W2, H2 = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
    nmf.nmf_mu_dense(Ad, m, n, k, W2, H2, 2, EPS)
    got = nmf.nmf_mu_dense_monitor(Ad, m, n, k, W2, H2, 1, EPS)[0]
    torch.cuda.synchronize()
    assert torch.equal(Wd, W2) and torch.equal(Hd, H2)
    Wr, Hr = orc.mu_dense(A, W, H, 3, eps)
    # three updates of each factor, sums of one sign: a few roundings of 2^-24 per sum
    assert orc.rel_fro(Wd.cpu().numpy(), Wr) < 3e-6 and orc.rel_fro(Hd.cpu().numpy(), Hr) < 3e-6
    want = orc.residual_dense(A, Wr, Hr)
    # ||A||^2 - 2 <A H^T, W> + <H H^T, W^T W>: three sums of relative error 2^-21 or less that cancel
    assert abs(got ** 2 - want ** 2) <= 1e-6 * float((A.astype(np.float64) ** 2).sum()) + 1e-5 * want ** 2
