"""Gram matrices of up to 16 factors in one launch: row counts around the shares and the line to the other kernels (131072), through
sparse runs against the oracle; a run cut in two gives the same bits."""
import numpy as np
import pytest

from oracle import nmf_oracle as orc

EPS = 1e-16


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", [(1, 5, 3), (63, 65, 1), (64, 129, 16), (1000, 4097, 15), (65536, 70, 12), (65537, 90, 16), (131072, 60, 5),
                                   (131073, 60, 9)])
def test_sparse_runs(m, n, k):
    import torch

    import paper_2202_09518_amd as nmf
    r = np.random.default_rng(m + n + k)
    per = 3
    rowptr = np.arange(0, m * per + 1, per, dtype=np.int64)
    col = r.integers(0, n, m * per).astype(np.int32)
    vals, W, H = (r.random(s, dtype=np.float32) for s in (m * per, (m, k), (k, n)))
    dev = [torch.from_numpy(x).cuda() for x in (rowptr, col, vals)]

    def run(*iters):
        Wd, Hd = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
        for it in iters:
            nmf.nmf_mu_csr(*dev, m, n, m * per, k, Wd, Hd, it, EPS)
        torch.cuda.synchronize()
        return Wd, Hd

    (Wd, Hd), (W2, H2) = run(3), run(2, 1)
    assert torch.equal(Wd, W2) and torch.equal(Hd, H2)
    Wr, Hr = orc.mu_csr(rowptr, col, vals, m, n, W, H, 3, float(np.float32(EPS)))
    # three updates of each factor, sums of one sign: a few roundings of 2^-24 per sum
    assert orc.rel_fro(Wd.cpu().numpy(), Wr) < 3e-6 and orc.rel_fro(Hd.cpu().numpy(), Hr) < 3e-6
