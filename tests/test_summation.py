"""Long sums of partial results: no value may pass through a long chain of fp32 roundings."""
import numpy as np
import pytest

from oracle import nmf_oracle as orc

EPS = 1e-16


# 65536 x 512: 256 partial results of W^T A and as many of W^T W, 32 of H H^T; 16384 x 2048: 256 of W^T W that a pass
# adds up, 32 of H H^T that a launch adds up
@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", [(65536, 512, 32), (65536, 512, 16), (16384, 2048, 32), (16384, 2048, 64)])
def test_one_iteration_of_long_factors(m, n, k):
    import torch

    import paper_2202_09518_amd as nmf
    r = np.random.default_rng(m + n + k)
    A, W, H = r.random((m, n), dtype=np.float32), r.random((m, k), dtype=np.float32), r.random((k, n), dtype=np.float32)
    Wd, Hd = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
    nmf.nmf_mu_dense(torch.from_numpy(A).cuda(), m, n, k, Wd, Hd, 1, EPS)
    Wr, Hr = orc.mu_dense(A, W, H, 1, float(np.float32(EPS)))
    # H: numerator, denominator, product and quotient, each within about one rounding of 2^-24 where its long sum goes
    # through few of them; four independent ones come to 2^-23.  A chain of 64 Gram tiles or 256 partial products
    # adds (64 / 12)^(1/2) 2^-24 and more by itself.
    assert orc.rel_fro(Hd.cpu().numpy(), Hr) < 2.0 ** -23
    # W adds the same for its own update, with the error of H in common
    assert orc.rel_fro(Wd.cpu().numpy(), Wr) < 1.5 * 2.0 ** -23
