"""||A - W H||_F by the fp32 streaming kernel: edges of its 32-row tiles, groups of four tiles, 256-column
slabs and factor steps, against the float64 oracle."""
import numpy as np
import pytest

from oracle import nmf_oracle as orc


@pytest.mark.gpu
@pytest.mark.parametrize("m,n", [(2017, 8200), (65541, 68), (65536, 4), (16385, 1000), (2304, 8448)])
@pytest.mark.parametrize("k", [1, 8, 9, 15, 17, 24, 25, 31, 33, 48, 49, 64])
@pytest.mark.parametrize("noise", [0.1, 1e-3])
def test_objective_of_streamed_sizes(m, n, k, noise):
    import torch

    import paper_2202_09518_amd as nmf
    r = np.random.default_rng(m + n + k)
    W, H = r.random((m, k), dtype=np.float32), r.random((k, n), dtype=np.float32)
    A = (W @ H * (np.float32(1) + np.float32(noise) * r.random((m, n), dtype=np.float32))).astype(np.float32)
    got = nmf.nmf_residual_dense(torch.from_numpy(A).cuda(), m, n, k, torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda())
    want = orc.residual_dense(A, W, H)
    # A - W H: at most 64 roundings of 2^-24 each per product of one sign, against a difference of noise / 2
    # on average: relative error of the norm below 64 2^-24 / noise
    assert abs(got - want) <= 64 * 2.0 ** -24 / noise * want
