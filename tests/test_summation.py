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


# a column of one value: every product has the same low bits, and an accumulator that takes in too many of them loses
# the same share of each
@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", [(4000, 516, 50), (4000, 4004, 64), (20011, 9996, 50)])
def test_products_with_columns_of_one_value(m, n, k):
    import torch

    import paper_2202_09518_amd as nmf
    r = np.random.default_rng(m + n + k)
    A = np.broadcast_to(r.random((1, n), dtype=np.float32), (m, n)).copy()
    W = r.random((m, k), dtype=np.float32)
    P = torch.empty((k, n), device="cuda")
    nmf.nmf_wta_dense(torch.from_numpy(A).cuda(), m, n, k, torch.from_numpy(W).cuda(), P)
    torch.cuda.synchronize()
    # few row splits (16, 8, 12), whose sum adds little: the float64 result to two roundings of 2^-24, one of the result,
    # and from the sums of up to 96 terms a loss of
    # the size of one
    assert orc.rel_fro(P.cpu().numpy(), W.astype(np.float64).T @ A.astype(np.float64)) < 2.0 ** -23


@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", [(2003, 4001, 64), (4001, 2003, 64), (5001, 3001, 40)])
def test_misaligned_matrices_at_33_to_64_factors(m, n, k):
    """One iteration on the padded copies, whose products are summed from pieces."""
    import torch

    import paper_2202_09518_amd as nmf
    r = np.random.default_rng(m + n + k)
    A, W, H = r.random((m, n), dtype=np.float32), r.random((m, k), dtype=np.float32), r.random((k, n), dtype=np.float32)
    Wd, Hd = torch.from_numpy(W).cuda(), torch.from_numpy(H).cuda()
    nmf.nmf_mu_dense(torch.from_numpy(A).cuda(), m, n, k, Wd, Hd, 1, EPS)
    Wr, Hr = orc.mu_dense(A, W, H, 1, float(np.float32(EPS)))
    # with the products on the fp32 matrix instruction 7.7e-8 to 9.0e-8: one and a half roundings of 2^-24
    assert orc.rel_fro(Hd.cpu().numpy(), Hr) < 1.5 * 2.0 ** -24
    assert orc.rel_fro(Wd.cpu().numpy(), Wr) < 1.5 * 2.0 ** -24


# few splits and a whole chain of each pass: W^T A of the row plan, A H^T of the row plan, W^T A of the one-pass plan
@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k,same", [(4096, 33024, 32, "columns"), (12288, 4096, 20, "rows"), (300000, 132, 16, "columns")])
def test_up_to_32_factors_and_one_value_per_column_or_row(m, n, k, same):
    import torch

    import paper_2202_09518_amd as nmf
    g = torch.Generator(device="cuda")
    g.manual_seed(m + n)
    W, H = torch.rand((m, k), generator=g, device="cuda"), torch.rand((k, n), generator=g, device="cuda")
    A = torch.rand((1, n) if same == "columns" else (m, 1), generator=g, device="cuda").expand(m, n).contiguous()
    Wd, Hd = W.clone(), H.clone()
    nmf.nmf_mu_dense(A, m, n, k, Wd, Hd, 1, EPS)
    A, W, H = A.double(), W.double(), H.double()
    # the factor whose long sums are over the equal values, W with the H that the library has
    if same == "columns":
        Wt = W.t().contiguous()
        got, want = Hd, H * (Wt @ A) / ((Wt @ W) @ H + EPS)
    else:
        Ht = Hd.double().t().contiguous()
        got, want = Wd, W * (A @ Ht) / (W @ (Hd.double() @ Ht) + EPS)
    # four roundings of 2^-24 as above, and a loss of two more in sums of up to 256 equal terms
    assert ((got - want).norm() / want.norm()).item() < 2.0 ** -22
