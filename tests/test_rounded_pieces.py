"""The cut of the streamed operand: three bf16 pieces by rounding to nearest even, six products per term.

The CPU tests check the arithmetic that the kernels rely on, with exact rationals on pieces produced here with
integer arithmetic; they say nothing about the kernels' own cut.  That is what the GPU tests are for: the passes
at the edges of the cut (values that would round to infinity, one repeated value, exact powers of two, zeros), and
on single products, where a wrong piece shows."""
from fractions import Fraction

import numpy as np
import pytest

LARGEST_BF16 = np.uint32(0x7f7f0000)


def rne_bf16(x):
    """float32 -> nearest bf16 (ties to even) as a float32."""
    u = np.asarray(x, dtype=np.float32).view(np.uint32).astype(np.uint64)
    u = (u + 0x7fff + ((u >> 16) & 1)) & 0xffff0000
    return u.astype(np.uint32).view(np.float32)


def rounded_pieces(x):
    x = np.asarray(x, dtype=np.float32)
    h = rne_bf16(x)
    h = np.where(np.isinf(h) & (x > 0), LARGEST_BF16.view(np.float32), h).astype(np.float32)
    r = x - h
    m = rne_bf16(r)
    return h, m, r - m


def truncated_pieces(x):
    x = np.asarray(x, dtype=np.float32)
    h = (x.view(np.uint32) & np.uint32(0xffff0000)).view(np.float32)
    r = x - h
    m = (r.view(np.uint32) & np.uint32(0xffff0000)).view(np.float32)
    return h, m, r - m


def sample(n, seed):
    r = np.random.default_rng(seed)
    x = r.random(n, dtype=np.float32) * np.float32(2.0) ** r.integers(-60, 60, n).astype(np.float32)
    x[:8] = [0.0, 1.0, np.float32(1.0) - np.float32(2.0) ** -24, 3.0e38, 3.395e38,
             np.finfo(np.float32).max, np.float32(1.0) + np.float32(2.0) ** -8, np.float32(255.5)]
    return x.astype(np.float32)


def test_rounded_pieces_are_bf16_sum_exactly_and_are_small():
    x = sample(3000, 11)
    with np.errstate(over="ignore"):
        h, m, l = rounded_pieces(x)
    for p in (h, m, l):
        assert ((p.view(np.uint32) & np.uint32(0xffff)) == 0).all()      # representable as bf16
        assert np.isfinite(p).all()
    for xi, hi, mi, li in zip(x, h, m, l):
        X, H, M, L = (Fraction(float(v)) for v in (xi, hi, mi, li))
        assert H + M + L == X
        # of a held value (above the largest bf16) the middle piece can be 2^-8 (1 + 2^-23) of it
        assert abs(M) * 2 ** 8 <= X * (1 + Fraction(1, 2 ** 23)) and abs(L) * 2 ** 16 <= X


def test_the_three_products_left_out_are_below_2_to_minus_22_and_cancel():
    w, a = sample(3000, 12), sample(3000, 13)
    w, a = w[8:], a[8:]
    pw, pa = truncated_pieces(w), rounded_pieces(a)
    rel = []
    for i in range(w.size):
        left_out = sum(Fraction(float(pw[p][i])) * Fraction(float(pa[q][i])) for p, q in ((1, 2), (2, 1), (2, 2)))
        exact = Fraction(float(w[i])) * Fraction(float(a[i]))
        if exact:
            assert abs(left_out) * 2 ** 22 <= exact
            rel.append(float(left_out / exact))
    rel = np.array(rel)
    # either sign: the mean of the ~3000 terms is within four standard errors of zero, and a term is 2^-25 or less typically
    assert abs(rel.mean()) < 4 * rel.std() / np.sqrt(rel.size)
    assert rel.std() < 2.0 ** -25


@pytest.mark.gpu
@pytest.mark.parametrize("k", [5, 32, 33, 64])
@pytest.mark.parametrize("n", [64, 260, 259])
@pytest.mark.parametrize("kind", ["huge", "constant", "powers", "zeros"])
def test_wta_at_the_edges_of_the_cut(k, n, kind):
    import torch

    import paper_2202_09518_amd as nmf
    m = 200
    r = np.random.default_rng(5 + k + n)
    W = r.random((m, k), dtype=np.float32)
    if kind == "huge":       # between the largest bf16 and the largest float: may not turn into infinity
        A = np.full((m, n), 3.4e38, dtype=np.float32)
        W = W * np.float32(1e-6)
    elif kind == "constant":
        A = np.full((m, n), np.float32(0.1), dtype=np.float32) * np.arange(1, n + 1, dtype=np.float32)
    elif kind == "powers":
        A = np.ldexp(np.ones((m, n), dtype=np.float32), r.integers(-30, 30, (m, n))).astype(np.float32)
    else:
        A = np.where(r.random((m, n)) < 0.5, 0, r.random((m, n))).astype(np.float32)
    P = torch.empty((k, n), device="cuda")
    nmf.nmf_wta_dense(torch.from_numpy(A).cuda(), m, n, k, torch.from_numpy(W).cuda(), P)
    torch.cuda.synchronize()
    want = W.astype(np.float64).T @ A.astype(np.float64)
    got = P.cpu().numpy().astype(np.float64)
    # left-out products 2^-22 of a term at most, sums of 200 terms of one sign in fp32: 200 * 2^-24 at most
    assert np.abs(got - want).max() <= (2.0 ** -22 + 200 * 2.0 ** -24) * np.abs(want).max()


@pytest.mark.gpu
@pytest.mark.parametrize("k", [32, 64])
def test_single_products_hold_to_the_products_left_out(k):
    """One row: every element of W^T A is one product, whose pieces cannot make up for one another."""
    import torch

    import paper_2202_09518_amd as nmf
    n = 1024
    r = np.random.default_rng(k)
    A = (r.random((1, n), dtype=np.float32) * np.float32(2.0) ** r.integers(-30, 30, (1, n))).astype(np.float32)
    W = (r.random((1, k), dtype=np.float32) * np.float32(2.0) ** r.integers(-30, 30, (1, k))).astype(np.float32)
    P = torch.empty((k, n), device="cuda")
    nmf.nmf_wta_dense(torch.from_numpy(A).cuda(), 1, n, k, torch.from_numpy(W).cuda(), P)
    torch.cuda.synchronize()
    want = W.astype(np.float64).T * A.astype(np.float64)
    # 2^-22 of the product left out, and the six that are added in fp32, smallest first: a loss of 2^-23 of the sum at
    # most for each of the last three, the others are below 2^-7 of it
    assert (np.abs(P.cpu().numpy() - want) <= (2.0 ** -22 + 4 * 2.0 ** -23) * want).all()
