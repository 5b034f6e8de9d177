"""Row splits of the W^T A pass (host function): enough workgroups for wide matrices, no more than are resident at once
where several splits fit, and never more partial results than the rounded-up count, which workspaces are sized for."""
import ctypes
import random

import pytest


def splits(rows, n, k):
    import paper_2202_09518_amd as nmf
    return getattr(nmf.lib(), "_ZN5nmfmu10wta_splitsElli")(ctypes.c_int64(rows), ctypes.c_int64(n), ctypes.c_int(k))


@pytest.mark.parametrize("k,width", [(1, 128), (32, 128), (33, 256), (64, 256)])
def test_splits_of_wide_matrices(k, width):
    for slabs in range(16, 700):
        for n in (slabs * width, slabs * width - width + 1):
            s = splits(16384, n, k)
            assert 1 <= s <= max(1, min(32, -(-512 // slabs)))
            if slabs <= 256:
                assert slabs * s <= 512 and (s == 32 or slabs * (s + 1) > 512)
            elif slabs <= 383:
                assert s == 2
            if slabs >= 128:
                assert splits(256, n, k) == 1       # at least 256 rows per split


def pair_splits(rows, cols, tiles, slices):
    import paper_2202_09518_amd as nmf
    return getattr(nmf.lib(), "_ZN5nmfmu11pair_splitsEllii")(ctypes.c_int64(rows), ctypes.c_int64(cols), ctypes.c_int(tiles), ctypes.c_int(slices))


@pytest.mark.parametrize("rows,cols,want", [(448, 111913, 1), (165, 224000, 1), (300, 400000, 1),      # few rows: every split is a partial
                                            (16384, 8192, 8), (9998, 20011, 3), (20011, 9998, 6)])     # result; large: a full last round
def test_pair_splits(rows, cols, want):
    assert pair_splits(rows, cols, 2, 1) == want


def test_pair_splits_beyond_one_round_stay_cheap():
    r = random.Random(1)
    for _ in range(4000):
        rows, cols = int(2 ** r.uniform(0, 20)), int(2 ** r.uniform(0, 20))
        tiles, slices = r.choice([(2, 1), (2, 2), (2, 4), (4, 1), (4, 3)])
        s = pair_splits(rows, cols, tiles, slices)
        each = -(-(-(-rows // 128)) // s)
        assert s >= 1 and (s - 1) * each * 128 < rows <= s * each * 128      # no empty split
        if -(-cols // 256) * slices * (s - 1) > 512:
            # partial results written and read, against the blocks of the streamed operand
            assert 2 * 32 * tiles * slices * s <= 128 * s * each


# 258 slabs and two splits at both widths; A and A^T just above and below what the cache is taken to hold of two
@pytest.mark.gpu
@pytest.mark.parametrize("m,n,k", [(600, 33024, 32), (600, 66048, 64), (9732, 4096, 33), (9724, 4096, 20)])
def test_one_iteration_at_the_lines(m, n, k):
    import torch

    import paper_2202_09518_amd as nmf
    g = torch.Generator(device="cuda")
    g.manual_seed(m + n)
    A, W, H = (torch.rand(s, generator=g, device="cuda") for s in ((m, n), (m, k), (k, n)))
    Wd, Hd = W.clone(), H.clone()
    nmf.nmf_mu_dense(A, m, n, k, Wd, Hd, 1, 1e-16)
    A, W, H = A.double(), W.double(), H.double()
    Wt = W.t().contiguous()
    H = H * (Wt @ A) / ((Wt @ W) @ H + 1e-16)
    Ht = H.t().contiguous()
    W = W * (A @ Ht) / (W @ (H @ Ht) + 1e-16)
    # numerator, denominator, product and quotient, a rounding of 2^-24 each, for H and again for W
    assert ((Hd - H).norm() / H.norm()).item() < 2.0 ** -22
    assert ((Wd - W).norm() / W.norm()).item() < 2.0 ** -22
