"""Row splits of the W^T A pass (host function): enough workgroups for wide matrices, no more than are resident at once
where several splits fit, and never more partial results than the rounded-up count, which workspaces are sized for."""
import ctypes

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
