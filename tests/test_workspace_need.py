"""Workspace sizes (host arithmetic only): a buffer that was sized for the Householder path of the refresh serves the
Cholesky path as well, at every rank."""
import pytest
import torch

from paper_2403_03507_amd import binding as gb


def _up(x):
    return (x + 255) // 256 * 256


def _householder_refresh(k, r):
    """The Householder path's working set for one tensor with short side k, as laid out in csrc/refresh.hip."""
    panels = (r + 31) // 32
    split = k % 32 == 0 and k >= 512 and r >= 8
    table = 8 + 16 * 168  # descriptors of 16 tensors
    sizes = [4 * k * k, 4 * k * r, 4 * k * r, 4 * r * r, 4 * r * r, 4 * r * r, 4 * r, 4 * r, 4 * 32 * panels * k, 4 * 1024 * panels, 8 * 4096,
             (panels + 1) * 4 * 4096, 4 * r, 4 * r, 44, table, 12 * k * k if split else 0, 12 * k * r if split else 0]
    return sum(_up(s) for s in sizes)


def _query(k, r, dtype):
    return gb.galore_workspace_bytes(gb.make_hparams(r), [gb.shape_desc(k, k, dtype)])


@pytest.mark.parametrize("k", [8, 31, 32, 33, 64, 100, 128, 255, 256, 257, 300, 512, 777, 1024])
def test_refresh_fits_what_the_householder_path_takes(k):
    ranks = sorted({r for r in (1, 2, 7, 8, 31, 32, 33, 63, 65, 96, 127, 128, 129, 160, 200, 225, 254, 255, 256, k // 4, k // 2, k - 1, k) if 1 <= r <= min(k, 256)})
    for r in ranks:
        for dtype in (torch.float32, torch.bfloat16):
            # a square tensor's step takes less than its refresh: R and N of k r entries each, up to four times R
            assert _query(k, r, dtype) <= max(_householder_refresh(k, r), _up(16 * k * r) + _up(4 * k * r)), (k, r)


@pytest.mark.parametrize("k,r", [(300, 257), (512, 384), (1024, 1024), (777, 500)])
def test_higher_ranks_take_the_householder_path_and_its_size(k, r):
    assert _query(k, r, torch.float32) == _householder_refresh(k, r)
