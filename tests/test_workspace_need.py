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


def _step(m, n, r, dtype):
    """R, N and, for a bf16 tensor with rows <= cols, rows % 64 == 0 and cols % 8 != 0, the padded copy of G."""
    k, l, s = min(m, n), max(m, n), 2 if dtype == torch.bfloat16 else 4
    pad = (l + 7) // 8 * 8 if m <= n and s == 2 and n % 8 and m % 64 == 0 else l
    return _up(4 * r * pad) + _up(s * r * l) + (_up(s * k * pad) if pad != l else 0)


def _init_status(m, n, r, dtype, nbytes):
    """Status of galore_init for a tensor of this shape and a second one whose projector is wrong: SHAPE where the first was
    accepted with this workspace, before anything touches a device."""
    fake = lambda rows, cols, dt: gb.shape_desc(rows, cols, dt, data=4096)
    k, l = min(m, n), max(m, n)
    mom = (r, l) if m <= n else (l, r)
    none = gb.galore_tensor(None, 0, 0, 0, gb.GALORE_F32)
    good = gb.galore_state(fake(k, r, dtype), fake(*mom, torch.float32), fake(*mom, torch.float32), fake(r, k, dtype), none, none)
    wrong = gb.galore_state(fake(k + 1, r, dtype), fake(*mom, torch.float32), fake(*mom, torch.float32), fake(r, k, dtype), none, none)
    w = gb.shape_desc(m, n, dtype)
    with pytest.raises(gb.GaloreError) as e:
        gb.galore_init(gb.make_hparams(r), [w, w], [good, wrong], 4096, nbytes, stream=gb.ctypes.c_void_p(None))
    return e.value.status


# projections of 1 to 223 tiles of 64 x 64 over contractions of 512 and more, which may be cut into pieces, and their neighbours
@pytest.mark.parametrize("m,n,r", [(512, 14272, 64), (14272, 512, 64), (512, 14273, 64), (511, 14272, 64), (1024, 7100, 128), (512, 4097, 256),
                                   (2048, 14003, 8), (8192, 8192, 8), (640, 40000, 8), (768, 2048, 256)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_a_workspace_for_one_copy_of_the_projected_gradient_is_accepted(m, n, r, dtype):
    need = max(_step(m, n, r, dtype), _householder_refresh(min(m, n), r))
    assert _init_status(m, n, r, dtype, need) == 2
    if _step(m, n, r, dtype) > _householder_refresh(min(m, n), r):
        assert _init_status(m, n, r, dtype, need - 256) == 6
    # and what galore_workspace_bytes asks for has room for the pieces
    assert gb.galore_workspace_bytes(gb.make_hparams(r), [gb.shape_desc(m, n, dtype)]) <= need + 3 * _up(4 * r * (max(m, n) + 7))
