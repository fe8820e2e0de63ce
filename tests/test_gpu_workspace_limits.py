"""Workspaces of exactly the size that a call states or asks for: accepted, and the results are those of any other size."""
import numpy as np
import pytest
import torch

from helpers import f32, relF, to64
from oracle import galore_oracle as orc
from paper_2403_03507_amd import binding as gb

pytestmark = pytest.mark.gpu


def _adafactor_bytes(rows, cols):
    """What include/galore.h states for galore_adafactor."""
    cb, rb = (cols + 255) // 256, (rows + 31) // 32
    return 4 * (cb * rows + rb * (cols + cb) + 4)


@pytest.mark.parametrize("shape", [(1, 1), (256, 40), (1024, 300), (1025, 300), (4097, 257), (17000, 8)])
def test_adafactor_stage_in_the_documented_workspace(shape):
    # up to 1024 rows the row statistics have 4 partial totals, beyond that more (67 at 17000)
    rows, cols = shape
    g = torch.Generator().manual_seed(rows)
    R = torch.randn(rows, cols, generator=g)
    M, row, col = torch.zeros(rows, cols, device="cuda"), torch.zeros(rows, device="cuda"), torch.zeros(cols, device="cuda")
    N = torch.empty(rows, cols, device="cuda")
    need = _adafactor_bytes(rows, cols)
    buf = torch.full((need + 1024,), 0x7F, dtype=torch.uint8, device="cuda")
    gb.galore_adafactor(R.cuda(), M, row, col, N, f32(0.9), 1, buf[:need])
    torch.cuda.synchronize()
    assert bool((buf[need:] == 0x7F).all())  # nothing is written beyond what was handed over
    Mo, ro, co = np.zeros((rows, cols)), np.zeros(rows), np.zeros(cols)
    No = orc.adafactor(to64(R), Mo, ro, co, f32(0.9), 1)
    # fp32 sums of up to 17000 terms against 64 bits, as in test_gpu_adafactor.py
    assert relF(to64(N), No) <= 1e-5 and relF(to64(row), ro) <= 1e-5 and relF(to64(col), co) <= 1e-5
    with pytest.raises(gb.GaloreError) as e:
        gb.galore_adafactor(R.cuda(), M, row, col, N, f32(0.9), 2, buf[:need - 4])
    assert e.value.status == 6
