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


def _context_in(opt, buf, nbytes):
    """The optimizer's context once more, in the first nbytes of buf."""
    none = gb.galore_tensor(None, 0, 0, 0, gb.GALORE_F32)
    states = [gb.galore_state(gb.desc(p), gb.desc(m), gb.desc(v), gb.desc(pt), none, none) for p, m, v, pt in zip(opt.proj, opt.M, opt.V, opt.proj_t)]
    ctx = gb.galore_init(opt.hp, [gb.shape_desc(m, n, dt) for (m, n), dt in zip(opt.shapes, opt.dtypes)], states, buf.data_ptr(), nbytes)
    opt.close()
    opt.ctx, opt.workspace = ctx, buf


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("copies", [0, 1.5, 2.9, 8])
def test_step_whose_k_pieces_get_what_room_there_is(dtype, copies):
    # Three pieces that leave as slabs of R where the workspace has room for them beside R and N, else fewer; the results agree to the fp32
    # rounding of R.  fp32: 175 tiles of 64 x 64, too few for a workgroup to add its pieces and too many for 16 pieces in one; bf16:
    # 223 tiles over a contraction too long for K groups at this rank.  Shapes whose step takes more than their refresh.
    m, n, r = (512, 11200, 64) if dtype == "f32" else (1027, 14272, 64)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(3)
    W0 = (0.02 * torch.randn(m, n, generator=g, device="cuda")).to(tdt)
    G = [torch.randn(m, n, generator=g, device="cuda").to(tdt) for _ in range(2)]
    P = torch.linalg.qr(torch.randn(m, r, generator=g, device="cuda"))[0]
    room = gb.galore_workspace_bytes(gb.make_hparams(r), [gb.shape_desc(m, n, tdt)])
    least = 4 * r * n + W0.element_size() * r * n   # R once, and N: more than the refresh needs
    out = []
    for nbytes in (8 * room, None):
        W = W0.clone()
        opt = gb.GaLore([W], r, update_gap=1000, auto_refresh=False)
        one = nbytes is None and copies < 1   # room for one R: a whole contraction
        if nbytes is None:
            nbytes = int(least + copies * 4 * r * n) // 256 * 256
        buf = torch.full((nbytes + 4096,), 0x55, dtype=torch.uint8, device="cuda")
        _context_in(opt, buf, nbytes)
        opt.proj[0].copy_(P)
        # moments of earlier steps: after zero moments N is the sign of R, which rounding decides where R is next to zero
        opt.M[0].normal_(generator=torch.Generator(device="cuda").manual_seed(4))
        opt.V[0].fill_(1.0)
        opt.set_step(0, 1000)
        gb.galore_profile_start(opt.ctx)
        for x in G:
            opt.step([W], [x], 1e-3)
        stages = gb.galore_profile_stop(opt.ctx)
        assert stages["adam"][1] == (0 if one else 2)   # an R this large runs Adam in its projection unless its pieces leave as slabs
        torch.cuda.synchronize()
        assert bool((buf[nbytes:] == 0x55).all())
        out.append((to64(W), to64(opt.M[0]), to64(opt.V[0])))
        opt.close()
    assert relF(out[1][1], out[0][1]) <= 1e-6 and relF(out[1][2], out[0][2]) <= 1e-6   # sums of 512 (bf16 1027) fp32 terms in another order: 2e-7
    # all three pieces in either workspace: the same bits; fewer in the smaller one: other roundings somewhere in 900 000 entries
    assert np.array_equal(out[1][1], out[0][1]) == (copies > 2)
    if dtype == "f32":
        # 1e-6 of an update that is itself under 1e-2 of W, and the rounding of W: half an ulp, 6e-8 at most, in each of two steps
        assert relF(out[1][0], out[0][0]) <= 1.3e-7
    else:
        assert np.mean(out[1][0] != out[0][0]) <= 1e-3   # a weight on the other side of a rounding boundary
