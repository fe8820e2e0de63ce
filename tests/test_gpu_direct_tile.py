"""The 128 x 128 tile with direct loads (aligned bf16 operands, one round of tiles) against the register-staged tiles, which an operand at an odd
stride takes: the same additions in the same order, so the same bits."""
import pytest
import torch

from helpers import relF, strided, to64
from paper_2403_03507_amd import binding as gb

pytestmark = pytest.mark.gpu
BF16 = torch.bfloat16


def _rand(seed, *shape):
    return torch.randn(*shape, generator=torch.Generator(device="cuda").manual_seed(seed), device="cuda")


# (k, l, r): 150 to 256 tiles of r x l; last rows and columns of a tile, and one above; the shortest contraction; a rank that fills half its tiles
@pytest.mark.parametrize("k,l,r", [(1024, 4096, 1024), (1024, 4872, 509), (2048, 10104, 129), (2112, 9728, 256), (1088, 19208, 128)])
@pytest.mark.parametrize("left", [True, False])
def test_products_equal_the_other_tiles(k, l, r, left):
    items = -(-l // 128) * -(-r // 128)
    assert 150 <= items <= 256
    P = _rand(r, r, k).to(BF16)
    G = (_rand(l, k, l) if left else _rand(l, l, k)).to(BF16)
    shape = (r, l) if left else (l, r)
    R = [torch.full(shape, float("nan"), device="cuda") for _ in range(2)]
    gb.galore_project(P, G, R[0])
    gb.galore_project(P, strided(G, 3), R[1])
    assert torch.equal(R[0], R[1])
    assert relF(to64(R[0]), to64((P.float() @ G.float() if left else G.float() @ P.float().t()))) <= 1e-5


@pytest.mark.parametrize("m,n,r", [(2048, 2048, 256), (1000, 2744, 320), (2752, 1016, 512)])
def test_weight_update_equals_the_other_tiles(m, n, r):
    assert 160 <= -(-m // 128) * -(-n // 128) <= 256
    k, l = min(m, n), max(m, n)
    P, N, W0 = _rand(1, k, r).to(BF16), _rand(2, l, r).to(BF16), _rand(3, m, n).to(BF16)
    W = [strided(W0, 16), strided(W0, 16)]
    gb.galore_project_back(P, N, W[0], 1e-2, 0.25, 0.01)
    gb.galore_project_back(strided(P, 3), N, W[1], 1e-2, 0.25, 0.01)
    assert torch.equal(W[0], W[1]) and not torch.equal(W[0], W0)
    for w in W:
        assert torch.isnan(w.as_strided((m, 16), w.stride(), n)).all()


@pytest.mark.parametrize("shapes,r", [([(1024, 2736)] * 2 + [(2736, 1024)] + [(1024, 1024)] * 4, 256), ([(1024, 19208)], 128), ([(19208, 1024)], 128)])
def test_adam_in_the_epilogue_equals_the_other_tiles(shapes, r):
    out = []
    for pad in (0, 3):
        W = [(0.02 * _rand(10 + i, m, n)).to(BF16) for i, (m, n) in enumerate(shapes)]
        G = [strided(_rand(30 + i, m, n).to(BF16), pad) if pad else _rand(30 + i, m, n).to(BF16) for i, (m, n) in enumerate(shapes)]
        opt = gb.GaLore(W, r, update_gap=1 << 30)
        for i, (m, n) in enumerate(shapes):
            opt.proj[i].copy_(torch.linalg.qr(_rand(50 + i, min(m, n), r))[0])
            opt.M[i].copy_(0.1 * _rand(70 + i, *opt.M[i].shape))
            opt.V[i].copy_(0.1 * _rand(90 + i, *opt.V[i].shape).square())
            opt.set_step(i, 7)
        for _ in range(2):
            opt.step(W, G, 1e-2)
        torch.cuda.synchronize()
        out.append(W + [x.clone() for x in opt.M + opt.V])
        opt.close()
    for i, (a, b) in enumerate(zip(*out)):
        assert torch.equal(a, b) and torch.isfinite(a.float()).all(), i


def test_two_sided_product_in_pieces():
    # T1 Q is 64 tiles of 128 x 128: four pieces of the contraction, in the place of T1's fp32 form.  T1 is rounded to bf16 on either side; an entry whose
    # two sums fall to either side of a rounding boundary (under one per cent of them) moves by 2^-8: 2^-8 sqrt(0.01) = 4e-4 of R.
    d, r = 4096, 1024
    W, G = (0.02 * _rand(1, d, d)).to(BF16), _rand(2, d, d).to(BF16)
    opt = gb.GaLoreTwoSided(W, r, update_gap=1 << 30)
    opt.t = 7
    opt.P.copy_(torch.linalg.qr(_rand(3, d, r))[0])
    opt.Q.copy_(torch.linalg.qr(_rand(4, d, r))[0])
    opt.M.zero_()
    R = (opt.P.double().t() @ G.double()).to(BF16).double() @ opt.Q.double()
    opt.step(W, G, 1e-3)
    assert relF(to64(opt.M), 0.1 * to64(R)) <= 4e-4


@pytest.mark.parametrize("dtype", [BF16, torch.float32])
@pytest.mark.parametrize("rows,cols,pad", [(64, 64, 0), (65, 127, 0), (1, 200, 0), (200, 1, 0), (4096, 1024, 0), (130, 72, 5), (61, 63, 1)])
def test_transpose(rows, cols, pad, dtype):
    src = _rand(rows + cols, rows, cols).to(dtype)
    dst = torch.full((cols, rows + pad), float("nan"), dtype=dtype, device="cuda")
    gb.galore_transpose(strided(src, pad) if pad else src, dst[:, :rows])
    assert torch.equal(dst[:, :rows], src.t()) and torch.isnan(dst[:, rows:]).all()
