"""How an fp32 projection of few tiles sums its contraction: in K pieces, whose sums are added."""
import pytest
import torch

from paper_2403_03507_amd import binding as gb

pytestmark = pytest.mark.gpu


def _one_large_product(k, l, rank, left, moments):
    """M (or its scales) over 1 - beta1 after one step from zero moments, and the sum in 64 bits: every entry of R is 1 + (k - 1) products just
    under half the spacing of fp32 numbers below 2, taken two at a time.  A single fp32 chain that starts at the 1 loses all of them."""
    small = 0.99 * 2.0 ** -25
    G = torch.full((k, l), small, device="cuda")
    G[0] = 1.0
    W = torch.zeros((k, l) if left else (l, k), device="cuda")
    opt = gb.GaLore([W], rank, update_gap=1 << 30, auto_refresh=False, moments=moments)
    opt.proj[0].fill_(1.0)
    opt.step([W], [G if left else G.t().contiguous()], 1e-3)
    torch.cuda.synchronize()
    b1 = float(torch.tensor(0.9))
    got = (opt.M_scale[0] if moments == "q8" else opt.M[0]).double() / (1 - b1)
    opt.close()
    return got, 1.0 + (k - 1) * float(G[1, 0])


def _chain(k, pieces):
    """The most products that one of `pieces` adds one after the other: K steps of 64."""
    steps = -(-k // 64)
    return 64 * max((s + 1) * steps // pieces - s * steps // pieces for s in range(pieces))


# 180 to 223 tiles of 64 x 64: three pieces.  8-bit moments: a row's blocks of 256 have the block maximum (1 - beta1) R as their scale
@pytest.mark.parametrize("k,l,rank", [(512, 12544, 64), (1024, 13312, 64), (600, 6400, 128)])
def test_pieces_of_a_projection_with_8_bit_moments(k, l, rank):
    got, want = _one_large_product(k, l, rank, True, "q8")
    # a chain of c products and the sums of the pieces, 2^-24 of the sum each; (1 - beta1) R in two roundings and its own division here
    assert float((got - want).abs().max()) <= want * 2.0 ** -24 * (_chain(k, 3) + 2 + 4)


@pytest.mark.parametrize("k,l,rank", [(512, 12544, 64), (1024, 13312, 64), (600, 6399, 127), (1537, 4100, 192)])
@pytest.mark.parametrize("left", [True, False])
def test_pieces_of_a_projection_with_adam_in_it(k, l, rank, left):
    got, want = _one_large_product(k, l, rank, left, "f32")
    assert float((got - want).abs().max()) <= want * 2.0 ** -24 * (_chain(k, 3) + 2 + 4)


@pytest.mark.parametrize("k,l,rank", [(512, 12544, 64), (1024, 12803, 63), (1537, 4100, 192)])
@pytest.mark.parametrize("left", [True, False])
@pytest.mark.parametrize("moments", ["f32", "q8"])
def test_a_workgroup_adds_pieces_as_slabs_are_added(k, l, rank, left, moments):
    # Beside a tensor whose R is small the pieces are slabs and Adam is a launch of its own; alone a workgroup adds them.  Same bits.
    if moments == "q8":
        if not left:
            rank = 256
            l = 3200   # 4 x 50 tiles
        l = l // 256 * 256
    g = torch.Generator(device="cuda").manual_seed(k)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda")
    shapes = [(k, l) if left else (l, k), (rank, 256)]
    W0, G = [0.02 * rand(*s) for s in shapes], [rand(*s) for s in shapes]
    P, out, adam = torch.linalg.qr(rand(k, rank))[0], [], []
    for count in (1, 2):
        W = [w.clone() for w in W0[:count]]
        opt = gb.GaLore(W, rank, update_gap=1 << 30, auto_refresh=False, moments=moments, workspace_factor=2)
        opt.proj[0].copy_(P)
        gb.galore_profile_start(opt.ctx)
        for _ in range(2):
            opt.step(W, G[:count], 1e-3)
        adam.append(gb.galore_profile_stop(opt.ctx)["adam"][1])
        torch.cuda.synchronize()
        out.append([W[0], opt.M[0].clone(), opt.V[0].clone()] + ([opt.M_scale[0].clone(), opt.V_scale[0].clone()] if moments == "q8" else []))
        opt.close()
    assert adam == ([0, 2] if moments == "f32" else [2, 2])
    assert all(torch.equal(a, b) for a, b in zip(*out))
    assert not torch.equal(out[0][0], W0[0])


# short side, rank, side, whether the pieces of 184 tiles add up in place (Adam in that launch) or leave as slabs
@pytest.mark.parametrize("k,rank,left,in_place", [(2047, 128, True, True), (2048, 128, True, False), (2049, 64, True, True), (3072, 65, True, False),
                                                  (2048, 128, False, True), (2049, 128, False, False), (3072, 64, False, False)])
def test_long_contractions_leave_slabs(k, rank, left, in_place):
    l = 184 // -(-rank // 64) * 64
    g = torch.Generator(device="cuda").manual_seed(k)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda")
    m, n = (k, l) if left else (l, k)
    W, G = 0.02 * rand(m, n), rand(m, n)
    opt = gb.GaLore([W], rank, update_gap=1 << 30, auto_refresh=False)
    opt.proj[0].copy_(torch.linalg.qr(rand(k, rank))[0])
    gb.galore_profile_start(opt.ctx)
    opt.step([W], [G], 1e-3)
    assert gb.galore_profile_stop(opt.ctx)["adam"][1] == (0 if in_place else 1)
    a, b = (opt.proj[0].t(), G) if left else (G, opt.proj[0])
    R, scale = a.double() @ b.double(), a.double().abs() @ b.double().abs()
    b1 = float(torch.tensor(0.9))
    # entries of R: a chain of products and the sums of the pieces, 2^-24 of the sum of absolute values each; M in two roundings
    assert bool(((opt.M[0].double() - (1 - b1) * R).abs() <= (1 - b1) * 2.0 ** -24 * (_chain(k, 3) + 2 + 4) * scale).all())
    opt.close()
