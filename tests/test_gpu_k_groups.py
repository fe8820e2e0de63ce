"""K pieces added, and updated, in the workgroup that formed them: edges of tiles and of pieces, 2, 3 and 4 pieces, both sides, against 64 bits."""
import pytest
import torch

from helpers import relF, strided, to64
from paper_2403_03507_amd import binding as gb

pytestmark = pytest.mark.gpu


# short sides of 2 pieces (512 .. 767), 3 (768 .. 1023), 4 (1024 and, above rank 128, up to 2048), none of them a multiple of the pieces' K step but two
@pytest.mark.parametrize("k,r", [(512, 64), (513, 65), (767, 8), (768, 128), (1023, 9), (1024, 130), (1025, 200), (2047, 129)])
@pytest.mark.parametrize("extra,pad", [(0, 0), (64, 0), (77, 3)])
@pytest.mark.parametrize("left", [True, False])
def test_pieces_in_one_workgroup(k, r, extra, pad, left):
    g = torch.Generator(device="cuda").manual_seed(k + r + extra)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda")
    m, n = (k, k + extra) if left or not extra else (k + extra, k)
    W0, G = (0.02 * rand(m, n)).to(torch.bfloat16), rand(m, n).to(torch.bfloat16)
    W = strided(W0, pad) if pad else W0.clone()
    opt = gb.GaLore([W], r, update_gap=1 << 30, beta2=0.99)
    opt.proj[0].copy_(torch.linalg.qr(rand(k, r))[0])
    opt.M[0].copy_(0.1 * rand(*opt.M[0].shape))
    opt.V[0].copy_(0.1 + 0.1 * rand(*opt.V[0].shape).square())   # away from zero: N is as good as R
    opt.set_step(0, 7)
    M0, V0, P = opt.M[0].double(), opt.V[0].double(), opt.proj[0].double()
    R = P.t() @ G.double() if m <= n else G.double() @ P
    opt.step([W], [strided(G, pad) if pad else G], 1e-2)
    b1, b2 = float(torch.tensor(0.9)), float(torch.tensor(0.99))
    M, V = b1 * M0 + (1 - b1) * R, b2 * V0 + (1 - b2) * R * R
    assert relF(to64(opt.M[0]), to64(M)) <= 1e-5 and relF(to64(opt.V[0]), to64(V)) <= 1e-5
    N = (M / (1 - b1 ** 8)) / ((V / (1 - b2 ** 8)).sqrt() + 1e-8)
    want = W0.double() - 1e-2 * 0.25 * (P @ N if m <= n else N @ P.t())
    # half an ulp of W where it is stored, and N rounded to bf16 (half an ulp, up to 2^-8 of an entry) on its way there; 2 % for sums in fp32
    ulp = 2.0 ** (torch.floor(torch.log2(torch.maximum(want.abs(), W0.double().abs()).clamp_min(2.0 ** -126))) - 7)
    n_err = 2.0 ** -8 * 1e-2 * 0.25 * (P.abs() @ N.abs() if m <= n else N.abs() @ P.abs().t())
    assert bool(((W.double() - want).abs() <= 1.02 * (0.5 * ulp + n_err)).all())
    assert not torch.equal(W, W0)
    opt.close()


# fp32: 32 x 32 tiles over 16 wavefronts; short sides that end inside a K step, ranks and long sides that end inside a tile
@pytest.mark.parametrize("k,r", [(512, 64), (513, 33), (575, 8), (640, 128), (1000, 4), (1024, 97)])
@pytest.mark.parametrize("extra,pad", [(0, 0), (64, 0), (77, 3)])
@pytest.mark.parametrize("left", [True, False])
def test_fp32_contraction_in_one_workgroup(k, r, extra, pad, left):
    g = torch.Generator(device="cuda").manual_seed(k + r + extra)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda")
    m, n = (k, k + extra) if left or not extra else (k + extra, k)
    W0, G = 0.02 * rand(m, n), rand(m, n)
    W = strided(W0, pad) if pad else W0.clone()
    opt = gb.GaLore([W], r, update_gap=1 << 30, beta2=0.99)
    opt.proj[0].copy_(torch.linalg.qr(rand(k, r))[0])
    opt.M[0].copy_(0.1 * rand(*opt.M[0].shape))
    opt.V[0].copy_(0.1 + 0.1 * rand(*opt.V[0].shape).square())
    opt.set_step(0, 7)
    M0, V0, P = opt.M[0].double(), opt.V[0].double(), opt.proj[0].double()
    R = P.t() @ G.double() if m <= n else G.double() @ P
    opt.step([W], [strided(G, pad) if pad else G], 1e-2)
    b1, b2 = float(torch.tensor(0.9)), float(torch.tensor(0.99))
    M, V = b1 * M0 + (1 - b1) * R, b2 * V0 + (1 - b2) * R * R
    # Every entry: the K steps of 64 are dealt to 4 groups, a wavefront sums 16 products of each of its group's steps, and the 16 sums are added: so many roundings at
    # most, of 2^-24 of the sum of the products' absolute values each, and a few of M and V themselves
    bound = 2.0 ** -24 * (16 * -(--(-k // 64) // 4) + 15) * (P.abs().t() @ G.double().abs() if m <= n else G.double().abs() @ P.abs())
    dM, dV = (1 - b1) * bound + 2.0 ** -22 * (M0.abs() + R.abs()), (1 - b2) * 2 * R.abs() * bound + 2.0 ** -21 * (V0 + R * R)
    assert bool(((opt.M[0].double() - M).abs() <= dM).all()) and bool(((opt.V[0].double() - V).abs() <= dV).all())
    N = (M / (1 - b1 ** 8)) / ((V / (1 - b2 ** 8)).sqrt() + 1e-8)
    want = W0.double() - 1e-2 * 0.25 * (P @ N if m <= n else N @ P.t())
    # half an ulp of W where it is stored, what M and V may be off by in N, and r products summed in fp32
    ulp = 2.0 ** (torch.floor(torch.log2(torch.maximum(want.abs(), W0.double().abs()).clamp_min(2.0 ** -126))) - 23)
    dN = N.abs() * (dV / V) + dM / (1 - b1 ** 8) / (V / (1 - b2 ** 8)).sqrt() + 2.0 ** -24 * (r + 16) * N.abs()
    n_err = 1e-2 * 0.25 * (P.abs() @ dN if m <= n else dN @ P.abs().t())
    assert bool(((W.double() - want).abs() <= 0.51 * ulp + n_err).all())
    assert not torch.equal(W, W0)
    opt.close()


# short side, rank, pieces: the same bits as the product of each piece, the sums in slab order, Adam and the weight update as calls of their own
@pytest.mark.parametrize("k,r,pieces", [(512, 64, 2), (700, 33, 2), (768, 128, 3), (1000, 40, 3), (1024, 96, 4), (1100, 200, 4), (2048, 136, 4)])
@pytest.mark.parametrize("left", [True, False])
def test_pieces_in_one_workgroup_have_the_bits_of_slabs(k, r, pieces, left):
    l = k + 65
    g = torch.Generator(device="cuda").manual_seed(k + r)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda")
    m, n = (k, l) if left else (l, k)
    W, G = (0.02 * rand(m, n)).to(torch.bfloat16), rand(m, n).to(torch.bfloat16)
    opt = gb.GaLore([W], r, update_gap=1 << 30, auto_refresh=False)
    opt.proj[0].copy_(torch.linalg.qr(rand(k, r))[0])
    opt.M[0].copy_(0.1 * rand(*opt.M[0].shape))
    opt.V[0].copy_(0.1 + 0.1 * rand(*opt.V[0].shape).square())
    opt.set_step(0, 7)
    M, V, W1 = opt.M[0].clone(), opt.V[0].clone(), W.clone()
    Pt = opt.proj[0].t().contiguous()
    steps, R = -(-k // 128), None   # K steps of 128
    for s in range(pieces):
        part = slice(s * steps // pieces * 128, min((s + 1) * steps // pieces * 128, k))
        one = torch.empty_like(M)
        gb.galore_project(Pt[:, part], G[part] if left else G[:, part], one)
        R = one if R is None else R + one
    N = torch.empty(l, r, dtype=torch.bfloat16, device="cuda")
    gb.galore_adam(R, M, V, N, left, 0.9, 0.999, 1e-8, 8)
    gb.galore_project_back(opt.proj[0], N, W1, 1e-2, 0.25)
    gb.galore_profile_start(opt.ctx)
    opt.step([W], [G], 1e-2)
    assert gb.galore_profile_stop(opt.ctx)["adam"][1] == 0
    assert torch.equal(opt.M[0], M) and torch.equal(opt.V[0], V) and torch.equal(W, W1)
    opt.close()


# A call takes the groups where they spare its Adam launch: one number of pieces (bf16), nothing in slabs, no R small enough for Adam to stay a launch
@pytest.mark.parametrize("dtype,rank,shapes,adam", [
    ("bf16", 32, [(512, 640), (600, 520)], 0), ("bf16", 32, [(512, 640), (768, 1024)], 1), ("bf16", 64, [(1024, 1024), (2304, 2304)], 1),
    ("bf16", 64, [(768, 768), (200, 1000)], 1), ("bf16", 66, [(768, 768), (200, 1000)], 0), ("bf16", 8, [(768, 768), (7, 40)], 1),
    ("f32", 32, [(512, 640), (1100, 600)], 0), ("f32", 32, [(512, 640), (2304, 2304)], 1), ("f32", 64, [(512, 640)] + [(1024, 1024)] * 4, 1),
    ("f32", 64, [(768, 768), (200, 1000)], 1), ("f32", 66, [(768, 768), (200, 1000)], 0)])
def test_calls_that_take_the_groups(dtype, rank, shapes, adam):
    rank = min(rank, min(min(s) for s in shapes))
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator(device="cuda").manual_seed(rank)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda").to(td)
    W, G = [0.02 * rand(*s) for s in shapes], [rand(*s) for s in shapes]
    opt = gb.GaLore(W, rank, update_gap=1 << 30, auto_refresh=False)
    for p in opt.proj:
        p.copy_(rand(*p.shape) / 16)
    gb.galore_profile_start(opt.ctx)
    opt.step(W, G, 1e-3)
    assert gb.galore_profile_stop(opt.ctx)["adam"][1] == adam
    for i, (m, n) in enumerate(shapes):
        a, b = (opt.proj[i].t(), G[i]) if m <= n else (G[i], opt.proj[i])
        R, scale = a.double() @ b.double(), a.double().abs() @ b.double().abs()
        # fp32 sums of min(m, n) products, whatever their order
        assert bool(((opt.M[i].double() - (1 - float(torch.tensor(0.9))) * R).abs() <= 0.1 * 2.0 ** -24 * (min(m, n) + 8) * scale).all()), i
    opt.close()
