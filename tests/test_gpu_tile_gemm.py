"""The small-tile GEMM (projection with K pieces or with Adam in its epilogue, weight update) against the fp64 oracle,
at the sizes where it can go wrong: one element to either side of a tile, contractions and rows of no multiple of
anything, the smallest sides it takes, the group sizes at which each tile shape and the K pieces are chosen."""
import os
import re

import pytest
import torch

from helpers import check_bf16_weights, f32, relF, strided, to64
from oracle import galore_oracle as orc
from paper_2403_03507_amd import binding as gb
from paper_2403_03507_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _tile(problems, update=False):
    """The tile of a launch of the small-tile GEMM over problems (M, N, K), as csrc/gemm_tile.hip chooses it (the constants are read
    from there: where the rule takes another form, this has to follow)."""
    src = open(os.path.join(os.path.dirname(gb.__file__), "csrc", "gemm_tile.hip")).read()
    padding = re.search(r"if \((\d+) \* items128 > (\d+) \* items64\) items128 = 0;\s*if \((\d+) \* items96 > (\d+) \* items64\) items96 = 0;", src)
    rule = re.search(r"if \(items128 >= (\d+) && \(!update \|\| longest >= (\d+)\)\) return launch<T, 128, 128>\(g, epi, stream\);\s*"
                     r"if \(items96 >= \(update \? (\d+) : (\d+)\)\) return launch<T, 128, 64>", src)
    many128, long_k, many96_update, many96 = (int(x) for x in rule.groups())
    a128, b128, a96, b96 = (int(x) for x in padding.groups())
    assert all(k % 64 for _, _, k in problems)   # nothing for the tile with direct loads

    def count(bm, bn):
        n64, items = (sum(-(-m // x) * -(-n // y) for m, n, _ in problems) for x, y in ((64, 64), (bm, bn)))
        a, b = (a128, b128) if bn == 128 else (a96, b96)
        return 0 if not update and a * items > b * n64 else items
    if count(128, 128) >= many128 and (not update or max(k for _, _, k in problems) >= long_k):
        return 128, 128
    return (128, 64) if count(128, 64) >= (many96_update if update else many96) else (64, 64)


def _projection(shapes, rank):
    return [(rank, n, m) if m <= n else (m, rank, n) for m, n in shapes]


def _update(shapes, rank):
    return [(m, n, rank) for m, n in shapes]


def _steps(shapes, rank, dtype, steps=2, fused=False, pad=0, static=False, adam_launches=None):
    # M, V: fp32 sums of at most a few thousand products, 1e-5 as everywhere; fp32 W: 1e-5; bf16 W per entry.
    # fp32 tensors start from moments as earlier steps leave them: from zero moments the first N is R / (|R| + eps), where an entry of R
    # at rounding distance of zero (1e-9 here, against eps = 1e-8) moves W by up to lr alpha |P column| = 2.5e-3, i.e. 3e-4
    # of |W| = 8.6 for a 130 x 1411 weight; with V of about 1e-5 the same error of R moves N by 1e-6.
    lr = f32(1e-2)
    lay = (lambda t: strided(t, pad)) if pad else (lambda t: t)
    srcs = [wl.GradientSource(m, n, 1300 + i, "lowrank", dtype=dtype, signal_rank=min(16, m, n), noise=0.01) for i, (m, n) in enumerate(shapes)]
    W0 = [wl.make_weight(m, n, 1320 + i, dtype) for i, (m, n) in enumerate(shapes)]
    Wd = [lay(w.cuda()) for w in W0]
    opt = gb.GaLore(Wd, rank, auto_refresh=False, weight_decay=0.01, workspace_factor=2)  # room for 16 tensors in a launch
    opt.set_fused_adam(fused)
    oracles = []
    for i, (m, n) in enumerate(shapes):
        P = wl.random_orthonormal(min(m, n), rank, 1340 + i).to(wl.TORCH_DTYPE[dtype])
        opt.proj[i].copy_(P)
        o = orc.GaLoreTensor(to64(W0[i]), rank, scale=f32(0.25), beta1=f32(0.9), beta2=f32(0.999), eps=f32(1e-8), dtype=dtype,
                             weight_decay=f32(0.01), auto_refresh=False)
        o.set_projector(to64(P))
        if dtype == "f32":
            gen = torch.Generator().manual_seed(1360 + i)
            opt.M[i].copy_(0.01 * torch.randn(opt.M[i].shape, generator=gen))
            opt.V[i].copy_(1e-5 * (0.5 + torch.rand(opt.V[i].shape, generator=gen)))
            o.M[:] = to64(opt.M[i])
            o.V[:] = to64(opt.V[i])
        oracles.append(o)
    for step in range(steps):
        G = [s.grad(step) for s in srcs]
        if adam_launches is not None:
            gb.galore_profile_start(opt.ctx)
        (opt.step_static if static else opt.step)(Wd, [lay(g.cuda()) for g in G], lr)
        if adam_launches is not None:
            assert gb.galore_profile_stop(opt.ctx)["adam"][1] == adam_launches
        torch.cuda.synchronize()
        for i, o in enumerate(oracles):
            o.step(to64(G[i]), lr)
            assert relF(to64(opt.M[i]), o.M) <= 1e-5, (step, i, shapes[i])
            assert relF(to64(opt.V[i]), o.V) <= 1e-5, (step, i, shapes[i])
            if dtype == "f32":
                assert relF(to64(Wd[i]), o.W) <= 1e-5, (step, i, shapes[i])
            else:
                check_bf16_weights(to64(Wd[i]), o.W, to64(W0[i]), step + 1, lr, 0.25, where=(step, i, shapes[i]))
    opt.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rank", [8, 63, 65])
def test_tile_edges_and_ragged_contractions(dtype, rank):
    _steps([(65, 127), (127, 65), (129, 130), (131, 191), (193, 128), (72, 72)], rank, dtype)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_rows_at_any_element_offset(dtype):
    _steps([(130, 257), (257, 130), (515, 519)], 33, dtype, pad=3)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("shapes,rank", [([(513, 521)], 24), ([(521, 513)], 9), ([(1030, 1024)], 40), ([(512, 600), (1100, 777)], 31)])
def test_contractions_in_pieces(dtype, shapes, rank):
    # few tiles and contractions of 512 and more: 2 to 4 pieces, the last one ragged, summed by the workgroup that forms them (bf16: 2 and 3 in one call leave as slabs)
    _steps(shapes, rank, dtype, adam_launches=1 if dtype == "bf16" and len(shapes) == 2 else 0)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("shapes,rank", [([(2052, 2100)], 33), ([(2100, 2052)], 40), ([(2049, 2051)], 130), ([(2060, 2055), (2055, 2300)], 41)])
@pytest.mark.parametrize("pad", [0, 3])
def test_pieces_summed_by_the_adam_kernel(dtype, shapes, rank, pad):
    # contractions above 2048: slabs, whatever the dtype; each R has 64 Ki entries and more, so that Adam would run in the projection were they whole
    _steps(shapes, rank, dtype, pad=pad, steps=1, adam_launches=1)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("fused", [False, True])
def test_adam_in_the_epilogue(dtype, fused):
    # 61 x 1101 entries and more run the update block in the epilogue by themselves, the small tensor only when asked to
    _steps([(300, 1101), (1101, 300), (67, 71)], 61, dtype, fused=fused)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("shape,rank,count", [((130, 1411), 130, 16), ((1411, 130), 130, 16), ((72, 2049), 70, 16)])
def test_larger_tiles(dtype, shape, rank, count):
    # 16 tensors: 384 tiles of 128 x 128 (or, with 70 rows, 528 of 128 x 64) in the projection, W in 128 x 64 tiles
    shapes = [shape] * count
    assert _tile(_projection(shapes, rank)) == ((128, 64) if rank == 70 else (128, 128)) and _tile(_update(shapes, rank), update=True) == (128, 64)
    _steps(shapes, rank, dtype, steps=1)


def test_larger_tiles_of_the_weight_update_with_a_long_contraction():
    # r = 257: 396 tiles of 128 x 128 and five K steps, the last of a single element
    assert _tile(_update([(261, 1300)] * 12, 257), update=True) == (128, 128)
    _steps([(261, 1300)] * 12, 257, "bf16", steps=1)


# One tensor with enough tiles by itself: rank, short and long side of no multiple of the tile, of the K step or of a 16-byte piece;
# the tile of its projection (with Adam in the epilogue: whole contractions, more than 64 Ki entries) and of its weight update.
LONE = [(129, 300, 22531, (128, 128), (128, 64)), (65, 131, 32003, (128, 64), (128, 64)), (130, 203, 21251, (128, 64), (128, 64)),
        (257, 259, 15002, (128, 128), (128, 128)), (66, 68, 8200, (64, 64), (64, 64))]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("wide", [True, False])
@pytest.mark.parametrize("rank,k,l,proj,update", LONE)
def test_every_tile_with_adam_and_weight_update(rank, k, l, proj, update, wide, dtype):
    shape = (k, l) if wide else (l, k)
    assert _tile(_projection([shape], rank)) == proj and _tile(_update([shape], rank), update=True) == update
    _steps([shape], rank, dtype, steps=1, pad=3 if rank == 257 else 0)


def _entrywise(got, ref, bound):
    worst = float(((got.double() - ref).abs() / bound).max())
    assert worst <= 1.0, worst


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("wide", [True, False])
@pytest.mark.parametrize("rank,k,l,proj,update", LONE)
def test_every_tile_of_the_plain_product_and_the_weight_update(rank, k, l, proj, update, wide, dtype):
    # the stage calls, each entry against 64 bits: K fp32 additions of exact products are off by at most K 2^-24 of the sum of
    # magnitudes (to first order), a stored bf16 weight (8 significant bits) by another 2^-8 of itself at most
    m, n = (k, l) if wide else (l, k)
    assert _tile(_projection([(m, n)], rank)) == proj and _tile(_update([(m, n)], rank), update=True) == update
    g = torch.Generator(device="cuda").manual_seed(l)
    tdt = wl.TORCH_DTYPE[dtype]
    rand = lambda *s: strided(torch.randn(*s, generator=g, device="cuda").to(tdt), 5)
    G, P = rand(m, n), rand(k, rank)
    Pt = strided(P.t().contiguous(), 1)
    Rbuf = torch.full((rank if wide else m, (n if wide else rank) + 2), 7.0, device="cuda")
    R = Rbuf[:, :-2]
    gb.galore_project(Pt, G, R)
    a, b = (P.double().t(), G.double()) if wide else (G.double(), P.double())
    _entrywise(R, a @ b, (k if wide else n) * 2.0 ** -24 * 1.01 * (a.abs() @ b.abs()))
    assert bool((Rbuf[:, -2:] == 7.0).all())
    W, N = rand(m, n), rand(l, rank)
    a, b = (P.double(), N.double().t()) if wide else (N.double(), P.double().t())
    lr, scale, decay = f32(1e-2), f32(0.25), f32(0.125)
    ref = (1 - lr * decay) * W.double() - lr * scale * (a @ b)
    bound = rank * 2.0 ** -24 * 1.01 * lr * scale * (a.abs() @ b.abs()) + 2.0 ** -22 * (W.double().abs() + ref.abs()) + (2.0 ** -8 if dtype == "bf16" else 0) * ref.abs()
    gb.galore_project_back(P, N, W, lr, scale, decay)
    torch.cuda.synchronize()
    _entrywise(W, ref, bound * 1.01)


def test_large_tile_projection_of_a_padded_copy():
    # r above 512, rows of no multiple of 8 elements, at least 160 tiles of 256 x 256: G is copied with padded rows
    _steps([(640, 13829)], 640, "bf16", steps=1)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_static_scratch_holds_the_pieces(dtype):
    # slabs for the first two, pieces in one workgroup for the third
    _steps([(2052, 2100), (2100, 2052), (512, 600)], 40, dtype, adam_launches=1)
    _steps([(2052, 2100), (2100, 2052), (512, 600)], 40, dtype, static=True)


@pytest.mark.parametrize("m,n,rank,tile", [(300, 22531, 129, (128, 128)), (22531, 300, 129, (64, 64)), (203, 31939, 66, (128, 64)), (200, 8203, 66, (64, 64))])
def test_products_rounded_in_the_epilogue(m, n, rank, tile):
    # the two-sided step's T1 = P^T G (r x n) and T2 = Q N^T (n x r) are rounded to bf16 by the product that forms them
    t1, t2 = (rank, n, m), (n, rank, rank)
    assert max(_tile([t1]), _tile([t2])) == tile
    g = torch.Generator(device="cuda").manual_seed(n)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda")
    b16 = lambda x: x.float().to(torch.bfloat16).double()
    W, G = (0.02 * rand(m, n)).to(torch.bfloat16), rand(m, n).to(torch.bfloat16)
    opt = gb.GaLoreTwoSided(W, rank, auto_refresh=False, update_gap=1 << 30)
    opt.P.copy_(torch.linalg.qr(rand(m, rank))[0])
    opt.Q.copy_(torch.linalg.qr(rand(n, rank))[0])
    opt.M.copy_(rand(rank, rank))
    opt.V.fill_(1.0)
    opt.t = 1000
    P, Q, M, V, W0 = (x.double().clone() for x in (opt.P, opt.Q, opt.M, opt.V, W))
    lr = f32(1e-2)
    opt.step(W, G, lr)
    torch.cuda.synchronize()
    b1, b2, k = f32(0.9), f32(0.999), 1001
    R = b16(P.t() @ G.double()) @ Q
    M = b1 * M + (1 - b1) * R
    V = b2 * V + (1 - b2) * R * R
    N = b16((M / (1 - b1 ** k)) / ((V / (1 - b2 ** k)).sqrt() + 1e-8))
    T2 = b16(Q @ N.t())
    ref = W0 - lr * f32(0.25) * (P @ T2.t())
    # An entry of T1 (N, T2) within fp32 rounding of a boundary of bf16 falls the other way: one in a thousand, by 2^-8, 1.2e-4 in norm
    assert relF(to64(opt.M), M.cpu().numpy()) <= 5e-4 and relF(to64(opt.V), V.cpu().numpy()) <= 5e-4
    # every entry of the update to the roundings of N and T2 (2^-8 each at most) and what T1's do to N, the weight to its own
    _entrywise(W, ref, 1.01 * 2.0 ** -8 * ref.abs() + lr * f32(0.25) * 2.0 ** -6 * (P.abs() @ (Q.abs() @ N.abs().t()).t()))
