"""The small-tile GEMM (projection with K pieces or with Adam in its epilogue, weight update) against the fp64 oracle,
at the sizes where it can go wrong: one element to either side of a tile, contractions and rows of no multiple of
anything, the smallest sides it takes, the group sizes at which each tile shape and the K pieces are chosen."""
import pytest
import torch

from helpers import check_bf16_weights, f32, relF, strided, to64
from oracle import galore_oracle as orc
from paper_2403_03507_amd import binding as gb
from paper_2403_03507_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _steps(shapes, rank, dtype, steps=2, fused=False, pad=0, static=False):
    # M, V: fp32 sums of at most a few thousand products, 1e-5 as everywhere; fp32 W: 1e-5; bf16 W per entry.
    # fp32 tensors start from moments as earlier steps leave them: from zero moments the first N is R / (|R| + eps), where an entry of R
    # at rounding distance of zero (1e-9 here, against eps = 1e-8) moves W by up to lr alpha |P column| = 2.5e-3, i.e. 3e-4
    # of |W| = 8.6 for a 130 x 1411 weight; with V of about 1e-5 the same error of R moves N by 1e-6.
    lr = f32(1e-2)
    lay = (lambda t: strided(t, pad)) if pad else (lambda t: t)
    srcs = [wl.GradientSource(m, n, 1300 + i, "lowrank", dtype=dtype, signal_rank=min(16, m, n), noise=0.01) for i, (m, n) in enumerate(shapes)]
    W0 = [wl.make_weight(m, n, 1320 + i, dtype) for i, (m, n) in enumerate(shapes)]
    Wd = [lay(w.cuda()) for w in W0]
    opt = gb.GaLore(Wd, rank, auto_refresh=False, weight_decay=0.01)
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
        (opt.step_static if static else opt.step)(Wd, [lay(g.cuda()) for g in G], lr)
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
    # few tiles and contractions of 512 and more: 2 to 4 pieces, the last one ragged, summed by the Adam kernel
    _steps(shapes, rank, dtype)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("fused", [False, True])
def test_adam_in_the_epilogue(dtype, fused):
    # 61 x 1101 entries and more run the update block in the epilogue by themselves, the small tensor only when asked to
    _steps([(300, 1101), (1101, 300), (67, 71)], 61, dtype, fused=fused)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("shape,rank,count", [((130, 1411), 130, 16), ((1411, 130), 130, 16), ((72, 2049), 70, 16)])
def test_larger_tiles(dtype, shape, rank, count):
    # 16 tensors: 352 tiles of 128 x 128 (or, with 70 rows, 528 of 128 x 64) in the projection, W in 128 x 64 tiles
    _steps([shape] * count, rank, dtype, steps=1)


def test_larger_tiles_of_the_weight_update_with_a_long_contraction():
    # r = 257: more than 350 tiles of 128 x 128 and five K steps, the last of a single element
    _steps([(261, 1300)] * 12, 257, "bf16", steps=1)


def test_large_tile_projection_of_a_padded_copy():
    # r above 512, rows of no multiple of 8 elements, at least 160 tiles of 256 x 256: G is copied with padded rows
    _steps([(640, 13829)], 640, "bf16", steps=1)


def test_static_scratch_holds_the_pieces():
    _steps([(1030, 1024), (512, 600)], 40, "bf16", static=True)
