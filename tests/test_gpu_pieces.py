"""K pieces of small projections: how a call is divided into chains and launches does not show in the results."""
import pytest
import torch

from paper_2403_03507_amd import binding as gb

pytestmark = pytest.mark.gpu

# rank and tensors (rows, cols, dtype) of one call, short sides of 512 and more, so that contractions may be cut; weight updates and separate Adam
# passes of one step by setting of galore_set_concurrency
CALLS = {
    # one launch of 512 tiles of 64 x 64, or two (at this rank never three) of 256: a call long enough to be divided into chains; R of 32 Ki entries
    "eight 4096": (8, [(4096, 4096, torch.bfloat16)] * 8, {3: (2, 2), 2: (2, 2), 1: (1, 1)}),
    # three chains, twice, as the workspace takes ten tensors at a time: the other eight are six more of the first block of 16 (whole contractions) and the two of
    # the next, of 132 and 44 tiles, which are cut, in slabs (K > 2048; the other follows)
    "eighteen": (256, [(520, 20000, torch.bfloat16)] * 16 + [(2051, 2112, torch.bfloat16), (520, 700, torch.bfloat16)], {3: (6, 2), 2: (4, 2), 1: (2, 1)}),
    # slabs of both dtypes and both sides
    "slabs": (33, [(2052, 2100, torch.bfloat16), (2100, 2052, torch.float32), (2300, 2055, torch.bfloat16), (2052, 2112, torch.float32)], {3: (2, 2), 2: (2, 2), 1: (2, 2)}),
    # one chain: 64 fp32 tiles cut into 4 pieces, in one workgroup each, and 23 of bf16 in 3 and 2, which leave as slabs
    "mixed": (40, [(512, 640, torch.float32), (1300, 520, torch.float32), (768, 777, torch.bfloat16), (640, 512, torch.bfloat16), (2050, 600, torch.float32)],
              {3: (2, 1), 2: (2, 1), 1: (2, 1)}),
    # more tensors than a launch takes, both dtypes
    "twenty": (32, [(512, 2048, torch.float32), (2048, 512, torch.bfloat16)] * 10, None),
}


@pytest.mark.parametrize("name", list(CALLS))
def test_chains_workspaces_and_the_static_array_give_the_same_bits(name):
    rank, tensors, launches = CALLS[name]
    g = torch.Generator(device="cuda").manual_seed(17)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda")
    W0 = [(0.02 * rand(m, n)).to(dt) for m, n, dt in tensors]
    G = [rand(m, n).to(dt) for m, n, dt in tensors]
    P = [torch.linalg.qr(rand(min(m, n), rank))[0] for m, n, _ in tensors]
    results = {}
    for variant in ("3 chains", "2 chains", "1 chain", "fused", "static", "overlap", "workspace x 4"):
        W = [w.clone() for w in W0]
        factor = 4 if variant in ("overlap", "workspace x 4") else 1
        nbytes = factor * 10 * 6 * 256 * 20000 if name == "eighteen" else None   # R and N of ten tensors
        opt = gb.GaLore(W, rank, update_gap=1 << 30, workspace_bytes=nbytes, workspace_factor=factor)
        for i, p in enumerate(P):
            opt.proj[i].copy_(p)
            opt.set_step(i, 7)
        if variant.endswith("chains") or variant == "1 chain":
            gb.galore_set_concurrency(opt.ctx, int(variant[0]))
        opt.set_fused_adam(variant == "fused")
        opt.set_call_overlap(2 if variant == "overlap" else 0)
        for step in range(2):
            counted = launches and step == 0 and "chain" in variant
            if counted:
                gb.galore_profile_start(opt.ctx)
            (opt.step_static if variant == "static" else opt.step)(W, G, 1e-3)
            if counted:
                stages = gb.galore_profile_stop(opt.ctx)
                assert (stages["back"][1], stages["adam"][1]) == launches[int(variant[0])], variant
        opt.join()
        torch.cuda.synchronize()
        results[variant] = W + [x.clone() for x in opt.M + opt.V]
        opt.close()
    for variant, out in results.items():
        for i, (a, b) in enumerate(zip(out, results["3 chains"])):
            assert torch.equal(a, b), (variant, i)
    assert not torch.equal(results["1 chain"][0], W0[0])


@pytest.mark.parametrize("d,f,rank,large", [(4096, 11008, 512, True), (4096, 11008, 256, True), (4096, 11008, 384, False), (2048, 5504, 512, True), (2048, 5461, 1024, False)])
def test_forked_chains_count_their_tiles_together(d, f, rank, large):
    # One layer in three chains of 100 to 130 tiles of 256 x 256 each: together enough for the large-tile kernel (whose Adam runs in
    # launches of its own here) or not (small tiles, which run Adam in their epilogue), as each is faster
    shapes = [(d, d)] * 4 + [(d, f)] * 2 + [(f, d)]
    W = [torch.zeros(m, n, dtype=torch.bfloat16, device="cuda") for m, n in shapes]
    G = [torch.full((m, n), 0.01, dtype=torch.bfloat16, device="cuda") for m, n in shapes]
    opt = gb.GaLore(W, rank, update_gap=1 << 30, auto_refresh=False)
    gb.galore_profile_start(opt.ctx)
    opt.step(W, G, 1e-3)
    stages = gb.galore_profile_stop(opt.ctx)
    assert stages["project_left"][1] == stages["back"][1] == 3   # three chains
    assert (stages["adam"][1] > 0) == large, stages
    opt.close()


# Steps by estimate between 150 and 190 us: a second chain where one chain leaves a second round of 128 x 128 tiles (512 a round) nearly empty
# (2048: 579, 1801: 531, two layers of 1536: 576) or takes large tiles alone (r = 384), not with one round (1792 at r = 352: 510, 2048 at r = 256: 386), on large
# tiles either way (r = 448), with a rank of no multiple of 64 beside large tiles (r = 400), or in fp32
@pytest.mark.parametrize("layers,d,f,rank,dtype,chains", [
    (1, 2048, 5504, 288, "bf16", 2), (1, 1801, 4871, 333, "bf16", 2), (2, 1536, 4096, 160, "bf16", 2), (1, 1792, 4864, 384, "bf16", 2), (1, 1792, 4864, 352, "bf16", 1),
    (1, 1664, 4480, 448, "bf16", 1), (1, 1792, 4864, 400, "bf16", 1), (1, 2048, 5504, 256, "bf16", 1), (1, 1024, 2736, 200, "f32", 1)])
def test_chains_of_a_short_step(layers, d, f, rank, dtype, chains):
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    shapes = ([(d, d)] * 4 + [(d, f)] * 2 + [(f, d)]) * layers
    g = torch.Generator(device="cuda").manual_seed(rank)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda").to(tdt)
    W0, G, P = [0.02 * rand(*s) for s in shapes], [rand(*s) for s in shapes], [rand(min(s), rank) / 64 for s in shapes]
    out, launches = [], []
    for lanes in (1, 3):
        W = [w.clone() for w in W0]
        opt = gb.GaLore(W, rank, update_gap=1 << 30, auto_refresh=False)
        gb.galore_set_concurrency(opt.ctx, lanes)
        for i, p in enumerate(P):
            opt.proj[i].copy_(p)
            opt.V[i].fill_(1.0)
            opt.set_step(i, 1000)
        gb.galore_profile_start(opt.ctx)
        for _ in range(2):
            opt.step(W, G, 1e-3)
        launches.append(gb.galore_profile_stop(opt.ctx)["back"][1])
        torch.cuda.synchronize()
        out.append(W + [x.clone() for x in opt.M + opt.V])
        opt.close()
    assert launches == [2, 2 * chains]
    for i, (a, b) in enumerate(zip(*out)):
        # K pieces of large tiles may differ between the settings (fp32 rounding of R); short sides of no multiple of 64 and ranks that fill no large tile never take them
        if rank == 384:
            assert float((a.double() - b.double()).norm() / b.double().norm()) <= (1e-6 if a.dtype == torch.float32 else 1e-4), i
        else:
            assert torch.equal(a, b), i
