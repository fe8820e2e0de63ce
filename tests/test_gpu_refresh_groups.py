"""A tensor's projector is the same bits alone and in any group of tensors: what else is refreshed, and how many of them the
workspace lets share a launch, does not show."""
import pytest
import torch

from paper_2403_03507_amd import binding as gb

pytestmark = pytest.mark.gpu

GROUPS = {
    # ranks above half of one short side and not of the others: the third orthonormalisation pass is the tensor's own
    "passes": (64, [(100, 300, torch.float32), (300, 400, torch.float32), (400, 128, torch.bfloat16), (127, 200, torch.bfloat16), (64, 90, torch.float32)]),
    "passes at 256": (256, [(512, 600, torch.bfloat16), (1024, 1100, torch.bfloat16), (256, 700, torch.bfloat16), (600, 511, torch.float32)]),
    # enough tiles together for the general kernel of the Gram matrix, few alone
    "gram f32": (16, [(2048, 2100, torch.float32)] * 5 + [(512, 600, torch.float32)]),
    "gram bf16": (16, [(2048, 2100, torch.bfloat16)] * 3 + [(2100, 2048, torch.bfloat16)] * 2),
    # 16 x 10 tiles of 256 x 256: the large-tile kernel for the split products, small tiles alone
    "large products": (256, [(2560, 2600, torch.bfloat16)] * 16),
    # products of 352 tiles of 128 x 128 and of 528 of 128 x 64, on 64 x 64 tiles alone, in fp32 and (short sides of a multiple of 32) split
    "tiles 128 x 128": (129, [(1301, 1310, torch.float32)] * 16),
    "tiles 128 x 128 split": (129, [(1312, 1320, torch.bfloat16)] * 16),
    "tiles 128 x 64": (70, [(2051, 2060, torch.float32)] * 16),
    # the Householder path
    "rank 300": (300, [(512, 600, torch.bfloat16), (1024, 700, torch.bfloat16), (320, 400, torch.float32)]),
}


@pytest.mark.parametrize("kind", ["noise", "low rank"])
@pytest.mark.parametrize("name", list(GROUPS))
def test_group_and_lone_refresh_agree_bit_for_bit(name, kind):
    rank, tensors = GROUPS[name]
    g = torch.Generator(device="cuda").manual_seed(23)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda")
    # low rank: columns of the iteration block depend on each other and are replaced
    G = [(rand(m, n) if kind == "noise" else rand(m, 5) @ rand(5, n)).to(dt) for m, n, dt in tensors]
    group = gb.GaLore(G, rank, refresh_iters=3, seed=9, workspace_factor=2)
    lone = gb.GaLore(G, rank, refresh_iters=3, seed=9)
    group.refresh(G)
    for i, x in enumerate(G):
        lone.refresh([x], first=i)
    torch.cuda.synchronize()
    for i in range(len(G)):
        assert torch.equal(group.proj[i], lone.proj[i]) and torch.equal(group.proj_t[i], lone.proj_t[i]), (name, i)
        assert bool(group.proj[i].isfinite().all())
    group.close()
    lone.close()
